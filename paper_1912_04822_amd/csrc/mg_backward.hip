// Step 6 of the path: the backward pass (GridMaker section: "computes atomic
// gradients").  With L = sum G*out, u = x'_a - p, d = |u|, x = d/r:
//   dL/dx'_a = sum_p G[p] rho'(x) u / (r d)
//            = (1/r^2) sum_p G[p] f(x^2) u,
//   f = -4 exp(-2x^2)            x <= g      (rho' = -4x exp(-2x^2))
//     = 2A (1 - c/x)             g < x < c   (rho' = 2A (x - c))
//     = 0                        x >= c
// (dividing rho' by x removes the square root from the Gaussian branch and makes
// d = 0 contribute exactly 0 through u = 0).  The kernels sum -f/4 instead,
//   -f/4 = exp(-2x^2)            x <= g
//        = (A/2) (c/x - 1)       g < x < c     (at most exp(-2g^2) <= 1 there)
//        = 0                     x >= c
// as a product without a select (see reduce_slot), and the factor -4 goes into the scale
// applied once per atom.  The gradient with respect to the caller's
// coordinates is R^T times that sum.
//
// One wavefront per atom record (four records per workgroup, no barrier).  The
// work items are "slots": runs of four voxels along z in the grid rows (x-plane,
// y) of the atom's cutoff box, read with one 16-byte load each.  Only the rows
// that meet the cutoff sphere are visited, and a row's slots start at the first
// voxel of its chord (so a chord of L voxels takes ceil(L/4) slots, wherever it
// lies; the last slot is pulled back into the row if need be -- voxels outside the
// sphere add exactly 0): per group of 128
// rows every lane works out the chord of its two rows, a prefix sum over
// the lanes numbers the live slots, and slot s finds its row through a byte
// array in LDS (the first slot of each lane's rows is marked with the lane, a
// running maximum over the slots gives the owner) and one register exchange.
// Index types are bound by the arrival of the scattered lines (50 x 2040 atoms, 28 x 48^3: 372 MB of 128-byte
// lines from HBM, 5.4 TB/s; wavefronts wait 59 % of their time) and by vector instruction issue (0.049 of
// 0.069 ms; a third of the instructions the density, the rest finding rows and slots).  The three partial sums
// are reduced across the wavefront together, in a fixed order (wave_sum4; with the slope as a
// product instead of a select 76 instead of 78.6 us a call).  Records are grouped by
// channel (and, within a channel, by x-plane), so neighbouring wavefronts read
// the same part of the same channel volume.
// (Consecutive lanes take consecutive slots of a row, so a 64-lane load touches about 25
// lines.  Two atoms per wavefront with every lane walking the slots of its own rows -- no
// slot list at all, a quarter fewer instructions -- touches 64 lines per load and measured
// 74-100 us against 62 us.)
#include <cmath>

#include "mg_common.h"
#include "mg_wave.h"
#include "mg_xform.h"

namespace mg {

namespace {

struct BwdParams {
    GridSpec gs;
    RawInputs raw;
    const float4 *rec;
    const int *idx;
    const int4 *meta;
    const float *rot;
    const int *rchan;       // [B][N] channel of each record (index types)
    const int *chan_order;  // [B][T] channels in order of radius (vector types)
    const float *weights;
    const float *radii;
    const float *gcen;
    const unsigned char *alive;     // [B][N] 1: the atom has a live record
    const unsigned *tag;            // what the workspace's tables were made for
    unsigned expect_tag;            // != 0: do nothing unless *tag equals it (calls on prepared tables)
    const void *G;          // upstream gradient grid, float or double
    float *grad_coords;
    float *grad_weights;
    int subgrids, N, T;
    unsigned wgs_per_example;       // workgroups (of four records) per example
    unsigned units, share;          // workgroups in all; per XCD (ceil(units / 8))
    unsigned long long wg_magic;    // ceil(2^64 / wgs_per_example), 0 if that is 1
    float k;                // 2 log2(e)
    float ng2k, nfA, fAc;   // -g^2 k, -2g^2, 2g^2 c
    float tg, tc;           // vector types: 2g, 2g c
};

// a value that is the same in all lanes, kept in a scalar register
__device__ inline float uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// 1 / r (the hardware's approximation, 1 ulp), small enough to be squared, and for its square times
// kTinyDistance2 to be nothing: an atom on a voxel has rho = 1 there however small its radius
__device__ inline float scale_of(float r)
{
    return fminf(__builtin_amdgcn_rcpf(r), 1.0e14f);
}

struct Box {
    int ilo, jlo, seg0;
    int np, nr, ns;
    int klo, khi;
};

constexpr int kSlotCap = 1024;      // live slots of a group of 128 rows: at most 8 per row
constexpr int kMaxCulledSegs = 8;   // boxes with more z-segments per row take the plain loop
constexpr int kMaxCulledRows = 32768;   // ... and so do boxes with more rows: below that, row / nr by a
                                        // float reciprocal is exact (error <= rows * 2e-7 < 0.5)

// grid points within `reach` of the atom along each axis, padded by 1e-3 steps
__device__ inline bool atom_box(const GridSpec &gs, float reach, const float4 &a, float ox, float oy,
                                float oz, Box &bx)
{
    const float hv = reach * gs.inv_res + 1.0e-3f;
    const float fx = (a.x - ox) * gs.inv_res, fy = (a.y - oy) * gs.inv_res,
                fz = (a.z - oz) * gs.inv_res;
    const int D = gs.D;
    const int ilo = max(0, (int)ceilf(fx - hv)), ihi = min(D - 1, (int)floorf(fx + hv));
    const int jlo = max(0, (int)ceilf(fy - hv)), jhi = min(D - 1, (int)floorf(fy + hv));
    const int klo = max(0, (int)ceilf(fz - hv)), khi = min(D - 1, (int)floorf(fz + hv));
    bx.ilo = ilo; bx.jlo = jlo; bx.seg0 = klo >> 2; bx.klo = klo; bx.khi = khi;
    bx.np = ihi - ilo + 1; bx.nr = jhi - jlo + 1; bx.ns = (khi >> 2) - (klo >> 2) + 1;
    return bx.np > 0 && bx.nr > 0 && bx.ns > 0 && khi >= klo;
}

// Accumulate over one channel volume: (sx, sy, sz) += sum G (-f/4) u, distances in Angstrom (differences of
// nearby numbers and whole steps of the spacing: a scaled spacing, rounded, times a row's length was the largest
// error of a gradient).  With E = exp(-2 min(x, g)^2) = exp2(max(-k d^2 / r^2, -g^2 k)), k = 2 log2(e),
//   -f/4 = E clamp(2g^2 (c r / d - 1), 0, 1)
// (2g^2 (c/g - 1) = 1, and A = 4 g^2 exp(-2g^2)): no select.
// One slot: the four voxels k4 .. k4+3 of the grid row at float offset `row_off` of the
// channel (a channel has at most 2^30 floats); ux, uy: the row's x and y distance.
struct SlotData {
    float gv[4];        // upstream gradient of the four voxels
    float ux, uy;
    int k4;
};

// 16-byte vectors that are only aligned like their elements (one wide load all the same)
typedef float Float4E __attribute__((ext_vector_type(4), aligned(4)));
typedef double Double2E __attribute__((ext_vector_type(2), aligned(8)));

// STREAM: the loads carry the non-temporal hint, so the lines they bring in do not settle in the
// memory-side cache.  The index-type kernel's reuse of a line is between neighbouring wavefronts,
// within microseconds, in L2 (1.38 reads from HBM per line), and the grid usually arrives
// behind hundreds of MB that an earlier kernel has just written and that still sit dirty in
// that cache: lines that settle there push those out, and the reads then wait behind the
// write-backs.  Kernel on the 48^3 batch, with / without the hint: 70 / 100 us right after a forward call, 71 / 72
// after a read-only pass over another buffer, 68 / 62 in a loop of nothing but backward calls (where the
// lines of the call before would otherwise still be cached); without: as measured with an earlier body.
// The vector-typed kernel visits every line once per group of channels and atoms far apart in time share
// lines: 1.9 ms with the hint, 0.76 without.
template <bool ALIGNED, bool STREAM, typename GT>
__device__ inline void load_slot(const BwdParams &p, const GT *Gc, unsigned row_off, int k4,
                                 float ux, float uy, SlotData &d)
{
    const GT *src = Gc + (row_off + (unsigned)k4);
    if (ALIGNED) {      // the four voxels lie in the row; k4 need not be a multiple of 4
        if (sizeof(GT) == 8) {      // a grid of doubles: two 16-byte loads, narrowed
            const Double2E *s2 = reinterpret_cast<const Double2E *>(src);
            const Double2E lo = STREAM ? __builtin_nontemporal_load(s2) : s2[0];
            const Double2E hi = STREAM ? __builtin_nontemporal_load(s2 + 1) : s2[1];
            d.gv[0] = (float)lo.x; d.gv[1] = (float)lo.y; d.gv[2] = (float)hi.x; d.gv[3] = (float)hi.y;
        } else {
            const Float4E *s4 = reinterpret_cast<const Float4E *>(src);
            const Float4E g4 = STREAM ? __builtin_nontemporal_load(s4) : *s4;
            d.gv[0] = g4.x; d.gv[1] = g4.y; d.gv[2] = g4.z; d.gv[3] = g4.w;
        }
    } else if (p.gs.D >= 4) {
        // Rows of any length: a slot that reaches past the row's end is read from the row's last four
        // voxels, and those of them that belong to the slot before count as 0.
        // (Four loads of a voxel each before: 178 instead of 85 us a call on 50 x 28 x 47^3.)
        const int back = max(k4 - (p.gs.D - 4), 0);
        load_slot<true, STREAM>(p, Gc, row_off, k4 - back, ux, uy, d);
#pragma unroll
        for (int u = 0; u < 3; ++u) d.gv[u] = u < back ? 0.0f : d.gv[u];
        return;
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            d.gv[u] = (k4 + u < p.gs.D) ? (float)(STREAM ? __builtin_nontemporal_load(src + u) : src[u]) : 0.0f;
    }
    d.ux = ux; d.uy = uy; d.k4 = k4;
}

struct ChannelCoef {
    float nr2;          // -k / r^2
    float fq;           // 2 g^2 c r
};

__device__ inline void reduce_slot(const BwdParams &p, const ChannelCoef &cc, float az, const SlotData &d,
                                   float &sx, float &sy, float &sz)
{
    const float ux = d.ux, uy = d.uy;
    const float *gv = d.gv;
    const float b2 = fmaf(ux, ux, uy * uy);
    const float uz0 = fmaf(-(float)d.k4, p.gs.res, az);
    float fsum = 0.0f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const float uz = fmaf(-(float)u, p.gs.res, uz0);
        const float d2 = fmaf(uz, uz, b2);
        const float e = __builtin_amdgcn_exp2f(fmaxf(d2 * cc.nr2, p.ng2k));
        const float ft = __builtin_amdgcn_fmed3f(fmaf(cc.fq, __builtin_amdgcn_rsqf(d2), p.nfA), 0.0f, 1.0f);
        const float gf = gv[u] * e * ft;
        fsum += gf;
        sz = fmaf(gf, uz, sz);
    }
    sx = fmaf(fsum, ux, sx);
    sy = fmaf(fsum, uy, sy);
}

// Every slot of the box (boxes with very many segments per row).
template <bool ALIGNED, typename GT>
__device__ inline void reduce_channel_box(const BwdParams &p, const GT *Gc, const float4 &a,
                                          const ChannelCoef &cc, const Box &bx, float ox, float oy, float oz,
                                          float &sx, float &sy, float &sz)
{
    const GridSpec &gs = p.gs;
    const int per_plane = bx.nr * bx.ns;
    const int slots = bx.np * per_plane;        // at most D^3 / 4 < 2^31
    // distances of the box's first row
    const float ux0 = a.x - (ox + (float)bx.ilo * gs.res), uy0 = a.y - (oy + (float)bx.jlo * gs.res);
    for (int sl = (int)(threadIdx.x & 63u); sl < slots; sl += 64) {
        // integer division: a box of hundreds of voxels per side has more slots than a float
        // holds exactly
        const int pi = sl / per_plane;
        const int rem = sl - pi * per_plane;
        const int row = rem / bx.ns;
        const int seg = rem - row * bx.ns;
        const float ux = fmaf(-(float)pi, gs.res, ux0), uy = fmaf(-(float)row, gs.res, uy0);
        SlotData d;
        load_slot<ALIGNED, false>(p, Gc, (unsigned)((bx.ilo + pi) * gs.D + bx.jlo + row) * (unsigned)gs.D,
                           (bx.seg0 + seg) << 2, ux, uy, d);
        reduce_slot(p, cc, a.z - oz, d, sx, sy, sz);
    }
}

// Only the slots that meet the cutoff sphere.  `marks` is this wavefront's kSlotCap bytes of
// LDS, all zero on entry and on return.
// The channel is G + t * D3 (index types: t comes with the record, from the workspace).
template <bool ALIGNED, typename GT>
__device__ inline void reduce_channel(const BwdParams &p, const GT *G, int t, size_t D3,
                                      const float4 &a, float r, const Box &bx, float ox, float oy,
                                      float oz, unsigned char *marks, float &sx, float &sy,
                                      float &sz)
{
    // reciprocals by the hardware approximation (1 ulp): the row split below has a margin of
    // 0.5/nr and the scale enters the result with a relative error of 1e-7
    const float inv_r = scale_of(r), reach = r * p.gs.c, reach2 = reach * reach;
    const ChannelCoef cc = {-(p.k * inv_r) * inv_r, p.fAc * r};
    if (bx.ns > kMaxCulledSegs || bx.np * bx.nr > kMaxCulledRows) {
        reduce_channel_box<ALIGNED>(p, G + (size_t)t * D3, a, cc, bx, ox, oy, oz, sx, sy, sz);
        return;
    }
    const GridSpec &gs = p.gs;
    const int lane = (int)(threadIdx.x & 63u);
    const int rows = bx.np * bx.nr;
    const float inv_nr = __builtin_amdgcn_rcpf((float)bx.nr);
    const float az = a.z - oz, fz = az * gs.inv_res;    // fz: the atom's z in grid steps
    // distances of the box's first row
    const float ux0 = a.x - (ox + (float)bx.ilo * gs.res), uy0 = a.y - (oy + (float)bx.jlo * gs.res);
    const unsigned D = (unsigned)gs.D;
    const unsigned off0 = ((unsigned)bx.ilo * D + (unsigned)bx.jlo) * D;   // the box's first row
    for (int row0 = 0; row0 < rows; row0 += 128) {
        // this lane's two rows of the group: which segments meet the sphere
        int cnt[2] = {0, 0}, slo[2] = {0, 0};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int row = row0 + 2 * lane + q;
            if (row < rows) {
                const int pi = (int)(((float)row + 0.5f) * inv_nr);
                const int jr = row - pi * bx.nr;
                const float ux = fmaf(-(float)pi, gs.res, ux0), uy = fmaf(-(float)jr, gs.res, uy0);
                const float h2 = reach2 - (ux * ux + uy * uy);
                if (h2 > 0.0f) {
                    // half chord in grid steps; the pad only adds voxels that contribute 0
                    const float hv = __builtin_amdgcn_sqrtf(h2) * gs.inv_res + 1.0e-3f;
                    const int klo = max(bx.klo, (int)ceilf(fz - hv));
                    const int khi = min(bx.khi, (int)floorf(fz + hv));
                    if (khi >= klo) {       // 4-voxel slots from the chord's first voxel, kept inside the row
                        cnt[q] = (khi - klo + 4) >> 2;
                        slo[q] = ALIGNED ? min(klo, gs.D - 4 * cnt[q]) : klo;
                    }
                }
            }
        }
        const int mine = cnt[0] + cnt[1];
        const int incl = wave_inclusive_scan(mine);
        const int total = bcast(incl, 63);
        const int excl = incl - mine;
        if (mine > 0) marks[excl] = (unsigned char)(lane + 1);
        // what a slot needs of its owner: first slot (11 bits) and slots of row 0 in one word,
        // the first voxel of row 0 and of row 1 (16 bits each) in another
        const int word = excl | (cnt[0] << 11), starts = slo[0] | (slo[1] << 16);
        lds_sync();
        asm volatile("" : "+v"(t));     // nothing above waits for t
        const GT *Gc = G + (size_t)t * D3;
        // Round k works on slots 64k .. 64k+63, one per lane.  (Issuing the reads of two or three
        // rounds before the arithmetic of the first was measured slower -- 69 against 62 us with
        // the gradient grid partly in the memory-side cache, 102 against 100 us with a grid that
        // has to come from HBM: more requests in flight do not shorten a wavefront's chain of
        // dependent trips, and instruction issue comes before the lines as the bound.)
        int carry = 0;
        for (int base = 0; base < total; base += 64) {
            const int sidx = base + lane;
            int v = sidx < total ? (int)marks[sidx] : 0;
            v = max(wave_inclusive_max(v), carry);      // owner of slot 0 is marked: v >= 1
            carry = bcast(v, 63);
            const int owner = v - 1;
            const int w = __builtin_amdgcn_ds_bpermute(owner << 2, word);
            const int st = __builtin_amdgcn_ds_bpermute(owner << 2, starts);
            if (sidx < total) {
                const int o = sidx - (w & 0x7ff);
                const int c0 = w >> 11;
                const int q = o >= c0 ? 1 : 0;
                const int k4 = q ? (st >> 16) + 4 * (o - c0) : (st & 0xffff) + 4 * o;
                const int row = row0 + 2 * owner + q;
                const int pi = (int)(((float)row + 0.5f) * inv_nr);
                const int jr = row - pi * bx.nr;
                const float ux = fmaf(-(float)pi, gs.res, ux0), uy = fmaf(-(float)jr, gs.res, uy0);
                SlotData d;
                load_slot<ALIGNED, true>(p, Gc, off0 + ((unsigned)pi * D + (unsigned)jr) * D, k4, ux,
                                   uy, d);
                reduce_slot(p, cc, az, d, sx, sy, sz);
            }
        }
        lds_sync();
        if (mine > 0) marks[excl] = 0;
        lds_sync();
    }
}

// ---------------------------------------------------------------------------
// Vector types: kChanGroup channels of one atom in one pass.  The channels differ only in radius, so
// the slots are found once, for the widest sphere of the group.  Beyond channel q's own cutoff f and rho
// are 0 by their formulas, so the voxels the narrower spheres do not reach add nothing.
// What depends on the channel's radius and the atom's weight is worked out once per atom, lane l for the
// channel of rank l (the tables' ranking where there are tables), and read into scalar registers group by
// group; the four weight sums of a group are reduced together (19 instructions instead of 52) and
// kept by the lanes of their channels, so that an atom's weight gradients leave in one store.  Distances
// are in Angstrom for all groups.  50 x 2040 atoms, 28 x 48^3: 778 instead of 907 us a call; 8 x 12 channels
// 87 / 95; 2 x 100 channels of 32^3 126 / 165; few channels alike.  Of 439 sizes 31 got slower, by 2 to 3 % at 0.25 A and few atoms
// (30 x 100, 28 x 64^3 449 / 437), by 11 % at most (20 x 500, 40 x 48^3 at 0.375 A 494 / 446): the same lines are asked of
// L2 by fewer instructions, but the wavefronts in flight spread over more groups and L2 misses more of them (2.34e7 / 1.91e7).
// Bound by the lines that the L2s deliver, 128 bytes for every 26 of a chord (1.39e8 of them, 17.8 GB a launch,
// 23.3 TB/s: the loads alone take 740 us; the L1s wait for L2 in two thirds of the kernel's 760 us) and by vector
// instruction issue (0.55 of the 0.76 ms; wavefronts wait 29 % of their time for memory and 44 % for their turn to issue).
// Measured and not kept: the slots of an atom listed once in LDS for all its channels, in shells of the
// row's distance, so that rounds of far slots take the tail's half of the density only: 33 % fewer
// load instructions and 20 % fewer vector instructions, and no faster (792 us a call, lines and waits not counted; 0.25 A: 332 against 256; only 24^3
// at 1 A gains, 225 against 255).
// ---------------------------------------------------------------------------
constexpr int kChanGroup = 4;
constexpr float kTinyDistance2 = 1.0e-37f;      // added to squared distances whose roots are divided by (see scale_of)

struct GroupCoef {              // wave-uniform
    float nr2[kChanGroup];          // -k / r_q^2
    float fq[kChanGroup];           // 2 g^2 c r_q: tail of -f/4
    float tq[kChanGroup];           // -2g / r_q: root of the tail of rho
    float cq[kChanGroup];           // -4 w_q / r_q^2: channel q's share of the coordinate sums
    unsigned live;                  // bit q: r_q > 0
};

// The four voxels from float `off` of the channel at Gc on, the first `back` of which count as 0.
template <bool ALIGNED, typename GT>
__device__ inline void load_voxels(const BwdParams &p, const GT *Gc, unsigned off, int back, float (&gv)[4])
{
    const GT *src = Gc + off;
    if (!ALIGNED && p.gs.D < 4) {           // (a row is one slot, from its first voxel)
#pragma unroll
        for (int u = 0; u < 4; ++u) gv[u] = u < p.gs.D ? (float)src[u] : 0.0f;
        return;
    }
    if (sizeof(GT) == 8) {      // a grid of doubles: two 16-byte loads, narrowed
        const Double2E *s2 = reinterpret_cast<const Double2E *>(src);
        const Double2E lo = s2[0], hi = s2[1];
        gv[0] = (float)lo.x; gv[1] = (float)lo.y; gv[2] = (float)hi.x; gv[3] = (float)hi.y;
    } else {
        const Float4E g4 = *reinterpret_cast<const Float4E *>(src);
        gv[0] = g4.x; gv[1] = g4.y; gv[2] = g4.z; gv[3] = g4.w;
    }
    if (!ALIGNED) {             // voxels that belong to the slot before count as 0
#pragma unroll
        for (int u = 0; u < 3; ++u) gv[u] = u < back ? 0.0f : gv[u];
    }
}

// One slot against the channels of a group; ux, uy: the distances of its row from the atom, uz0: that of its first
// voxel.
// The two branches of the density and of its slope are taken as a product without a select: with
// E = exp(-2 min(x, g)^2),
//   rho  = E clamp(2g (c - x), 0, 1)^2        (2g (c - g) = 1, and A = 4 g^2 exp(-2g^2))
//   -f/4 = E clamp(2g^2 (c/x - 1), 0, 1)      (2g^2 (c/g - 1) = 1)
// so the channels share one reciprocal square root per voxel (the distance is the square times that).
//   (sx, sy, sz) += sum_q cq sum G_q f_q u,  sv[q] += sum G_q rho_q
template <bool ALIGNED, bool WANT_W, bool ALL_LIVE, typename GT>
__device__ inline void reduce_slot_group(const BwdParams &p, const GT *const (&Gq)[kChanGroup], unsigned off, int back,
                                         float ux, float uy, float uz0, const GroupCoef &gc, float ng2k, float nfA,
                                         float tc, float &sx, float &sy, float &sz, float (&sv)[kChanGroup])
{
    const float b2 = fmaf(ux, ux, fmaf(uy, uy, kTinyDistance2));
    float gv[kChanGroup][4];
#pragma unroll
    for (int q = 0; q < kChanGroup; ++q)
        if (ALL_LIVE || (gc.live >> q) & 1u) load_voxels<ALIGNED>(p, Gq[q], off, back, gv[q]);
    float fsum = 0.0f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const float uz = fmaf(-(float)u, p.gs.res, uz0);
        const float x2 = fmaf(uz, uz, b2);
        const float rs = __builtin_amdgcn_rsqf(x2), d = x2 * rs;
        float F = 0.0f;
#pragma unroll
        for (int q = 0; q < kChanGroup; ++q) {
            if (!ALL_LIVE && !((gc.live >> q) & 1u)) continue;
            const float ge = gv[q][u] * __builtin_amdgcn_exp2f(fmaxf(x2 * gc.nr2[q], ng2k));
            const float ft = __builtin_amdgcn_fmed3f(fmaf(gc.fq[q], rs, nfA), 0.0f, 1.0f);
            F = fmaf(gc.cq[q], ge * ft, F);
            if (WANT_W) {
                const float tl = __builtin_amdgcn_fmed3f(fmaf(gc.tq[q], d, tc), 0.0f, 1.0f);
                sv[q] = fmaf(ge * tl, tl, sv[q]);
            }
        }
        fsum += F;
        sz = fmaf(F, uz, sz);
    }
    sx = fmaf(fsum, ux, sx);
    sy = fmaf(fsum, uy, sy);
}

// Every slot of the box that meets the sphere of radius `reach` about the atom (the same enumeration as
// reduce_channel; marks: this wavefront's kSlotCap bytes of LDS, zero on entry and return).
template <bool ALIGNED, bool WANT_W, bool ALL_LIVE, typename GT>
__device__ inline void reduce_group(const BwdParams &p, const GT *const (&Gq)[kChanGroup], const float4 &a, float reach,
                                    const Box &bx, float ox, float oy, float oz, unsigned char *marks,
                                    const GroupCoef &gc, float &sx, float &sy, float &sz, float (&sv)[kChanGroup])
{
    const GridSpec &gs = p.gs;
    const int lane = (int)(threadIdx.x & 63u);
    const unsigned D = (unsigned)gs.D;
    const float ux0 = a.x - (ox + (float)bx.ilo * gs.res), uy0 = a.y - (oy + (float)bx.jlo * gs.res);
    const float az = a.z - oz, fz = az * gs.inv_res;        // fz: the atom's z in grid steps
    const unsigned off0 = ((unsigned)bx.ilo * D + (unsigned)bx.jlo) * D;   // the box's first row
    float ng2k = p.ng2k, nfA = p.nfA, tc = p.tc;
    asm volatile("" : "+v"(ng2k), "+v"(nfA), "+v"(tc));
    // the slot of voxels k4 .. k4 + 3 of row (pi, jr) of the box
    const auto slot = [&](int pi, int jr, int k4) {
        const int back = ALIGNED ? 0 : max(k4 - max(gs.D - 4, 0), 0);      // reaches past the row's end
        k4 -= back;
        reduce_slot_group<ALIGNED, WANT_W, ALL_LIVE>(p, Gq, off0 + ((unsigned)pi * D + (unsigned)jr) * D + (unsigned)k4, back,
                                                     fmaf(-(float)pi, gs.res, ux0), fmaf(-(float)jr, gs.res, uy0),
                                                     fmaf(-(float)k4, gs.res, az), gc, ng2k, nfA, tc, sx, sy, sz, sv);
    };
    if (bx.ns > kMaxCulledSegs || bx.np * bx.nr > kMaxCulledRows) {     // a very large box: every slot of it
        const int per_plane = bx.nr * bx.ns;
        const int slots = bx.np * per_plane;        // at most D^3 / 4 < 2^31
        for (int sl = lane; sl < slots; sl += 64) {
            const int pi = sl / per_plane;          // integer division: exact for any box
            const int rem = sl - pi * per_plane;
            const int jr = rem / bx.ns;
            slot(pi, jr, (bx.seg0 + rem - jr * bx.ns) << 2);
        }
        return;
    }
    const int rows = bx.np * bx.nr;
    const float inv_nr = __builtin_amdgcn_rcpf((float)bx.nr);
    const float reach2 = fmaxf(reach * reach, kTinyDistance2);      // (the square of a very small reach is 0)
    for (int row0 = 0; row0 < rows; row0 += 128) {
        int cnt[2] = {0, 0}, slo[2] = {0, 0};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int row = row0 + 2 * lane + q;
            if (row < rows) {
                const int pi = (int)(((float)row + 0.5f) * inv_nr);
                const int jr = row - pi * bx.nr;
                const float ux = fmaf(-(float)pi, gs.res, ux0), uy = fmaf(-(float)jr, gs.res, uy0);
                const float h2 = reach2 - (ux * ux + uy * uy);
                if (h2 > 0.0f) {
                    const float hv = __builtin_amdgcn_sqrtf(h2) * gs.inv_res + 1.0e-3f;
                    const int klo = max(bx.klo, (int)ceilf(fz - hv));
                    const int khi = min(bx.khi, (int)floorf(fz + hv));
                    if (khi >= klo) {       // 4-voxel slots from the chord's first voxel, kept inside the row
                        cnt[q] = (khi - klo + 4) >> 2;
                        slo[q] = max(min(klo, gs.D - 4 * cnt[q]), 0);
                    }
                }
            }
        }
        const int mine = cnt[0] + cnt[1];
        const int incl = wave_inclusive_scan(mine);
        const int total = bcast(incl, 63);
        const int excl = incl - mine;
        if (mine > 0) marks[excl] = (unsigned char)(lane + 1);
        const int word = excl | (cnt[0] << 11), starts = slo[0] | (slo[1] << 16);
        lds_sync();
        int carry = 0;
        for (int base = 0; base < total; base += 64) {
            const int sidx = base + lane;
            int v = sidx < total ? (int)marks[sidx] : 0;
            v = max(wave_inclusive_max(v), carry);
            carry = bcast(v, 63);
            const int owner = v - 1;
            const int w = __builtin_amdgcn_ds_bpermute(owner << 2, word);
            const int st = __builtin_amdgcn_ds_bpermute(owner << 2, starts);
            if (sidx < total) {
                const int o = sidx - (w & 0x7ff);
                const int c0 = w >> 11;
                const int q = o >= c0 ? 1 : 0;
                const int row = row0 + 2 * owner + q;
                const int pi = (int)(((float)row + 0.5f) * inv_nr);
                slot(pi, row - pi * bx.nr, q ? (st >> 16) + 4 * (o - c0) : (st & 0xffff) + 4 * o);
            }
        }
        lds_sync();
        if (mine > 0) marks[excl] = 0;
        lds_sync();
    }
}

// The value of another lane of the same four: quad_perm [1,0,3,2] (0xB1) or [2,3,0,1] (0x4E).
template <int CTRL>
__device__ inline float quad_swap(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// Four sums over the wavefront at once, in a fixed order: sum (lane & 3) in every lane.
__device__ inline float wave_sum4(float a, float b, float c, float d)
{
    const int lane = (int)(threadIdx.x & 63u);
    const auto bits = [](float x) { return __float_as_int(x); };
    const bool odd = (lane & 1) != 0, upper = (lane & 2) != 0;
    // lane l keeps one of a pair and gets the neighbour's part of it
    const float ab = (odd ? b : a) + quad_swap<0xB1>(odd ? a : b);
    const float cd = (odd ? d : c) + quad_swap<0xB1>(odd ? c : d);
    float r = (upper ? cd : ab) + quad_swap<0x4E>(upper ? ab : cd);
    r += __int_as_float(__builtin_amdgcn_update_dpp(0, bits(r), 0x124, 0xf, 0xf, false));     // row_ror:4
    r += __int_as_float(__builtin_amdgcn_update_dpp(0, bits(r), 0x128, 0xf, 0xf, false));     // row_ror:8
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)bits(r), (unsigned)bits(r), false, false);
    r = __uint_as_float(h[0]) + __uint_as_float(h[1]);          // rows 0 + 1, rows 2 + 3
    const auto w = __builtin_amdgcn_permlane32_swap((unsigned)bits(r), (unsigned)bits(r), false, false);
    return __uint_as_float(w[0]) + __uint_as_float(w[1]);
}

// WANT_W: gradients of the weights are asked for (vector types).
template <bool VECTOR, bool ALIGNED, typename GT, bool FUSED, bool WANT_W = false>
__global__ __launch_bounds__(256, VECTOR ? (sizeof(GT) == 8 ? 5 : 6) : 1) void backward_kernel(BwdParams p)
{
    const GridSpec &gs = p.gs;
    // The kernel arguments the first loads need are fetched together (they are inputs of an
    // asm statement whose result, zero, enters the example index) instead of in several
    // dependent trips to the scalar cache.
    unsigned zero;
    asm("s_mov_b32 %0, 0"
        : "=s"(zero)
        : "s"((unsigned long long)p.meta), "s"((unsigned long long)p.rec),
          "s"((unsigned long long)p.idx), "s"((unsigned long long)p.gcen),
          "s"((unsigned long long)p.rot), "s"(p.N), "s"(p.T), "s"(p.share), "s"(p.units),
          "s"(p.wgs_per_example), "s"(p.wg_magic));
    // Workgroup ids go round the 8 XCDs (id % 8), each with its own L2.  XCD k takes the k-th
    // eighth of the (example, record) list, so the gradient volume of an example -- and the
    // lines of it that neighbouring records share -- is read through one L2 only.
    if (!FUSED && p.expect_tag != 0u && *p.tag != p.expect_tag) return;      // not the tables this call expects
    const unsigned lin = blockIdx.x + zero;
    const unsigned v = (lin & 7u) * p.share + (lin >> 3);
    if (v >= p.units || (lin >> 3) >= p.share) return;
    const unsigned bu = p.wg_magic == 0ull ? v : (unsigned)__umul64hi((unsigned long long)v, p.wg_magic);
    const int b = (int)bu, slot = (int)((v - bu * p.wgs_per_example) * 4u + (threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63u);
    const int N = p.N, T = p.T, D = gs.D;

    __shared__ __attribute__((aligned(16))) unsigned char s_marks[4][kSlotCap];
    unsigned char *marks = s_marks[threadIdx.x >> 6];
    static_assert(kSlotCap == 64 * 16, "one 16-byte store per lane clears the marks");
    reinterpret_cast<int4 *>(marks)[lane] = make_int4(0, 0, 0, 0);
    lds_sync();
    __shared__ float s_rot[4][9];       // (vector types, one launch)
    float4 a, gc, Ra, Rb;       // record, grid centre, rotation (rows, 9 values)
    float Rc;
    int ai, t_rec;
    if (FUSED) {
        // No tables: the wavefront of atom `slot` places it itself, with the arithmetic and the
        // tests of the prep kernel (every value here is the same in all lanes).
        if (slot >= N) return;
        const int at = __builtin_amdgcn_readfirstlane(slot);
        ai = at;
        const size_t k = (size_t)b * N + at;
        t_rec = VECTOR ? 0 : p.raw.types[k];
        float pos[3] = {p.raw.coords[3 * k], p.raw.coords[3 * k + 1], p.raw.coords[3 * k + 2]};
        const int n = p.raw.natoms ? p.raw.natoms[b] : N;
        float r_in = 0.0f;
        if (!VECTOR && !gs.radius_type_indexed) r_in = p.raw.radii[k];
        Xform X;
        load_xform(X, b, p.raw.centers, p.raw.quats, p.raw.translations);
        const bool member = at < n && t_rec >= 0 && t_rec < T;
        if (!VECTOR && gs.radius_type_indexed && member) r_in = p.raw.radii[t_rec];
        float r = gs.radius_scale * r_in, reach = r * gs.c;
        if (VECTOR) {
            r = 1.0f;
            float widest = 0.0f;        // of all channels
            for (int c = lane; c < T; c += 64) widest = fmaxf(widest, gs.radius_scale * p.radii[c]);
#pragma unroll
            for (int m = 32; m > 0; m >>= 1) widest = fmaxf(widest, __shfl_xor(widest, m));
            reach = widest * gs.c;
        }
        apply_xform(X, pos, pos);
        gc = make_float4((float)X.c[0], (float)X.c[1], (float)X.c[2], 0.0f);
        const float org[3] = {gc.x - gs.half, gc.y - gs.half, gc.z - gs.half};
        const bool inside = meets_grid(gs, org, pos, r, reach);
        if (!(member & inside)) {
            if (p.grad_coords && lane < 3) p.grad_coords[k * 3 + lane] = 0.0f;
            if (WANT_W)
                for (int c = lane; c < T; c += 64) p.grad_weights[k * T + c] = 0.0f;
            return;
        }
        a = make_float4(pos[0], pos[1], pos[2], r);
        if (VECTOR) {           // past the loop over the slots, which needs all registers (or it spills some)
            if (lane == 0)
                for (int m = 0; m < 9; ++m) s_rot[threadIdx.x >> 6][m] = (float)X.R[m];
        } else {
            Ra = make_float4((float)X.R[0], (float)X.R[1], (float)X.R[2], (float)X.R[3]);
            Rb = make_float4((float)X.R[4], (float)X.R[5], (float)X.R[6], (float)X.R[7]);
            Rc = (float)X.R[8];
        }
    } else {
        // Everything the wavefront needs first is requested in one go (one trip to memory, not
        // four in a row): the group table's last entry, the record and its atom index (slot
        // clamped into the array; whether the slot is live is decided afterwards), the grid
        // centre and the rotation.
        const int cslot = min(slot, N - 1);
        const unsigned char atom_alive = p.alive[(size_t)b * N + cslot];    // of ATOM number `slot`, see below
        const int4 last = p.meta[(size_t)b * T + (VECTOR ? 0 : T - 1)];
        a = p.rec[(size_t)b * N + cslot];
        ai = p.idx[(size_t)b * N + cslot];
        t_rec = VECTOR ? 0 : p.rchan[(size_t)b * N + cslot];
        gc = *reinterpret_cast<const float4 *>(p.gcen + 4 * b);
        const float *Rp = p.rot + b * 12;
        Ra = *reinterpret_cast<const float4 *>(Rp);
        Rb = *reinterpret_cast<const float4 *>(Rp + 4);
        Rc = Rp[8];
        asm volatile("" ::"s"(last.x), "s"(last.z), "s"(gc.x), "s"(gc.y), "s"(gc.z), "s"(Ra.x), "s"(Ra.y),
                     "s"(Ra.z), "s"(Ra.w), "s"(Rb.x), "s"(Rb.y), "s"(Rb.z), "s"(Rb.w), "s"(Rc));
        // Every output element is written by someone: the wavefront of record slot s also looks
        // after ATOM s -- if that atom has no live record (culled, past natoms, type out of range)
        // nobody else writes its gradient, so its zeros are stored here.
        if (slot < N && atom_alive == 0) {
            const size_t atom = (size_t)b * N + slot;
            if (p.grad_coords && lane < 3) p.grad_coords[atom * 3 + lane] = 0.0f;
            if (WANT_W)
                for (int k = lane; k < T; k += 64) p.grad_weights[atom * T + k] = 0.0f;
        }
        if (slot >= last.x + last.z) return;            // past the last group's slots (per wavefront)
        if (!(a.w > 0.0f)) return;                      // dead record: its atom's zeros are written above, by slot
    }
    const size_t D3 = (size_t)D * D * D;
    const int bs = source_example(p.subgrids, b);          // types and weights are the source example's
    float ox = gc.x - gs.half, oy = gc.y - gs.half, oz = gc.z - gs.half;
    if (FUSED && VECTOR) {
        ox = uniform(ox);
        oy = uniform(oy);
        oz = uniform(oz);
    }

    float tx = 0.0f, ty = 0.0f, tz = 0.0f;          // gradient in the transformed frame
    if (!VECTOR) {
        const int t = t_rec;
        const float r = a.w;
        Box bx;
        float sx = 0.0f, sy = 0.0f, sz = 0.0f;
        if (atom_box(gs, r * gs.c, a, ox, oy, oz, bx))
            reduce_channel<ALIGNED>(p, reinterpret_cast<const GT *>(p.G) + (size_t)b * T * D3, t, D3, a, r, bx, ox, oy, oz,
                                    marks, sx, sy, sz);
        const float inv_r2 = -4.0f * scale_of(r) * scale_of(r);         // (the sums hold -f/4)
        tx = sx * inv_r2;
        ty = sy * inv_r2;
        tz = sz * inv_r2;
    } else {
        // the atom is the wavefront's: what depends on it and on the channel stays in scalar registers
        ai = __builtin_amdgcn_readfirstlane(ai);
        a = make_float4(uniform(a.x), uniform(a.y), uniform(a.z), a.w);
        const size_t arow = ((size_t)bs * N + ai) * T, grow = ((size_t)b * N + ai) * T;
        // 64 channels at a time, in order of radius (so that the spheres of a group are nearly the same
        // size): lane l holds the l-th of them
        for (int base = 0; base < T; base += 64) {
            const int count = min(64, T - base);
            int chan = base + lane;         // of rank `lane`
            if (count <= kChanGroup) {
                chan = base + min(lane, count - 1);     // one group, in any order
            } else if (!FUSED && T <= 64) {
                chan = p.chan_order[(size_t)b * T + min(lane, T - 1)];
            } else {
                __shared__ unsigned char s_perm[4][64];
                unsigned char *perm = s_perm[threadIdx.x >> 6];
                float mine = lane < count ? p.radii[base + lane] : 0.0f;
                mine = mine > 0.0f ? mine : 0.0f;       // NaN and negative radii rank as 0: still a permutation
                int rank = 0;
                for (int m = 0; m < count; ++m) {
                    const float other = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), m));
                    rank += (other < mine || (other == mine && m < lane)) ? 1 : 0;
                }
                lds_sync();
                if (lane < count) perm[rank] = (unsigned char)lane;
                lds_sync();
                chan = base + (lane < count ? min((int)perm[lane], count - 1) : 0);
            }
            const float r = lane < count ? gs.radius_scale * p.radii[chan] : 0.0f;
            const float w = lane < count ? p.weights[arow + chan] : 0.0f;
            const unsigned long long live = __ballot(r > 0.0f);
            // the widest of each group of four, in whatever order the channels are: the tables' order is that
            // of the radii they were made with, and these are read in this call
            float v_reach = r * gs.c;
            v_reach = fmaxf(v_reach, quad_swap<0xB1>(v_reach));
            v_reach = fmaxf(v_reach, quad_swap<0x4E>(v_reach));
            const float inv = r > 0.0f ? scale_of(r) : 0.0f;
            const float v_nr2 = -(p.k * inv) * inv, v_fq = p.fAc * r, v_tq = -(p.tg * inv), v_cq = -4.0f * (w * inv) * inv;
            const auto lane_value = [](float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
            float gw = 0.0f;                // lane l: the weight gradient of the channel of rank l
            for (int t0 = 0; t0 < count; t0 += kChanGroup) {
                GroupCoef gc;
                gc.live = (unsigned)(live >> t0) & ((1u << kChanGroup) - 1u);
                if (gc.live == 0u) continue;
                const GT *Gq[kChanGroup];
#pragma unroll
                for (int q = 0; q < kChanGroup; ++q) {
                    const int l = min(t0 + q, 63);
                    Gq[q] = reinterpret_cast<const GT *>(p.G) + ((size_t)b * T + bcast(chan, l)) * D3;
                    gc.nr2[q] = lane_value(v_nr2, l);
                    gc.fq[q] = lane_value(v_fq, l);
                    gc.tq[q] = lane_value(v_tq, l);
                    gc.cq[q] = lane_value(v_cq, l);
                }
                const float reach = lane_value(v_reach, t0);
                Box bx;
                if (!atom_box(gs, reach, a, ox, oy, oz, bx)) continue;
                float sv[kChanGroup] = {0.0f, 0.0f, 0.0f, 0.0f};
                if (gc.live == (1u << kChanGroup) - 1u)         // a full group needs no test per voxel and channel
                    reduce_group<ALIGNED, WANT_W, true>(p, Gq, a, reach, bx, ox, oy, oz, marks, gc, tx, ty, tz, sv);
                else
                    reduce_group<ALIGNED, WANT_W, false>(p, Gq, a, reach, bx, ox, oy, oz, marks, gc, tx, ty, tz, sv);
                if (WANT_W) {
                    const float sum = wave_sum4(sv[0], sv[1], sv[2], sv[3]);
                    gw = (lane >> 2) == (t0 >> 2) ? sum : gw;
                }
            }
            if (WANT_W && lane < count) p.grad_weights[grow + chan] = gw;
        }
    }
    if (p.grad_coords) {
        const float t = wave_sum4(tx, ty, tz, 0.0f);
        tx = __int_as_float(bcast(__float_as_int(t), 0));
        ty = __int_as_float(bcast(__float_as_int(t), 1));
        tz = __int_as_float(bcast(__float_as_int(t), 2));
    }
    if (FUSED && VECTOR) {
        lds_sync();
        const float *R = s_rot[threadIdx.x >> 6];
        Ra = make_float4(R[0], R[1], R[2], R[3]);
        Rb = make_float4(R[4], R[5], R[6], R[7]);
        Rc = R[8];
    }
    if (lane == 0 && p.grad_coords) {
        float *o = p.grad_coords + ((size_t)b * N + ai) * 3;
        o[0] = (Ra.x * tx + Ra.w * ty) + Rb.z * tz;         // R^T: column m of R
        o[1] = (Ra.y * tx + Rb.x * ty) + Rb.w * tz;
        o[2] = (Ra.z * tx + Rb.y * ty) + Rc * tz;
    }
}

// out[b][k] = sum over s < sub3 of tmp[b * sub3 + s][k], summed in order of s
__global__ __launch_bounds__(256) void sum_subgrids_kernel(int sub3, size_t per_example,
                                                           const float *tmp, float *out)
{
    const size_t k = (size_t)blockIdx.x * 256u + threadIdx.x;
    if (k >= per_example) return;
    const size_t b = blockIdx.y;
    const float *src = tmp + b * (size_t)sub3 * per_example + k;
    float acc = 0.0f;
    for (int s = 0; s < sub3; ++s) acc += src[(size_t)s * per_example];
    out[b * per_example + k] = acc;
}

}  // namespace

hipError_t launch_sum_subgrids(int subgrid_count, int B_source, size_t per_example,
                               const float *tmp, float *grad, hipStream_t stream)
{
    const dim3 grd((unsigned)((per_example + 255) / 256), B_source), blk(256);
    hipLaunchKernelGGL(sum_subgrids_kernel, grd, blk, 0, stream, subgrid_count, per_example, tmp, grad);
    return hipGetLastError();
}

// Few atoms: no prep kernel, every atom's wavefront places its atom itself, in the caller's order.
// What is lost is the order by channel and plane (neighbouring wavefronts then share fewer lines of
// the gradient grid) and, per atom, the transform worked out by a whole wavefront; what is saved is
// the prep kernel's 10 us and the gap behind it.  Whole calls, one launch / prep kernel and backward kernel, us;
// atoms at 0.076 per cubic Angstrom about the grid's centre.
// Index types, 2040 atoms and 28 channels of 48^3 per example: 9.4 / 14.7 for 1 example, 33.7 / 35.4
// for 16, 46.2 / 46.4 for 24, 58.5 / 58.3 for 32, 90.9 / 85.0 for 50.
// Vector types read every channel for every atom.  Four channels of a grid of 48^3 are 1.8 MB and stay in
// an XCD's L2 whatever the order of the atoms; those of larger grids stay there only in the order of the
// tables, so the line lies at a product of atoms, channels and points.  2040 atoms, 28 x 48^3: one example 41.2 / 46.3,
// two 66.9 / 67.1, three 104 / 89; 12 x 64^3 25.8 / 29.5, two 46.8 / 41.7; 28 x 64^3 51.9 / 48.5; 12 x 96^3 33.9 / 31.9;
// 4 x 96^3 15.2 / 19.3, two 22.3 / 25.3; 28 x 96^3 at 0.25 A 228 / 191.
// One example of more than 4096 atoms: the tables list the atoms out of the grid's reach last and each XCD takes an
// eighth of the records, so that with a share f of the atoms within reach (what such a grid can hold: 0.08 atoms per
// cubic Angstrom, 2 A for their reach) as large a share of the XCDs works; and spacings beyond 0.5 A have fewer rows in a
// sphere.  Reads (atoms within reach x channels x points) x f^2 x min(1, (0.5 / spacing)^2) x sqrt(channels) tell the
// two apart, 1e9: 40 x 96^3 at 0.25 A of 5000 atoms (49) 422 / 671, 28 x 96^3 of 8000 (11) 356 / 585, 28 x 64^3 of 8000 (32)
// 121 / 125, 5 x 80^3 of 8000 (28) 41 / 51, 5 x 96^3 of 5000 (49) 40 / 41, 28 x 48^3 at 1 A of 8000 (33) 57 / 67, 40 x 48^3 (56)
// 81 / 88, but 28 x 64^3 of 6000 (56) 117 / 100; of 4500 (100) 107 / 88; 20 x 72^3 of 8000 (70) 117 / 102; 28 x 64^3 at 1 A of
// 8000 (78) 78 / 70; 28 x 80^3 at 0.375 A of 5000 (94) 196 / 158; 8 x 96^3 of 5000 (100) 60 / 47; 12 x 96^3 of 6000 (221) 109 / 65.
// Up to four channels are one pass over each atom's rows: 2 x 128^3 of 8000 24 / 35, 3 x 120^3 33 / 38, 4 x 96^3 46 / 47,
// 4 x 112^3 59 / 50.
constexpr long long kSingleAtoms = 49152;           // index types
constexpr long long kSingleAtomsVector = 8192;      // vector types, and ...
constexpr double kSingleReads = 1.5e10;             // atoms x channels x points
constexpr double kSingleReadsLong = 5.7e10;         // ... of one example of more than 4096, weighted as above
constexpr double kSingleReadsGroup = 6.5e10;        // ... and of no more than four channels: atoms within reach
bool backward_takes_single_launch(const GridSpec &gs, const Batch &bt)
{
    if (bt.sub.count != 1) return false;
    const long long atoms = (long long)bt.B * bt.N;
    if (!bt.vec) return atoms <= kSingleAtoms;
    if (atoms > kSingleAtomsVector) return false;
    const double points = (double)bt.T * gs.D * gs.D * gs.D;
    if (bt.B > 1 || bt.N <= 4096) return atoms * points <= kSingleReads;
    const double side = (double)gs.D * gs.res + 4.0, held = std::fmin((double)atoms, 0.08 * side * side * side);
    if (bt.T <= kChanGroup) return held * points <= kSingleReadsGroup;
    const double f = held / (double)atoms, rows = std::fmin(1.0, 0.25 / ((double)gs.res * gs.res));
    return held * points * f * f * rows * std::sqrt((double)bt.T) <= kSingleReadsLong;
}

hipError_t launch_backward(const GridSpec &gs, const Batch &bt, const Workspace &ws,
                           const void *grad_out, bool grad_is_double, float *grad_coords,
                           float *grad_weights, bool single_launch, unsigned expect_tag,
                           KernelEvents ev, hipStream_t stream)
{
    BwdParams p;
    p.gs = gs;
    p.rec = ws.rec; p.idx = ws.idx; p.meta = ws.meta; p.rot = ws.rot;
    p.rchan = ws.rchan; p.chan_order = ws.chan_order; p.weights = bt.weights; p.radii = bt.radii; p.gcen = ws.gcen;
    p.alive = ws.alive; p.tag = ws.tag; p.expect_tag = expect_tag;
    p.G = grad_out; p.grad_coords = grad_coords; p.grad_weights = grad_weights;
    p.subgrids = bt.sub.count; p.N = bt.N; p.T = bt.T;
    p.raw = raw_inputs(bt);
    {
        const double k = 2.8853900817779268;    // 2 / ln 2
        // (beyond x = 100 the density is 0 in float whatever the branch: larger g need no larger constants)
        const double g2 = std::fmax(std::fmin((double)gs.g2, 1.0e4), 1.0e-30), g = std::sqrt(g2), c = g + 0.5 / g;
        p.ng2k = (float)(-g2 * k);
        p.nfA = (float)(-2.0 * g2);
        p.fAc = (float)(2.0 * g2 * c);
        p.tg = (float)(2.0 * g);
        p.tc = (float)(2.0 * g * c);
        p.k = (float)k;
    }
    const bool aligned = (gs.D % 4 == 0) && (((uintptr_t)grad_out & 15u) == 0);
    p.wgs_per_example = (unsigned)((bt.N + 3) / 4);
    p.units = p.wgs_per_example * (unsigned)bt.B;
    p.share = (p.units + 7u) / 8u;
    p.wg_magic = p.wgs_per_example <= 1u ? 0ull : (~0ull / p.wgs_per_example) + 1ull;
    const dim3 grd(p.share * 8u), blk(256);
#define MG_BWD(V, Al, Gt, Fu, Ww) \
    hipExtLaunchKernelGGL((backward_kernel<V, Al, Gt, Fu, Ww>), grd, blk, 0, stream, ev.start, ev.stop, 0, p)
#define MG_BWD_FUSED(V, Al, Gt, Ww) \
    do { if (single_launch) MG_BWD(V, Al, Gt, true, Ww); else MG_BWD(V, Al, Gt, false, Ww); } while (0)
#define MG_BWD_ALIGNED(V, Gt, Ww) \
    do { if (aligned) MG_BWD_FUSED(V, true, Gt, Ww); else MG_BWD_FUSED(V, false, Gt, Ww); } while (0)
#define MG_BWD_TYPE(Gt)                                                 \
    do {                                                                \
        if (!bt.vec) MG_BWD_ALIGNED(false, Gt, false);                  \
        else if (grad_weights) MG_BWD_ALIGNED(true, Gt, true);          \
        else MG_BWD_ALIGNED(true, Gt, false);                           \
    } while (0)
    if (grad_is_double) MG_BWD_TYPE(double); else MG_BWD_TYPE(float);
#undef MG_BWD_TYPE
#undef MG_BWD_ALIGNED
#undef MG_BWD_FUSED
#undef MG_BWD
    return hipGetLastError();
}

}  // namespace mg
