// Steps 3-5 of the path: the forward atom-to-grid kernel (index types, vector
// types, binary occupancy), GridMaker section of the paper.
//
// Design (gfx950, wave64).  Each channel of the output (D*D*D floats, z fastest)
// is cut into flat tiles of `tile_floats` consecutive floats (1024 = 4096 B by
// default, 2048 when a tile is expected to meet many records), whatever rows and
// x-planes that run happens to cover; with the usual grids (D = 48, 96) every
// tile starts on a 4 KB boundary of the output.
// One workgroup of 1, 2 or 4 wavefronts produces one tile; its wavefronts split
// the atoms and, at the end, the 2 KB chunks of the tile between them:
//   1. the workgroup loads the records of the channel's atoms that can reach the
//      x-planes the tile touches (spans the prep kernel computed), one atom per
//      lane, atom e going to wavefront e mod (number of wavefronts);
//   2. each lane tests its atom against the tile's rows in two x-planes at a
//      time (disc of the atom's cutoff sphere in the plane versus the row
//      range).  Every surviving (atom, row) pair is a task; a wavefront scan
//      gives each atom the index of its first task, which the lane marks in a
//      byte array, so that a later max-scan over the marks tells every lane
//      which atom its task belongs to: all 64 lanes work even though one
//      atom's footprint is small, and no lane loops over its rows to list them;
//   3. each lane takes one task: the chord of the atom's sphere along that
//      z-row, clipped to the tile in its first and last row.  It evaluates the
//      density voxel by voxel and adds it into the tile held in LDS with LDS
//      atomics (two atoms may hit one voxel in the same instruction).  The tile
//      accumulates in unsigned fixed point (2^-26 steps, integer LDS atomics):
//      integer adds run ~40x faster in LDS than float adds on this chip, are
//      exact and order-independent, and a contribution is rounded by at most
//      7.5e-9.  Where more than 63 atoms reach a tile a sum could pass 2^32: the
//      adds are then watched, and if one comes near a second pass finds the sums'
//      upper bits, so that a grid never depends on the order of the atoms or on
//      how they are split over wavefronts;
//   4. the finished tile is streamed to HBM, each lane writing 32 contiguous
//      bytes (two adjacent 16-byte stores), every output element exactly once,
//      zeros included.  Tiles no atom touches skip LDS and store zeros.
// The tile sits in LDS in output order (LDS index = output index - first index of
// the tile).  With more than one wavefront there are two barriers per tile: after
// the zero fill, and before the tile is read back.  The default is
// one wavefront per 4 KB tile (no barrier at all; 8 KB when a tile meets many
// records).  A grid of doubles takes 512 voxels per workgroup (4 KB of output) and
// stores 1 KB per instruction.
//
// Why 4 KB / 8 KB tiles on 4 KB boundaries: measured on this chip, one-wavefront
// workgroups that each write one aligned 4 KB or 8 KB run sustain 6.3-6.6 TB/s
// when nothing else is going on, while runs of 6, 9, 18 or 36 KB per wavefront
// (whole x-planes of a 48^3 grid are 9 KB) fall to 5.2-5.4 TB/s.  Reads do not
// disturb that stream as long as a cache serves them; reads that must come from
// HBM do, far beyond their bytes.  The tables this kernel reads (a few MB, written
// by the prep kernel just before) would be pushed out to HBM by the hundreds of MB
// of stores before the later examples' turn, so every wavefront also touches 1 KB
// of them (see the kernel's preamble): 102 us against 108 us per launch on the
// 48^3 batch of 50, 257 us against 328 us on a 96^3 batch of 16.
//
// The density is rho(x) = exp(-2x^2) for x <= g, A(x-c)^2 for g < x < c, else 0
// (x = d/r).  Distances are carried in units of r/sqrt(k), k = 2*log2(e), so
// that the Gaussian is exp2(-x'^2) with the hardware exp2 and the tail is
// (sqrt(x'^2)*sA - cA)^2 with sA = sqrt(A/k), cA = c*sqrt(A).
//
// Binary mode decides d^2 <= r^2 in float with this fixed order (the file is
// compiled with -ffp-contract=off, nothing fuses):
//   gx = o_x + (float)i*res   (o = center - half)      dx = gx - ax
//   d2 = (dx*dx + dy*dy) + dz*dz                        r2 = r*r
#include <cmath>

#include "mg_common.h"
#include "mg_wave.h"
#include "mg_xform.h"

namespace mg {

namespace {

constexpr int kTaskCap = 256;                   // (atom, row) tasks staged per round
constexpr int kFusedAtoms = 2048;               // single launch: most atoms a workgroup of several wavefronts looks through
constexpr unsigned kKeepAliveBytes = 256;       // what every wavefront re-reads of the tables by default
// Index types: steps of 2^-26.  (With 2^-24, which leaves room for 255 atoms, the error against 64 bits
// of 2040 atoms in one channel of 48^3 was 2.6e-7, 2.2e-7 for sums in floats; sums past 64 hardly occur.)
constexpr float kFixedOne = 67108864.0f;        // 2^26
constexpr float kAlmostHalf = 0.49999997f;       // rounds to the nearest step: 0.5 would push odd whole numbers of 24 bits up
constexpr int kSafeHits = 63;                   // this many densities of at most 1 stay below 2^32 steps
constexpr int kDigitBits = 13;                  // ... and fewer than 2^19 of their upper or lower digits
constexpr int kDigitHits = 1 << 19;
constexpr float kFixedLimit = 120.0f;           // vector types: largest sum of |weights| trusted to fixed point
constexpr float kSignedTerm = 60.0f;            // ... and largest weight next to negative ones (signed conversion: 64)
// Vector types: steps of 2^-25.  A voxel's sum lies between minus the negative weights that reach the tile
// and the positive ones; while the two together stay below 128 the 32 bits name it, whatever its sign.
constexpr int kVecFixedBits = 25;

struct FwdParams {
    GridSpec gs;
    RawInputs raw;
    const float4 *rec;
    const int *idx;
    const int2 *range;
    const float *weights;
    const float *radii;
    const float *gcen;          // [B][4] grid centres, written by the prep kernel
    const int *chan_order;      // [B][T] vector types: channels in order of radius
    unsigned groups;            // vector types: groups of kVecGroup channels per example
    const unsigned *tag;        // what the workspace's tables were made for
    unsigned expect_tag;        // != 0: do nothing unless *tag equals it (calls on prepared tables)
    void *out;                      // float or double grid
    int subgrids, N, T;             // subgrids: virtual examples per example (weights are per example)
    int tile_floats;                // floats per tile (a multiple of 512)
    unsigned tiles;                 // divisor of the workgroup id: tiles per channel, or channels (B*T) when pos_major
    unsigned shifted;               // 1: tiles lie on tile boundaries of the whole output, not of the channel (see tile_geom)
    unsigned pos_major;             // 0: all tiles of a channel, then the next channel; 1: tile k of every channel, then tile k+1
    unsigned long long div_magic;   // ceil(2^40 / D): x / D = (x * div_magic) >> 40 for x < D^3
    unsigned long long tiles_magic; // ceil(2^64 / tiles), see div_u32
    unsigned long long t_magic;     // ceil(2^64 / T)
    int xcd_shift;                  // >= 0: runs of 2^xcd_shift consecutive tiles go to one XCD
    unsigned n_remap;               // workgroups covered by that mapping (the rest map 1:1)
    int debug;
    unsigned ka_chunks, ka_last;    // keep-alive reads: chunks of the tables (0: none), byte offset of the last one
    unsigned ka_shift;              // log2 of the chunk size in bytes (6..10)
    unsigned ka_skip;               // 0, 1, 3 or 7: wavefronts whose id has none of these bits set do the read
    float sk;           // sqrt(k), k = 2 log2(e)
    float inv_sk;
    float g2k, c2k;     // g^2 k (index types), c^2 k
    float sA, cA;       // tail coefficients (index types)
    float vg2k, tk, tc; // vector types: g^2 k, 2g/sqrt(k), 2g c
};

// what a wavefront keeps for the tile it is working on (all wave-uniform)
struct TileCtx {
    float *tile;                // LDS: tile_floats floats, in output order
    unsigned char *marks;       // LDS (per wavefront): marks[first task of the atom in lane l] = l + 1
    int *shared;                // LDS (workgroup): [0] bound on |sum| (1/256 units; vector types), [1] bit 0:
                                // any task, bit 1: sums may have passed 2^32; vector types: [4 + q] what channel
                                // q's negative weights add up to (1/256 units)
    int lane, wave;
    int D, n;                   // points per side; floats in this tile
    int nrows;                  // grid rows the tile touches
    int c0, c1;                 // first column of its first row, last column of its last row
    int rowA, rowB;             // tile row of row 0 of plane A / plane B (may be negative)
    float res, inv_res, oy, oz;     // oy, oz: grid origin (binary mode works from it)
    float cen_x, cen_y, cen_z, hD;  // grid centre; (D-1)/2.  The real density works in
                                    // coordinates relative to the centre: differences of
                                    // nearby numbers, no rounding of an origin
    float g2k, c2k, sA, cA;
    int debug;
};

__device__ inline int div_by_d(int x, unsigned long long magic)
{
    return (int)(((unsigned long long)(unsigned)x * magic) >> 40);
}

// x / d for any 32-bit x, with magic = ceil(2^64 / d) (d >= 2; d == 1 is passed as magic 0).
__device__ inline unsigned div_u32(unsigned x, unsigned long long magic)
{
    return magic == 0ull ? x : (unsigned)__umul64hi((unsigned long long)x, magic);
}

// One atom of the current batch as its lane holds it.
struct Atom {
    float4 a;           // x', y', z', r
    bool valid;
};

// What a task needs of its atom; it stays in the registers of the atom's lane and the
// task's lane fetches it with ds_bpermute (register exchange, no LDS storage).
struct Cand {
    float c0, c1, c2, c3;       // fy, fz (grid steps from the centre), stepk, inv_stepk | w
                                // (binary: y', z', r^2, reach^2)
    float pxA, pxB;             // plane term of d^2 for plane A, plane B
    int start;                  // index of the atom's first task
    int pack;                   // jloA | nA << 10 | jloB << 20
};

__device__ inline float fetch(int byte_addr, float v)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(byte_addr, __float_as_int(v)));
}

// How fixed-point densities are added up.
enum class Sum {
    kPlain,
    kWatch,     // and the values found before each add collected in `seen`
    kDigit      // only `bits` bits of each from bit `shift`
};
struct SumArgs {
    unsigned shift = 0, bits = 0;
    unsigned seen = 0;
};

// Run the staged tasks [0, ntasks): one (atom, row) chord per lane.
template <bool BINARY, Sum SUM>
__device__ inline void run_tasks(const TileCtx &cx, const Cand &cd, int ntasks, SumArgs &sa)
{
    int carry = 0;
    for (int base = 0; base < ntasks; base += 64) {
        const int tau = base + cx.lane;
        bool act = tau < ntasks;
        // which atom: the last mark at or before this task
        const int owner = max(carry, wave_inclusive_max((int)cx.marks[tau]));
        carry = bcast(owner, 63);
        const int src = (act ? owner - 1 : 0) << 2;
        const float4 p0 = make_float4(fetch(src, cd.c0), fetch(src, cd.c1), fetch(src, cd.c2),
                                      fetch(src, cd.c3));
        const float2 p1 = make_float2(fetch(src, cd.pxA), fetch(src, cd.pxB));
        const int pack = __builtin_amdgcn_ds_bpermute(src, cd.pack);
        const int k = tau - __builtin_amdgcn_ds_bpermute(src, cd.start);   // row number within the atom
        const int nA = (pack >> 10) & 1023;
        const bool inB = k >= nA;
        const int j = inB ? (pack >> 20) + (k - nA) : (pack & 1023) + k;   // row in its plane
        const int trow = (inB ? cx.rowB : cx.rowA) + j;                    // row in the tile
        const float px2 = inB ? p1.y : p1.x;                               // plane term of d^2
        const int clip_lo = trow == 0 ? cx.c0 : 0;
        const int clip_hi = trow == cx.nrows - 1 ? cx.c1 : cx.D - 1;
        float *rowp = cx.tile + (trow * cx.D - cx.c0);
        if (BINARY) {
            const float ay = p0.x, az = p0.y, r2 = p0.z, reach2 = p0.w;
            const float gy = cx.oy + (float)j * cx.res;
            const float dy = gy - ay;
            const float dy2 = dy * dy;
            const float rem = (reach2 - px2) - dy2;
            act = act && rem > 0.0f;
            const float hz = __builtin_amdgcn_sqrtf(fmaxf(rem, 0.0f)) * cx.inv_res + 1.0e-3f;
            const float fz = (az - cx.oz) * cx.inv_res;
            const int klo = max(clip_lo, (int)ceilf(fz - hz));
            const int khi = min(clip_hi, (int)floorf(fz + hz));
            const int nz = act ? khi - klo + 1 : 0;
            const float base2 = px2 + dy2;
            for (int i = 0; i < nz; ++i) {
                const float gz = cx.oz + (float)(klo + i) * cx.res;
                const float dz = gz - az;
                const float d2 = base2 + dz * dz;
                if (d2 <= r2) rowp[klo + i] = 1.0f;
            }
        } else {
            const float fy = p0.x, fz = p0.y, stepk = p0.z, inv_stepk = p0.w;
            const float dyk = (((float)j - cx.hD) - fy) * stepk;
            const float x2b = fmaf(dyk, dyk, px2);
            const float rem = cx.c2k - x2b;
            act = act && rem > 0.0f;
            const float hz = __builtin_amdgcn_sqrtf(fmaxf(rem, 0.0f)) * inv_stepk + 1.0e-3f;
            const float fzi = fz + cx.hD;                                   // as a grid index
            const int first = (int)ceilf(fzi - hz);         // of the whole chord
            const int klo = max(clip_lo, first);
            const int khi = min(clip_hi, (int)floorf(fzi + hz));
            const int nz = act ? khi - klo + 1 : 0;
            // counted from the whole chord's first voxel: the same density wherever the tile cuts the row
            const float z0 = (((float)first - cx.hD) - fz) * stepk;
            float cA = cx.cA;
            asm volatile("" : "+v"(cA));        // keep it in a VGPR across the loop
            float fi = (float)(klo - first);
            unsigned old = 0u;
            for (int i = 0; i < nz; ++i) {
                const float zs = fmaf(fi, stepk, z0);
                fi += 1.0f;
                const float x2 = fmaf(zs, zs, x2b);
                const float e = __builtin_amdgcn_exp2f(-x2);
                // sqrt(A) (c - x), at most exp(-g^2) <= 1 where the tail applies: the multiply-add's
                // clamp to [0, 1] cuts it off at the cutoff
                const float u = __builtin_amdgcn_fmed3f(fmaf(-__builtin_amdgcn_sqrtf(x2), cx.sA, cA), 0.0f, 1.0f);
                const float rho = x2 <= cx.g2k ? e : u * u;             // 0 beyond the cutoff
                unsigned v = (unsigned)fmaf(rho, kFixedOne, kAlmostHalf);
                if (SUM == Sum::kDigit) v = __builtin_amdgcn_ubfe(v, sa.shift, sa.bits);
                if (SUM == Sum::kWatch) {
                    asm volatile("" : "+v"(old) : "v"(v));      // the answer to the add before is not waited for until here
                    sa.seen |= old;
                }
                old = __hip_atomic_fetch_add(reinterpret_cast<unsigned *>(rowp) + klo + i, v, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            if (SUM == Sum::kWatch) sa.seen |= old;
        }
    }
    lds_sync();
}

// Rows of one x-plane (rows [ja, jb) of it belong to the tile) that the lane's atom reaches.
//   out: px2 = plane term of the squared distance (scaled units; binary: dx^2), rows [jlo, jlo+n)
template <bool BINARY>
__device__ inline int plane_rows(const TileCtx &cx, const FwdParams &p, const Atom &at, float gx,
                                 float xc, int ja, int jb, float sks, float inv_stepk, float fy,
                                 float fz, float &px2, int &jlo)
{
    // gx: x of the plane; xc: the same relative to the grid centre; fy, fz: grid indices
    float hv;
    bool ok = at.valid && ja < jb;
    if (BINARY) {
        const float dx = gx - at.a.x;
        const float reach = at.a.w + 1.0e-3f * cx.res;
        px2 = dx * dx;
        const float h2 = reach * reach - px2;
        ok = ok && h2 > 0.0f;
        hv = __builtin_amdgcn_sqrtf(fmaxf(h2, 0.0f)) * cx.inv_res + 1.0e-3f;
    } else {
        const float dxk = (xc - (at.a.x - cx.cen_x)) * sks;
        px2 = dxk * dxk;
        const float h2 = cx.c2k - px2;
        ok = ok && h2 > 0.0f;
        hv = __builtin_amdgcn_sqrtf(fmaxf(h2, 0.0f)) * inv_stepk + 1.0e-3f;
    }
    // half-width of the footprint in this plane, in grid steps, padded
    jlo = max(ja, (int)ceilf(fy - hv));
    const int jhi = min(jb - 1, (int)floorf(fy + hv));
    ok = ok && (jlo <= jhi) && (fz + hv >= 0.0f) && (fz - hv <= (float)(cx.D - 1));
    return ok ? jhi - jlo + 1 : 0;
}

// What one lane found for its atom in planes iA and iA + 1 of the tile.
struct PairHit {
    Cand cd;
    int nA, nB;         // rows reached in plane A, plane B
};

// One atom per lane against the rows of planes A and B that belong to the tile.
template <bool BINARY>
__device__ inline PairHit pair_test(const TileCtx &cx, const FwdParams &p, const Atom &at, float ox,
                                    int iA, int jaA, int jbA, int jaB, int jbB)
{
    PairHit h;
    const float r = at.a.w;
    // per atom: position in grid steps, scale of its distances
    const float fy = (at.a.y - cx.cen_y) * cx.inv_res;      // from the grid centre
    const float fz = (at.a.z - cx.cen_z) * cx.inv_res;
    const float fyi = BINARY ? (at.a.y - cx.oy) * cx.inv_res : fy + cx.hD;   // as grid indices
    const float fzi = BINARY ? (at.a.z - cx.oz) * cx.inv_res : fz + cx.hD;
    const float sks = at.valid ? p.sk * __builtin_amdgcn_rcpf(r) : 0.0f;
    const float stepk = cx.res * sks;
    const float inv_stepk = r * cx.inv_res * p.inv_sk;
    int jloA, jloB = 0;
    const float gxA = ox + (float)iA * cx.res, gxB = ox + (float)(iA + 1) * cx.res;
    const float xcA = ((float)iA - cx.hD) * cx.res, xcB = ((float)(iA + 1) - cx.hD) * cx.res;
    h.nA = plane_rows<BINARY>(cx, p, at, gxA, xcA, jaA, jbA, sks, inv_stepk, fyi, fzi, h.cd.pxA, jloA);
    h.nB = 0;
    h.cd.pxB = 0.0f;
    if (jaB < jbB)      // uniform: most tiles of small tile sizes lie in one plane
        h.nB = plane_rows<BINARY>(cx, p, at, gxB, xcB, jaB, jbB, sks, inv_stepk, fyi, fzi, h.cd.pxB, jloB);
    if (MG_DEBUG_IS(cx, 1)) { h.nA = 0; h.nB = 0; }
    if (h.nA == 0) jloA = 0;        // both are packed into bit fields below
    if (h.nB == 0) jloB = 0;
    if (BINARY) {
        const float reach = r + 1.0e-3f * cx.res;
        h.cd.c0 = at.a.y; h.cd.c1 = at.a.z; h.cd.c2 = r * r; h.cd.c3 = reach * reach;
    } else {
        h.cd.c0 = fy; h.cd.c1 = fz; h.cd.c2 = stepk; h.cd.c3 = inv_stepk;
    }
    h.cd.start = 0;
    h.cd.pack = jloA | (h.nA << 10) | (jloB << 20);
    return h;
}

// Stage the tasks of the hits (rows of plane A, then rows of plane B, atom after atom)
// and run them.
// Returns whether there was any task.
template <bool BINARY>
__device__ inline bool pair_run(const TileCtx &cx, PairHit &h, Sum sum, SumArgs &sa)
{
    int todo = h.nA + h.nB;         // lanes still to be staged have todo > 0
    if (__ballot(todo > 0) == 0ull) return false;
    while (true) {
        const int incl = wave_inclusive_scan(todo);
        int total = bcast(incl, 63);
        if (total == 0) break;
        bool now = todo > 0;
        if (total > kTaskCap) {     // rare: the rest waits for the next round
            now = now && incl <= kTaskCap;
            total = bcast(wave_inclusive_scan(now ? todo : 0), 63);
            if (total == 0) break;
        }
        if (cx.lane < kTaskCap / 16)
            reinterpret_cast<float4 *>(cx.marks)[cx.lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (now) {
            h.cd.start = incl - todo;
            cx.marks[h.cd.start] = (unsigned char)(cx.lane + 1);
            todo = 0;
        }
        lds_sync();
        if (BINARY || sum == Sum::kPlain) run_tasks<BINARY, Sum::kPlain>(cx, h.cd, total, sa);
        else if (sum == Sum::kWatch) run_tasks<BINARY, Sum::kWatch>(cx, h.cd, total, sa);
        else run_tasks<BINARY, Sum::kDigit>(cx, h.cd, total, sa);
    }
    return true;
}

// 16-byte stores to places that are only aligned like their elements
typedef float Float4E __attribute__((ext_vector_type(4), aligned(4)));
typedef double Double2E __attribute__((ext_vector_type(2), aligned(8)));

// Stream the finished tile to HBM (zeros if no atom touched it).  ITERS = tile_floats / 512
// chunks of 2 KB; wavefront w of NW takes chunks w, w + NW, ...
// VECTOR: in steps of 2^-kVecFixedBits, the sums at least -neg.
// LOOSE: the output is only aligned like its elements.
template <bool ALIGNED, int ITERS, int NW, typename OUT, bool VECTOR = false, bool LOOSE = false>
__device__ inline void store_tile(const TileCtx &cx, OUT *dst, bool touched, bool fixed, unsigned neg = 0u)
{
    const auto value = [&](float bits) {
        return (float)__float_as_uint(bits) * (VECTOR ? 1.0f / (float)(1 << kVecFixedBits) : 1.0f / kFixedOne);
    };
    const auto signed_value = [&](float bits) {
        const unsigned i = __float_as_uint(bits);
        const bool minus = i + neg < neg;           // [-neg, 0)
        const float v = (float)(minus ? 0u - i : i) * (1.0f / (float)(1 << kVecFixedBits));
        return minus ? -v : v;
    };
    constexpr bool kWide = sizeof(OUT) == 8;        // a grid of doubles: the same values, widened
    if (ALIGNED && kWide) {
        // Doubles: every store instruction writes 1 KB in one piece (lane l its 16 bytes at
        // 16 l), four per 512-voxel chunk.
        constexpr int MINE = ITERS / NW;
        const int n2 = cx.n >> 1;
        Double2E *dst2 = reinterpret_cast<Double2E *>(dst);
        const float2 *src2 = reinterpret_cast<const float2 *>(cx.tile);
        const bool convert = touched && fixed;
#pragma unroll
        for (int it = 0; it < MINE; ++it) {
            float2 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int o = ((it * NW + cx.wave) * 4 + k) * 64 + cx.lane;
                v[k] = touched ? src2[o] : make_float2(0.0f, 0.0f);
                if (convert && VECTOR && neg != 0u)
                    v[k] = make_float2(signed_value(v[k].x), signed_value(v[k].y));
                else if (convert)
                    v[k] = make_float2(value(v[k].x), value(v[k].y));
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int o = ((it * NW + cx.wave) * 4 + k) * 64 + cx.lane;
                if (o < n2) dst2[o] = Double2E{(double)v[k].x, (double)v[k].y};
            }
        }
    } else if (ALIGNED) {
        constexpr int MINE = ITERS / NW;            // chunks per wavefront
        const int n4 = cx.n >> 2;                   // even: D^3 and the tile size are multiples of 8
        float4 *dst4 = reinterpret_cast<float4 *>(dst);         // float grids
        Float4E *dst4e = reinterpret_cast<Float4E *>(dst);
        const float4 *src4 = reinterpret_cast<const float4 *>(cx.tile);
        // Constant trip count, fully unrolled; the tile comes from LDS into registers
        // under a uniform branch (zeros otherwise), so that the stores below are one
        // straight sequence with no load between them.
        float4 v[2 * MINE];
        if (touched) {
#pragma unroll
            for (int it = 0; it < 2 * MINE; ++it)
                v[it] = src4[((it >> 1) * NW + cx.wave) * 128 + cx.lane * 2 + (it & 1)];
        } else {
#pragma unroll
            for (int it = 0; it < 2 * MINE; ++it) v[it] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        const bool convert = touched && fixed;
        // chunk after chunk: convert its two float4s, then the two 16-byte halves of a lane's
        // 32 bytes go out back to back, under one predicate (separated by other instructions
        // they are markedly slower); the first stores leave while later chunks are converted
#pragma unroll
        for (int it = 0; it < MINE; ++it) {
            float4 a = v[2 * it], b = v[2 * it + 1];
            if (convert && VECTOR && neg != 0u) {
                a = make_float4(signed_value(a.x), signed_value(a.y), signed_value(a.z), signed_value(a.w));
                b = make_float4(signed_value(b.x), signed_value(b.y), signed_value(b.z), signed_value(b.w));
            } else if (convert) {
                a = make_float4(value(a.x), value(a.y), value(a.z), value(a.w));
                b = make_float4(value(b.x), value(b.y), value(b.z), value(b.w));
            }
            const int o = (it * NW + cx.wave) * 128 + cx.lane * 2;
            if (o < n4) {
                if (LOOSE) {
                    dst4e[o] = Float4E{a.x, a.y, a.z, a.w};
                    dst4e[o + 1] = Float4E{b.x, b.y, b.z, b.w};
                } else {
                    dst4[o] = a;
                    dst4[o + 1] = b;
                }
            }
        }
    } else {
        for (int o = cx.wave * 64 + cx.lane; o < cx.n; o += 64 * NW) {
            float v = 0.0f;
            if (touched)
                v = !fixed ? cx.tile[o] : VECTOR && neg != 0u ? signed_value(cx.tile[o]) : value(cx.tile[o]);
            dst[o] = (OUT)v;
        }
    }
}

// ALIGNED: all channels begin on 16 bytes; else full tiles do if the tiles are `shifted`.  (Vector types
// store full tiles 16 bytes at a time wherever they begin.)
template <bool ALIGNED, int ITERS, int NW, typename OUT, bool VECTOR = false>
__device__ inline void store_any_tile(const FwdParams &p, const TileCtx &cx, OUT *dst, bool touched, bool fixed,
                                      unsigned neg = 0u)
{
    if (ALIGNED || ((VECTOR || p.shifted) && cx.n == ITERS * 512))
        store_tile<true, ITERS, NW, OUT, VECTOR, !ALIGNED && VECTOR>(cx, dst, touched, fixed, neg);
    else
        store_tile<false, ITERS, NW, OUT, VECTOR>(cx, dst, touched, fixed, neg);
}

// Where a tile lies: floats [f0, f1) of the channel = rows [R0, R1) of its D*D rows, which
// belong to x-planes i_lo .. i_hi.  f0 is the skip-th float of the tile in LDS.
// A channel of D*D*D floats that is no multiple of 16 bytes begins anywhere in a line; its tiles then
// lie on tile boundaries of the whole output (`shifted`), the first and the last of a channel are
// shorter (and the last may be empty: f1 <= f0), and all others are stored like those of aligned
// channels, 32 bytes per lane, where a tile on boundaries of its channel had to be stored 4 bytes at
// a time: 50 x 28 x 47^3 (581 MB) 119 instead of 152 us a call, 20 ragged examples of 28 x 49^3 59
// instead of 78 us.
struct TileGeom {
    int f0, f1, R0, R1, i_lo, i_hi, skip;
};

template <bool ALIGNED, int ITERS>
__device__ inline TileGeom tile_geom(const FwdParams &p, int D, unsigned tile_in_chan, unsigned chan)
{
    TileGeom g;
    const int total = D * D * D;
    const int from = (int)tile_in_chan * (ITERS * 512) -
                     (!ALIGNED && p.shifted ? (int)((chan * (unsigned)total) & (unsigned)(ITERS * 512 - 1)) : 0);
    g.f0 = max(from, 0);
    g.skip = g.f0 - from;
    g.f1 = min(total, from + ITERS * 512);
    if (!ALIGNED && g.f1 <= g.f0) return g;
    g.R0 = div_by_d(g.f0, p.div_magic);
    g.R1 = div_by_d(g.f1 - 1, p.div_magic) + 1;
    g.i_lo = div_by_d(g.R0, p.div_magic);
    g.i_hi = div_by_d(g.R1 - 1, p.div_magic);
    return g;
}

// One tile of channel (b, t): the records [r0, r1) of the example can reach it; cen is the
// grid centre.
// FUSED (small problems, index types): there are no records; the "records" [r0, r1) are the
// example's atoms themselves, and a lane transforms, culls and filters by type the atom it takes,
// with the arithmetic and the tests of the prep kernel.
// With more than one wavefront `list` names the atoms of type t (find_atoms).
template <bool BINARY, bool ALIGNED, int ITERS, int NW, typename OUT, bool FUSED = false>
__device__ __forceinline__ void tile_body(const FwdParams &p, float *lds, int b, int t,
                                          const TileGeom &tg, int r0, int r1, const float4 &cen,
                                          const unsigned short *list = nullptr)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const GridSpec &gs = p.gs;
    const int D = gs.D, T = p.T, N = p.N;
    const int total = D * D * D;
    const int f0 = tg.f0, f1 = tg.f1, R0 = tg.R0, R1 = tg.R1, i_lo = tg.i_lo, i_hi = tg.i_hi;
    TileCtx cx;
    cx.tile = lds + (ALIGNED ? 0 : tg.skip);
    cx.marks = reinterpret_cast<unsigned char *>(lds + ITERS * 512) + wave * kTaskCap;
    cx.shared = reinterpret_cast<int *>(lds + ITERS * 512 + NW * (kTaskCap / 4));
    cx.lane = lane;
    cx.wave = wave;
    cx.D = D;
    cx.n = f1 - f0;
    cx.nrows = R1 - R0;
    cx.c0 = f0 - R0 * D;
    cx.c1 = f1 - 1 - (R1 - 1) * D;
    cx.rowA = 0;
    cx.rowB = 0;
    cx.res = gs.res;
    cx.inv_res = gs.inv_res;
    cx.g2k = p.g2k; cx.c2k = p.c2k; cx.sA = p.sA; cx.cA = p.cA;
    cx.debug = p.debug;

    OUT *dst = reinterpret_cast<OUT *>(p.out) + ((size_t)b * T + t) * (size_t)total + f0;
    cx.cen_x = cen.x;
    cx.cen_y = cen.y;
    cx.cen_z = cen.z;
    cx.hD = 0.5f * (float)(D - 1);
    const float ox = cx.cen_x - gs.half;
    cx.oy = cx.cen_y - gs.half;
    cx.oz = cx.cen_z - gs.half;

    const float4 *rec = p.rec + (size_t)b * N + r0;
    const int count = r1 - r0;
    if (count <= 0) {           // uniform: nothing can reach this tile
        store_any_tile<ALIGNED, ITERS, NW, OUT>(p, cx, dst, false, false);
        return;
    }
    Xform X;

    // How the wavefronts share the work: the `nsplit` wavefronts of a set take the atoms of
    // the span in turn (atom e goes to lane e / nsplit of member e % nsplit, round after
    // round) and every set works through the plane pairs pA0, pA0 + 2, ... pA1.  Usually
    // there is one set (all wavefronts, all pairs); four wavefronts on a tile with exactly
    // two plane pairs form two sets of two, one per pair.
    int nsplit = NW, sub = wave, pA0 = i_lo, pA1 = i_hi;
    if (NW == 4 && i_hi - i_lo >= 2 && i_hi - i_lo <= 3) {
        nsplit = 2;
        sub = wave & 1;
        pA0 = i_lo + 2 * (wave >> 1);
        pA1 = min(pA0 + 1, i_hi);
    }
    // FUSED: an atom's type, coordinates and radius are requested together (one trip to memory),
    // whatever the type turns out to be; finish_raw transforms, culls and filters by type with
    // the prep kernel's arithmetic and tests.
    struct RawAtom {
        int te;
        float cc[3], rad;
    };
    auto fetch_raw = [&](int base) {
        RawAtom ra;
        int ec = min(base + lane * nsplit + sub, count - 1);            // count >= 1 here
        if (NW > 1) ec = list[ec];
        ra.te = NW > 1 ? t : p.raw.types[(size_t)b * N + ec];           // (the list has type t only)
        const float *c3 = p.raw.coords + ((size_t)b * N + ec) * 3;
        ra.cc[0] = c3[0]; ra.cc[1] = c3[1]; ra.cc[2] = c3[2];
        ra.rad = p.raw.radii[gs.radius_type_indexed ? (size_t)t : (size_t)b * N + ec];
        return ra;
    };
    auto finish_raw = [&](const RawAtom &ra, int e) {
        Atom at;
        at.a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (e < count && ra.te == t) {
            float pp[3];
            apply_xform(X, ra.cc, pp);
            const float r = gs.radius_scale * ra.rad;
            const float reach = BINARY ? r : r * gs.c;
            const float org[3] = {ox, cx.oy, cx.oz};
            if (meets_grid(gs, org, pp, r, reach)) at.a = make_float4(pp[0], pp[1], pp[2], r);
        }
        at.valid = at.a.w > 0.0f;
        return at;
    };
    auto load_atom = [&](int base) {
        const int e = base + lane * nsplit + sub;
        Atom at;
        at.a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (FUSED) return finish_raw(fetch_raw(base), e);
        if (e < count) at.a = rec[e];
        at.valid = (e < count) && (at.a.w > 0.0f);
        return at;
    };
    auto test_pair = [&](const Atom &at, int iA) {
        cx.rowA = iA * D - R0;
        cx.rowB = cx.rowA + D;
        const int jaA = max(-cx.rowA, 0), jbA = min(R1 - R0 - cx.rowA, D);
        const int jaB = max(-cx.rowB, 0), jbB = iA < i_hi ? min(R1 - R0 - cx.rowB, D) : 0;
        return pair_test<BINARY>(cx, p, at, ox, iA, jaA, jbA, jaB, jbB);
    };

    // the loads of the first round are under way; clear the tile meanwhile
    // (FUSED: the first atoms are requested before the pose is waited for and worked out)
    Atom at0;
    if (FUSED) {
        const RawAtom ra0 = fetch_raw(0);
        load_xform(X, b, p.raw.centers, p.raw.quats, p.raw.translations);
        at0 = finish_raw(ra0, lane * nsplit + sub);
    } else {
        at0 = load_atom(0);
    }
    {
        const float4 z4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);     // same bits as integer zeros
#pragma unroll
        for (int it = 0; it < 2 * ITERS / NW; ++it)
            reinterpret_cast<float4 *>(lds)[it * 64 * NW + threadIdx.x] = z4;
        if (threadIdx.x < 2) cx.shared[threadIdx.x] = 0;
    }
    // What a wavefront may add to a voxel unwatched.  Alone: all that is safe; the add that carries a sum
    // past 2^32 (64) comes after that and finds one of the two top bits set (16 or more).  Next to others:
    // a share of 46, so that a sum which passes 64 has more than 17 of watched adds, the last of which
    // found 16 or more.
    const int unwatched = NW == 1 ? kSafeHits : 46 / nsplit;
    constexpr bool kAhead = !FUSED;     // the next round's records are requested before this round's tasks run
    // single launch: a watched pass places its first atoms again rather than keep them in registers (six
    // instead of five wavefronts per SIMD: 11.9 instead of 12.7 us for 2040 atoms, 28 x 48^3; small tiles,
    // which are watched more often, 8.0 instead of 8.4 us for 28 x 24^3 at 1 A)
    constexpr bool kAgain = FUSED && NW != 2;
    constexpr int kShare = kDigitHits - 256;        // records of a pass over digits (whole rounds)
    float *park = reinterpret_cast<float *>(dst);
    constexpr int kPark = sizeof(OUT) / sizeof(float);
    auto each = [&](auto body) {
        for (int o = threadIdx.x; o < cx.n; o += 64 * NW) body(o);
    };
    auto sync = [&]() {
        if (NW > 1) __syncthreads();
        else lds_sync();
    };
    SumArgs sa;
    bool any = false;
    const bool short_span = BINARY || count <= kSafeHits;      // nothing needs watching
    const bool single = count <= 64 * nsplit && pA1 - pA0 <= 1;        // one round, one pair of planes
    if (single) {
        PairHit h = test_pair(at0, pA0);
        const bool safe = short_span || (int)__builtin_popcountll(__ballot(h.nA + h.nB > 0)) <= unwatched;
        if (NW > 1) __syncthreads();                // the tile and shared[] are clear
        any = safe ? pair_run<BINARY>(cx, h, Sum::kPlain, sa) : pair_run<BINARY>(cx, h, Sum::kWatch, sa);
    } else {
        if (NW > 1) __syncthreads();
        if (short_span) {
            Atom at = at0;
            for (int base = 0; base < count; base += 64 * nsplit) {
                if (!kAhead && base != 0) at = load_atom(base);
                Atom next = at;
                if (kAhead && base + 64 * nsplit < count) next = load_atom(base + 64 * nsplit);
                for (int iA = pA0; iA <= pA1; iA += 2) {
                    PairHit h = test_pair(at, iA);
                    any = pair_run<BINARY>(cx, h, Sum::kPlain, sa) || any;
                }
                at = next;
            }
        }
    }
    if (short_span) {
        if (NW > 1) {
            if (any && lane == 0) cx.shared[1] = 1;
            __syncthreads();                        // every wavefront's additions are in the tile
            any = cx.shared[1] != 0;
        }
        store_any_tile<ALIGNED, ITERS, NW, OUT>(p, cx, dst, any, !BINARY);
        return;
    }
    Atom at = {};
    if (!kAgain) at = at0;
    Sum sum = Sum::kWatch;
    for (int s0 = 0, s1 = count; ;) {               // a pass over the records [s0, s1): all of them but in rare cases
        int hits[2] = {0, 0};       // what this wavefront can have added to a voxel so far (first pair of planes, others)
        for (int base = single && sum == Sum::kWatch ? s1 : s0; base < s1; base += 64 * nsplit) {
            if ((!kAhead && (kAgain || base != s0)) || sum == Sum::kDigit) at = load_atom(base);
            Atom next = at;
            if (kAhead && sum != Sum::kDigit && base + 64 * nsplit < s1) next = load_atom(base + 64 * nsplit);
            for (int iA = pA0; iA <= pA1; iA += 2) {
                PairHit h = test_pair(at, iA);
                Sum how = sum;
                if (sum == Sum::kWatch) {
                    int &n = hits[iA == pA0 ? 0 : 1];
                    n = min(n + (int)__builtin_popcountll(__ballot(h.nA + h.nB > 0)), kSafeHits + 1);
                    if (n <= unwatched) how = Sum::kPlain;
                }
                any = pair_run<BINARY>(cx, h, how, sa) || any;
            }
            at = next;
        }
        if (sum != Sum::kDigit) {
            bool over = __ballot(sa.seen >= 1u << 30) != 0ull;
            if (NW > 1) {
                if (lane == 0 && any) atomicOr(&cx.shared[1], over ? 3 : 1);
                __syncthreads();                    // every wavefront's additions are in the tile
                any = cx.shared[1] != 0;
                over = (cx.shared[1] & 2) != 0;
            }
            if (!over) break;                       // uniform over the workgroup
            // Some sum has come to 16 and may have passed 64.  What the tile has is the sums modulo 2^32;
            // they wait in the output while a second pass adds up the densities without their last
            // kDigitBits bits.  Fewer than kDigitHits densities of a voxel lose less than 2^32 together,
            // so the two make the exact sum.
            // Hundreds of thousands of records in reach of one tile instead: share by share, in order, a
            // digit at a time, added up in floats.
            sum = Sum::kDigit;
            sa.bits = 32 - kDigitBits;
            sa.shift = kDigitBits;
            if (count < kDigitHits) {
                each([&](int o) { park[(size_t)o * kPark] = cx.tile[o]; });
            } else {
                s1 = kShare;
                each([&](int o) { dst[o] = (OUT)0.0f; });
            }
        } else if (count < kDigitHits) {
            sync();
            each([&](int o) {
                const unsigned long long least = (unsigned long long)__float_as_uint(cx.tile[o]) << kDigitBits;
                const unsigned lost = __float_as_uint(park[(size_t)o * kPark]) - (unsigned)least;
                dst[o] = (OUT)(float)((double)(least + lost) * (1.0 / (double)kFixedOne));
            });
            return;
        } else {
            sync();
            const float step = (float)(1u << sa.shift) / kFixedOne;
            each([&](int o) { dst[o] = (OUT)((float)dst[o] + (float)__float_as_uint(cx.tile[o]) * step); });
            if (sa.shift != 0) {
                sa.shift = 0;
                sa.bits = kDigitBits;
            } else {
                if (s1 == count) return;
                s0 = s1;
                s1 = min(count, s0 + kShare);
                sa.shift = kDigitBits;
                sa.bits = 32 - kDigitBits;
            }
        }
        each([&](int o) { cx.tile[o] = 0.0f; });    // (by the thread that has read the word)
        sync();
    }
    store_any_tile<ALIGNED, ITERS, NW, OUT>(p, cx, dst, any, !BINARY);
}


// The atoms of type t among the first n (at most kFusedAtoms) of an example, in order, into `list`
// (LDS); every wavefront looks at its own run of them.  Returns how many there are.
template <int NW>
__device__ inline int find_atoms(const int32_t *types, int n, int t, unsigned short *list, unsigned short *counts)
{
    constexpr int kPer = kFusedAtoms / (64 * NW);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int first = wave * (64 * kPer);
    int v[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int a = first + k * 64 + lane;
        v[k] = a < n ? types[a] : -1;           // t >= 0
    }
    int mine = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) mine += (int)__builtin_popcountll(__ballot(v[k] == t));
    if (lane == 0) counts[wave] = (unsigned short)mine;
    __syncthreads();
    int at = 0, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int c = counts[w];
        if (w < wave) at += c;
        total += c;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const unsigned long long m = __ballot(v[k] == t);
        if (v[k] == t)
            list[at + (int)__builtin_popcountll(m & ((1ull << lane) - 1ull))] = (unsigned short)(first + k * 64 + lane);
        at += (int)__builtin_popcountll(m);
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(total);
}

// One workgroup per tile.  OUT: float, or double for a grid of doubles.
template <bool BINARY, bool ALIGNED, int ITERS, int NW, typename OUT, bool FUSED = false>
__global__ __launch_bounds__(64 * NW) void forward_kernel(FwdParams p)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];   // tile | marks per wave | shared

    // Workgroup ids go round the 8 XCDs (id % 8), each with its own L2: runs of consecutive
    // tiles, which read the same atom records, can be given to one XCD.
    const GridSpec &gs = p.gs;
    const int D = gs.D, T = p.T, N = p.N;
    // Every kernel argument the preamble needs is fetched now, in one go, instead of in five
    // dependent trips to the scalar cache spread over the preamble: they are inputs of an
    // asm statement whose result (zero) enters the very first computation.  (Not `asm
    // volatile`: after one, the compiler no longer uses scalar loads for the spans.)
    unsigned zero;
    asm("s_mov_b32 %0, 0"
        : "=s"(zero)
        : "s"((unsigned long long)p.range), "s"((unsigned long long)p.rec),
          "s"((unsigned long long)p.gcen), "s"((unsigned long long)p.out), "s"(p.tiles_magic),
          "s"(p.t_magic), "s"(p.div_magic), "s"(p.tiles), "s"(p.pos_major), "s"(p.ka_chunks), "s"(p.ka_last), "s"(p.ka_shift), "s"(p.ka_skip), "s"(p.xcd_shift), "s"(p.n_remap), "s"(D),
          "s"(T), "s"(N), "s"(p.debug), "s"(gs.half));
    if (p.expect_tag != 0u && *p.tag != p.expect_tag) return;      // not the tables this call expects
    unsigned u = blockIdx.x + zero;
    if (p.xcd_shift >= 0 && u < p.n_remap) {
        const unsigned xcd = u & 7u, slot = u >> 3, sh = (unsigned)p.xcd_shift;
        u = ((slot >> sh) << (sh + 3)) + (xcd << sh) + (slot & ((1u << sh) - 1u));
    }
    // Keep-alive read: the tables the prep kernel wrote (records, spans, poses: a few MB) are read
    // example by example, so those of the later examples would lie untouched while hundreds of
    // MB of stores pass and be written back to HBM before their turn -- and a read that has to
    // come from HBM while the chip streams stores costs far more than its bytes.  Every
    // wavefront therefore also reads 1 KB of the tables, at a position scattered by its id
    // (the result is not used): every line is touched every few microseconds and stays cached.
    float4 ka = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (p.ka_chunks) {
        const unsigned c = __umulhi((blockIdx.x + zero) * 2654435761u, p.ka_chunks);
        const unsigned off = min(c << p.ka_shift, p.ka_last) + ((threadIdx.x & 63u) << 4);
        if ((threadIdx.x & 63u) < (1u << (p.ka_shift - 4)) &&   // the chunk's lanes, 16 bytes each
            ((blockIdx.x + zero) & p.ka_skip) == 0u)            // (every wavefront, or one in 2, 4, 8)
            ka = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(p.rec) + off);
    }
    const unsigned uq = div_u32(u, p.tiles_magic), ur = u - uq * p.tiles;
    const unsigned chan = p.pos_major ? ur : uq;
    const unsigned tile_in_chan = p.pos_major ? uq : ur;
    const int b = (int)div_u32(chan, p.t_magic);
    const int t = (int)chan - b * T;
    if (FUSED) {
        // small problems: no tables; the grid centre is the example's centre, the candidates are
        // the example's atoms (tile_body transforms and filters them)
        const TileGeom tgf = tile_geom<ALIGNED, ITERS>(p, D, tile_in_chan, chan);
        if (!ALIGNED && tgf.f1 <= tgf.f0) return;
        float4 cenf = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (p.raw.centers) {
            cenf.x = p.raw.centers[3 * b];
            cenf.y = p.raw.centers[3 * b + 1];
            cenf.z = p.raw.centers[3 * b + 2];
        }
        int n = N;
        if (p.raw.natoms) {
            n = p.raw.natoms[b];
            n = n < 0 ? 0 : (n > N ? N : n);
        }
        const unsigned short *list = nullptr;
        if (NW > 1) {
            unsigned short *out = reinterpret_cast<unsigned short *>(lds + ITERS * 512 + NW * (kTaskCap / 4) + 4);
            n = find_atoms<NW>(p.raw.types + (size_t)b * N, n, t, out, out + kFusedAtoms);
            list = out;
        }
        tile_body<BINARY, ALIGNED, ITERS, NW, OUT, true>(p, lds, b, t, tgf, 0, n, cenf, list);
        return;
    }
    const size_t group = (size_t)b * T + t;
    // All the scalar loads of the preamble are issued together (one trip to L2, which is
    // slow while the chip streams stores): the span of records that can reach the planes
    // of the tile (counted from the example's first record) and the grid centre.
    const int2 *span = p.range + group * D;
    const float4 cen = *reinterpret_cast<const float4 *>(p.gcen + 4 * b);   // one 16-byte load
    const TileGeom tg = tile_geom<ALIGNED, ITERS>(p, D, tile_in_chan, chan);
    if (!ALIGNED && tg.f1 <= tg.f0) return;
    int r0 = 0, r1 = 0;
    if (!MG_DEBUG_IS(p, 3)) {   // timing aid 3: nothing but the zero stores
        r0 = span[tg.i_lo].x;
        r1 = span[tg.i_hi].y;
    }
    asm volatile("" ::"s"(r0), "s"(r1), "s"(cen.x), "s"(cen.y), "s"(cen.z));  // all in flight before the first wait
    if (MG_DEBUG_IS(p, 2)) r1 = r0;
    tile_body<BINARY, ALIGNED, ITERS, NW, OUT>(p, lds, b, t, tg, r0, r1, cen);
    asm volatile("" ::"v"(ka.x), "v"(ka.y), "v"(ka.z), "v"(ka.w));     // the keep-alive read is waited for here
}


// ---------------------------------------------------------------------------
// Vector types, real density: kVecGroup channels of one spatial tile per wavefront.
//
// Every atom feeds every channel, and the channels differ only in the radius that scales
// the distance (radii are looked up by type id) and in the atom's weight.  One pass over the
// atoms in reach of the tile therefore serves several channels: the records are loaded and
// tested against the tile's rows once, the tasks are staged once, and per voxel the squared
// distance x'^2 (in units of rmax/sqrt(k), rmax the widest radius of the group) is worked
// out once; channel q rescales it, x'^2_q = x'^2 (rmax/r_q)^2, evaluates its density and adds
// w_q rho_q into its own tile in LDS.  Beyond channel q's own cutoff rho_q is 0 by its
// formula, so the voxels of the widest sphere that a narrower one does not reach add nothing.
// The channels are taken in order of radius (chan_order, written by the prep kernel), so the
// spheres of a group are nearly the same size.
// The Gaussian and the quadratic tail are taken as a product, without a select between them:
//   rho(x) = exp(-2 min(x, g)^2) clamp(2g (c - x), 0, 1)^2
// (2g (c - g) = 1 and A = 4 g^2 exp(-2 g^2), so the second factor is 1 up to g and the tail's
// A (x - c)^2 over exp(-2 g^2) beyond):
//   w rho_q = w exp2(max(-ratio2_q x'^2, -g^2 k)) clamp(2gc - s tq_q, 0, 1)^2,   s = sqrt(x'^2).
// The weight, with the steps of the fixed point, is all a chord needs per channel; the lanes that walk
// the chord fetch it from the lane that holds the atom.  It is a factor and not part of the exponent: an
// exponent of log2|w| + 25 is rounded at 2^-20, which cost 38 -> 34 instructions per step but made the
// error of weights of one and more 2.5 times as large (2.1e-7 -> 5.1e-7).
// Bound by vector instruction issue: 38 instructions per step of 64 chords and four channels (some 137 cycles: 24
// of them at 2.3, nine at 4.4, the five roots and exponentials at 8.5), with 54 % of the lanes inside the
// sphere; issue is 0.45 of the kernel's 0.51 ms on 50 x 2040 atoms, 28 x 48^3.  Measured and slower, us a call against 501: chords cut into slots of four voxels and
// queued in LDS (7 % fewer instructions, 12 instead of 16 wavefronts per CU: 612 us); tasks in order of the
// row's distance from the atom (523 us); tile rows padded in LDS (half the bank conflicts, 509 us); no chords at
// all, a voxel per lane in bricks of 4 x 4 x 4 that visit the atoms in reach one after the other, sums in
// doubles, far visits with the tail's half of the density only (541 us: 30 % of the lanes are inside, a
// visit of seven channels takes 290 cycles, 145 in the tail).  A clamped multiply in place of a med3 was 1 %
// faster, for one rounding more, and is not taken.
// ---------------------------------------------------------------------------
constexpr int kVecGroup = 4;

struct VecGroup {           // wave-uniform: the channels of this workgroup
    int chan[kVecGroup];        // channel index (for dead slots: any valid channel)
    bool live[kVecGroup];       // slot q holds a channel with a positive radius
    float nr2[kVecGroup];       // -(rmax / r_q)^2
    float tq[kVecGroup];        // 2g/sqrt(k) rmax / r_q
    float r2[kVecGroup];        // binary mode: r_q * r_q (float, as the predicate's right-hand side)
    float rmax;
    float ng2k, tc;             // -g^2 k; 2g c
};

struct VecAtom {            // per atom, per channel of the group
    float w[kVecGroup];         // w_q; fixed point: in steps
    int neg;                    // bit q: w_q < 0  (binary mode: bit q: w_q > 0, the atom marks channel q)
};

// Run the staged tasks [0, ntasks): one (atom, row) chord per lane, kVecGroup channels per voxel.
// tiles: channel q's tile starts at cx.tile + q * stride floats.
template <bool FIXED, bool SIGNED>
__device__ inline void run_tasks_group(const TileCtx &cx, const VecGroup &vg, const Cand &cd,
                                       const VecAtom &va, int stride, int ntasks)
{
    int carry = 0;
    for (int base = 0; base < ntasks; base += 64) {
        const int tau = base + cx.lane;
        bool act = tau < ntasks;
        const int owner = max(carry, wave_inclusive_max((int)cx.marks[tau]));
        carry = bcast(owner, 63);
        const int src = (act ? owner - 1 : 0) << 2;
        const float fy = fetch(src, cd.c0), fz = fetch(src, cd.c1), stepk = fetch(src, cd.c2),
                    inv_stepk = fetch(src, cd.c3);
        const float pxA = fetch(src, cd.pxA), pxB = fetch(src, cd.pxB);
        const int pack = __builtin_amdgcn_ds_bpermute(src, cd.pack);
        const int k = tau - __builtin_amdgcn_ds_bpermute(src, cd.start);   // row number within the atom
        float w[kVecGroup], half[kVecGroup];
#pragma unroll
        for (int q = 0; q < kVecGroup; ++q) {
            w[q] = fetch(src, va.w[q]);
            half[q] = SIGNED ? copysignf(kAlmostHalf, w[q]) : kAlmostHalf;
        }
        const int nA = (pack >> 10) & 1023;
        const bool inB = k >= nA;
        const int j = inB ? (pack >> 20) + (k - nA) : (pack & 1023) + k;   // row in its plane
        const int trow = (inB ? cx.rowB : cx.rowA) + j;                    // row in the tile
        const float px2 = inB ? pxB : pxA;                                 // plane term of x'^2
        const int clip_lo = trow == 0 ? cx.c0 : 0;
        const int clip_hi = trow == cx.nrows - 1 ? cx.c1 : cx.D - 1;
        float *rowp = cx.tile + (trow * cx.D - cx.c0);
        const float dyk = (((float)j - cx.hD) - fy) * stepk;
        const float x2b = fmaf(dyk, dyk, px2);
        const float rem = cx.c2k - x2b;
        act = act && rem > 0.0f;
        const float hz = __builtin_amdgcn_sqrtf(fmaxf(rem, 0.0f)) * inv_stepk + 1.0e-3f;
        const float fzi = fz + cx.hD;                                       // as a grid index
        const int klo = max(clip_lo, (int)ceilf(fzi - hz));
        const int khi = min(clip_hi, (int)floorf(fzi + hz));
        const int nz = act ? khi - klo + 1 : 0;
        const float z0 = (((float)klo - cx.hD) - fz) * stepk;
        const float fnz = (float)nz;
        float *q0 = rowp + klo;
        float tc = vg.tc;
        asm volatile("" : "+v"(tc));        // keep it in a VGPR across the loop
        for (float fi = 0.0f; fi < fnz; fi += 1.0f, ++q0) {
            const float zs = fmaf(fi, stepk, z0);
            const float x2 = fmaf(zs, zs, x2b);
            const float sx = __builtin_amdgcn_sqrtf(x2);
#pragma unroll
            for (int q = 0; q < kVecGroup; ++q) {
                const float e = __builtin_amdgcn_exp2f(__builtin_amdgcn_fmed3f(x2 * vg.nr2[q], vg.ng2k, 0.0f));
                const float u = __builtin_amdgcn_fmed3f(fmaf(-sx, vg.tq[q], tc), 0.0f, 1.0f);
                const float u2 = u * u;                                     // 0 beyond the cutoff
                if (FIXED) {
                    // w rho 2^kVecFixedBits and a half, truncated: rounded to the nearest fixed-point step
                    const float v = fmaf(e * w[q], u2, half[q]);
                    __hip_atomic_fetch_add(reinterpret_cast<unsigned *>(q0) + q * stride, SIGNED ? (unsigned)(int)v : (unsigned)v,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                } else {
                    // (a weight may be infinite here; beyond the cutoff it adds nothing all the same)
                    __hip_atomic_fetch_add(q0 + q * stride, u > 0.0f ? e * w[q] * u2 : 0.0f, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
    }
    lds_sync();
}

// Binary occupancy for a group of channels: the chord of the widest sphere is walked once, d^2 is
// worked out once per voxel in the fixed float order of the predicate, and channel q is marked
// where the atom's weight is positive and d^2 <= r_q^2.
__device__ inline void run_tasks_group_binary(const TileCtx &cx, const VecGroup &vg, const Cand &cd,
                                              const VecAtom &va, int stride, int ntasks)
{
    int carry = 0;
    for (int base = 0; base < ntasks; base += 64) {
        const int tau = base + cx.lane;
        bool act = tau < ntasks;
        const int owner = max(carry, wave_inclusive_max((int)cx.marks[tau]));
        carry = bcast(owner, 63);
        const int src = (act ? owner - 1 : 0) << 2;
        const float ay = fetch(src, cd.c0), az = fetch(src, cd.c1), reach2 = fetch(src, cd.c3);
        const float pxA = fetch(src, cd.pxA), pxB = fetch(src, cd.pxB);
        const int pack = __builtin_amdgcn_ds_bpermute(src, cd.pack);
        const int k = tau - __builtin_amdgcn_ds_bpermute(src, cd.start);   // row number within the atom
        const int pos = __builtin_amdgcn_ds_bpermute(src, va.neg);         // channels the atom marks
        const int nA = (pack >> 10) & 1023;
        const bool inB = k >= nA;
        const int j = inB ? (pack >> 20) + (k - nA) : (pack & 1023) + k;   // row in its plane
        const int trow = (inB ? cx.rowB : cx.rowA) + j;                    // row in the tile
        const float px2 = inB ? pxB : pxA;                                 // dx^2
        const int clip_lo = trow == 0 ? cx.c0 : 0;
        const int clip_hi = trow == cx.nrows - 1 ? cx.c1 : cx.D - 1;
        float *rowp = cx.tile + (trow * cx.D - cx.c0);
        const float gy = cx.oy + (float)j * cx.res;
        const float dy = gy - ay;
        const float dy2 = dy * dy;
        const float rem = (reach2 - px2) - dy2;
        act = act && rem > 0.0f;
        const float hz = __builtin_amdgcn_sqrtf(fmaxf(rem, 0.0f)) * cx.inv_res + 1.0e-3f;
        const float fz = (az - cx.oz) * cx.inv_res;
        const int klo = max(clip_lo, (int)ceilf(fz - hz));
        const int khi = min(clip_hi, (int)floorf(fz + hz));
        const int nz = act ? khi - klo + 1 : 0;
        const float base2 = px2 + dy2;
        for (int i = 0; i < nz; ++i) {
            const float gz = cx.oz + (float)(klo + i) * cx.res;
            const float dz = gz - az;
            const float d2 = base2 + dz * dz;
#pragma unroll
            for (int q = 0; q < kVecGroup; ++q)
                if (((pos >> q) & 1) && d2 <= vg.r2[q]) rowp[klo + i + q * stride] = 1.0f;
        }
    }
    lds_sync();
}

// Stage the tasks of the hits and run them (as pair_run, for a group of channels).
template <bool BINARY, bool SIGNED>
__device__ inline bool pair_run_group(const TileCtx &cx, const VecGroup &vg, PairHit &h,
                                      const VecAtom &va, int stride, bool fixed)
{
    int todo = h.nA + h.nB;
    if (__ballot(todo > 0) == 0ull) return false;
    while (true) {
        const int incl = wave_inclusive_scan(todo);
        int total = bcast(incl, 63);
        if (total == 0) break;
        bool now = todo > 0;
        if (total > kTaskCap) {     // rare: the rest waits for the next round
            now = now && incl <= kTaskCap;
            total = bcast(wave_inclusive_scan(now ? todo : 0), 63);
            if (total == 0) break;
        }
        if (cx.lane < kTaskCap / 16)
            reinterpret_cast<float4 *>(cx.marks)[cx.lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (now) {
            h.cd.start = incl - todo;
            cx.marks[h.cd.start] = (unsigned char)(cx.lane + 1);
            todo = 0;
        }
        lds_sync();
        if (BINARY) run_tasks_group_binary(cx, vg, h.cd, va, stride, total);
        else if (fixed) run_tasks_group<true, SIGNED>(cx, vg, h.cd, va, stride, total);
        else run_tasks_group<false, SIGNED>(cx, vg, h.cd, va, stride, total);
    }
    return true;
}

// One workgroup of NW wavefronts per (example, group of kVecGroup channels, tile).  The
// wavefronts share the group's tiles in LDS and take the rounds of 64 records in turn; every
// wavefront stages and runs its own tasks.  The tiles accumulate in fixed point; the bound on
// what can reach one voxel is summed up on the way, and a workgroup whose bound passes the
// limit at the end (rare) starts over in floats, all records taken by its first wavefront so
// that the order of the float additions is the same in every run.
template <bool BINARY, bool ALIGNED, int ITERS, int NW, typename OUT>
__global__ __launch_bounds__(64 * NW) void forward_vector_kernel(FwdParams p)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];   // kVecGroup tiles | marks per wave | bound
    constexpr int kTile = ITERS * 512;
    const GridSpec &gs = p.gs;
    const int D = gs.D, T = p.T, N = p.N;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (p.expect_tag != 0u && *p.tag != p.expect_tag) return;      // not the tables this call expects
    const unsigned u = blockIdx.x;
    const unsigned uq = div_u32(u, p.tiles_magic), tile_in_chan = u - uq * p.tiles;
    const int b = (int)div_u32(uq, p.t_magic);          // t_magic: ceil(2^64 / groups)
    const int g = (int)uq - b * (int)p.groups;
    const int2 *span = p.range + (size_t)b * T * D;     // vector types: one record list per example
    const float4 cen = *reinterpret_cast<const float4 *>(p.gcen + 4 * b);
    // (the channels of a group begin at different places of a tile, so their tiles are never shifted)
    const TileGeom tg = tile_geom<true, ITERS>(p, D, tile_in_chan, 0u);
    const int r0 = span[tg.i_lo].x, r1 = span[tg.i_hi].y;

    // the channels of this group and what depends on their radii only
    VecGroup vg;
    vg.rmax = 0.0f;
    vg.ng2k = -p.vg2k;
    vg.tc = p.tc;
    float rq[kVecGroup];
#pragma unroll
    for (int q = 0; q < kVecGroup; ++q) {
        const int pos = g * kVecGroup + q;
        vg.chan[q] = p.chan_order[(size_t)b * T + min(pos, T - 1)];
        rq[q] = gs.radius_scale * p.radii[vg.chan[q]];
        vg.live[q] = pos < T && rq[q] > 0.0f && rq[q] < 1.0e30f;
        if (vg.live[q]) vg.rmax = fmaxf(vg.rmax, rq[q]);
    }
#pragma unroll
    for (int q = 0; q < kVecGroup; ++q) {
        const float ratio = vg.live[q] ? vg.rmax / rq[q] : 1.0f;
        vg.nr2[q] = -(ratio * ratio);
        vg.tq[q] = p.tk * ratio;
        vg.r2[q] = vg.live[q] ? rq[q] * rq[q] : -1.0f;     // (nothing is within a dead channel's radius)
    }

    TileCtx cx;
    cx.tile = lds;
    cx.marks = reinterpret_cast<unsigned char *>(lds + kVecGroup * kTile) + wave * kTaskCap;
    cx.shared = reinterpret_cast<int *>(lds + kVecGroup * kTile + NW * (kTaskCap / 4));
    cx.lane = lane;
    cx.wave = wave;
    cx.D = D;
    cx.n = tg.f1 - tg.f0;
    cx.nrows = tg.R1 - tg.R0;
    cx.c0 = tg.f0 - tg.R0 * D;
    cx.c1 = tg.f1 - 1 - (tg.R1 - 1) * D;
    cx.rowA = 0;
    cx.rowB = 0;
    cx.res = gs.res;
    cx.inv_res = gs.inv_res;
    cx.c2k = p.c2k;
    cx.debug = 0;
    cx.cen_x = cen.x; cx.cen_y = cen.y; cx.cen_z = cen.z;
    cx.hD = 0.5f * (float)(D - 1);
    const float ox = cx.cen_x - gs.half;
    cx.oy = cx.cen_y - gs.half;
    cx.oz = cx.cen_z - gs.half;

    const size_t total = (size_t)D * D * D;
    OUT *out = reinterpret_cast<OUT *>(p.out);
    int negs[kVecGroup] = {0, 0, 0, 0};     // what the negative weights of channel q add up to (1/256 units)
    auto store_all = [&](bool touched, bool fixed) {
#pragma unroll
        for (int q = 0; q < kVecGroup; ++q) {
            if (g * kVecGroup + q >= T) break;              // uniform
            TileCtx cq = cx;
            cq.tile = lds + q * kTile;
            OUT *dst = out + ((size_t)b * T + vg.chan[q]) * total + tg.f0;
            store_any_tile<ALIGNED, ITERS, NW, OUT, true>(p, cq, dst, touched && vg.live[q], fixed,
                                                          (unsigned)negs[q] << (kVecFixedBits - 8));
        }
    };
    const int count = r1 - r0;
    if (count <= 0 || !(vg.rmax > 0.0f)) {      // uniform: nothing can reach these tiles
        store_all(false, false);
        return;
    }

    const float4 *rec = p.rec + (size_t)b * N + r0;
    const int *idx = p.idx + (size_t)b * N + r0;
    const float *wbase = p.weights + (size_t)source_example(p.subgrids, b) * N * T;
    struct Raw {
        float4 a;
        int ai;
    };
    auto load_raw = [&](int base) {
        Raw r;
        r.a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        r.ai = 0;
        if (base + lane < count) {
            r.a = rec[base + lane];
            r.ai = idx[base + lane];
        }
        return r;
    };
    struct Wq {
        float w[kVecGroup];
    };
    auto gather = [&](const Raw &r) {
        Wq o;
        const float *row = wbase + (size_t)r.ai * T;
#pragma unroll
        for (int q = 0; q < kVecGroup; ++q)
            o.w[q] = (r.a.w > 0.0f && vg.live[q]) ? row[vg.chan[q]] : 0.0f;
        return o;
    };
    auto clear_tiles = [&]() {
        const float4 z4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);     // same bits as integer zeros
#pragma unroll
        for (int it = 0; it < kVecGroup * kTile / (256 * NW); ++it)
            reinterpret_cast<float4 *>(lds)[it * 64 * NW + threadIdx.x] = z4;
        if (threadIdx.x < 4 + kVecGroup) cx.shared[threadIdx.x] = 0;
    };

    // One pass over the rounds first, first + stride, ...: returns whether any task ran; adds
    // what the hits can put into one voxel at most to `bound` (1/256 units).  Records and
    // indices are requested two rounds ahead, the weights (gathered through the indices) one
    // round ahead; clear_first: the tiles are cleared while the first loads are in flight.
    auto pass = [&](int first, int stride, bool fixed, bool clear_first, int &bound) {
        bool any = false;
        int add[kVecGroup] = {0, 0, 0, 0};      // what this lane's atoms can add to one voxel of channel q
        int sub[kVecGroup] = {0, 0, 0, 0};      // ... of which negative
        Raw rc = load_raw(64 * first);
        Raw rn = load_raw(64 * (first + stride));
        Wq wc = gather(rc);
        if (clear_first) {
            clear_tiles();
            if (NW > 1) __syncthreads();
        }
        Wq wn = gather(rn);
        for (int base = 64 * first; base < count; base += 64 * stride) {
            const Raw rnn = load_raw(base + 128 * stride);
            // this round's atom: what its chords will need, per channel
            Atom at;
            at.a = rc.a;
            VecAtom va;
            int wb[kVecGroup];      // |w_q| rounded up to 1/256
            va.neg = 0;
            bool wany = false;
#pragma unroll
            for (int q = 0; q < kVecGroup; ++q) {
                if (BINARY) {       // the atom marks the channels where its weight is positive
                    va.w[q] = 0.0f;
                    va.neg |= (wc.w[q] > 0.0f ? 1 : 0) << q;
                    continue;
                }
                const float aw = fabsf(wc.w[q]);
                wb[q] = aw > 0.0f ? (int)ceilf(fminf(aw, 4096.0f) * 256.0f) : 0;
                wany = wany || aw > 0.0f;
                va.w[q] = wc.w[q] * (fixed ? (float)(1 << kVecFixedBits) : 1.0f);
                va.neg |= (wc.w[q] < 0.0f ? 1 : 0) << q;
            }
            at.valid = (rc.a.w > 0.0f) && (BINARY ? va.neg != 0 : wany);
            at.a.w = vg.rmax;
            const bool any_neg = !BINARY && __ballot(at.valid && va.neg != 0) != 0ull;
            if (!BINARY && any_neg) {       // a signed conversion holds less
#pragma unroll
                for (int q = 0; q < kVecGroup; ++q)
                    if (fabsf(wc.w[q]) > kSignedTerm) wb[q] = 1 << 20;
            }
            for (int iA = tg.i_lo; iA <= tg.i_hi; iA += 2) {
                cx.rowA = iA * D - tg.R0;
                cx.rowB = cx.rowA + D;
                const int jaA = max(-cx.rowA, 0), jbA = min(tg.R1 - tg.R0 - cx.rowA, D);
                const int jaB = max(-cx.rowB, 0), jbB = iA < tg.i_hi ? min(tg.R1 - tg.R0 - cx.rowB, D) : 0;
                PairHit h = pair_test<BINARY>(cx, p, at, ox, iA, jaA, jbA, jaB, jbB);
                if (!BINARY) {
#pragma unroll
                    for (int q = 0; q < kVecGroup; ++q) {
                        const int b = h.nA + h.nB > 0 ? wb[q] : 0;
                        add[q] = min(add[q] + b, 1 << 24);
                        if (any_neg) sub[q] = min(sub[q] + (wc.w[q] < 0.0f ? b : 0), 1 << 24);
                    }
                }
                const bool ran = any_neg ? pair_run_group<BINARY, true>(cx, vg, h, va, kTile, fixed)
                                         : pair_run_group<BINARY, false>(cx, vg, h, va, kTile, fixed);
                any = ran || any;
            }
            rc = rn;
            wc = wn;
            rn = rnn;
            wn = gather(rn);
        }
        if (!BINARY) {      // the channel they add most to (summed exactly by DPP adds, no LDS traffic)
#pragma unroll
            for (int q = 0; q < kVecGroup; ++q)
                bound = max(bound, min(bcast(wave_inclusive_scan(add[q]), 63), 1 << 26));
            if (__ballot((sub[0] | sub[1] | sub[2] | sub[3]) != 0) != 0ull) {
#pragma unroll
                for (int q = 0; q < kVecGroup; ++q) negs[q] = min(bcast(wave_inclusive_scan(sub[q]), 63), 1 << 26);
            }
        }
        return any;
    };

    const int limit = (int)(kFixedLimit * 256.0f);
    int bound = 0;
    bool fixed = !BINARY;       // (binary tiles hold 0.0f / 1.0f as they are)
    bool any = pass(wave, NW, fixed, true, bound);
    if (NW > 1) {
        if (lane == 0) {
            atomicAdd(&cx.shared[0], bound);
            if (any) cx.shared[1] = 1;
#pragma unroll
            for (int q = 0; q < kVecGroup; ++q)
                if (negs[q] != 0) atomicAdd(&cx.shared[4 + q], negs[q]);
        }
        __syncthreads();                    // every wavefront's additions are in the tiles
        bound = cx.shared[0];
        any = cx.shared[1] != 0;
#pragma unroll
        for (int q = 0; q < kVecGroup; ++q) negs[q] = __builtin_amdgcn_readfirstlane(cx.shared[4 + q]);
    }
    if (!BINARY && bound > limit) {         // uniform over the workgroup: the sums may not fit; again, in floats
        if (NW > 1) __syncthreads();        // shared[] has been read by all
        fixed = false;
        clear_tiles();
        if (NW > 1) __syncthreads();
        int unused = 0;
        if (wave == 0) pass(0, 1, false, false, unused);
        if (NW > 1) __syncthreads();
    }
    store_all(any, fixed);
}

}  // namespace

// Whether a channel's tiles lie on boundaries of the whole output (tile_geom).  That takes one tile more per
// channel, which pays where several of them are whole: from three tiles' floats on.  28 channels of 1000
// atoms, 200 examples (15^3 and less) to 68 (25^3), shifted / not, us: 5^3 23.1 / 19.3, 9^3 31.4 / 27.3, 13^3
// 47.5 / 37.8, 14^3 44.6 / 37.6, 15^3 42.1 / 46.4, 17^3 48.1 / 47.9, 19^3 49.8 / 47.1, 21^3 44.3 / 48.8, 25^3
// 39.9 / 45.5; only 11^3 gains below that (33.6 / 37.7).
static bool tiles_shift(int D, int tile_floats)
{
    return D % 4 != 0 && (long long)D * D * D >= 3LL * tile_floats;
}

ForwardGeometry forward_geometry(int D, int tile_floats, bool shifted)
{
    ForwardGeometry fg;
    fg.tile_floats = tile_floats;
    const long long total = (long long)D * D * D;
    // (shifted: a channel may begin at the last float of a tile)
    fg.tiles = (int)((total + (shifted ? tile_floats - 1 : 0) + tile_floats - 1) / tile_floats);
    return fg;
}

namespace {
unsigned long long magic64(unsigned d)      // ceil(2^64 / d); 0 stands for d == 1
{
    if (d <= 1) return 0ull;
    const unsigned long long q = ~0ull / d;             // floor((2^64 - 1) / d)
    return q + 1ull;        // = ceil(2^64 / d): d >= 2 never divides 2^64 - 1 and 2^64 both, and
                            // when d divides 2^64, q = 2^64/d - 1
}
}  // namespace

// Vector types (real density and binary occupancy): one workgroup per (example, group of kVecGroup
// channels, tile).
static hipError_t launch_forward_vector(const GridSpec &gs, const Batch &bt, const Workspace &ws,
                                        void *out, bool out_is_double, int tile_floats,
                                        int waves_per_tile, unsigned expect_tag, KernelEvents ev,
                                        hipStream_t stream)
{
    // 2048-float tiles and four wavefronts per workgroup: the four channel tiles of a group take
    // 33 KB of LDS, so four workgroups (sixteen wavefronts, what 98 registers allow too) fit a CU.
    // Measured on the 48^3 batch of 50 x 2040 atoms x 28 channels (0.51 ms now): relative to it, 1024
    // floats x 2 wavefronts +10 % (each tile tests the atoms in reach anew), 2048 x 2 and 1024 x 1
    // +43 % (too few wavefronts), 512 x 1 +33 %.  A grid of doubles takes 512 voxels per tile.
    if (tile_floats != 512 && tile_floats != 1024 && tile_floats != 2048) tile_floats = 2048;
    if (out_is_double) tile_floats = 512;
    const ForwardGeometry fg = forward_geometry(gs.D, tile_floats);
    FwdParams p;
    p.gs = gs;
    p.shifted = 0u;
    p.rec = ws.rec;
    p.idx = ws.idx;
    p.range = ws.range;
    p.weights = bt.weights;
    p.radii = bt.radii;
    p.gcen = ws.gcen;
    p.chan_order = ws.chan_order;
    p.tag = ws.tag;
    p.expect_tag = expect_tag;
    p.raw = RawInputs{};
    p.groups = (unsigned)((bt.T + kVecGroup - 1) / kVecGroup);
    p.out = out;
    p.subgrids = bt.sub.count; p.N = bt.N; p.T = bt.T;
    p.tile_floats = fg.tile_floats;
    p.div_magic = ((1ULL << 40) + (unsigned long long)gs.D - 1ULL) / (unsigned long long)gs.D;
    p.pos_major = 0u;
    p.tiles = (unsigned)fg.tiles;
    p.tiles_magic = magic64(p.tiles);
    p.t_magic = magic64(p.groups);
    p.xcd_shift = -1;
    p.n_remap = 0;
    p.debug = 0;
    p.ka_chunks = 0;
    p.ka_last = 0;
    p.ka_shift = 8;
    p.ka_skip = 0;
    const double k = 2.8853900817779268;        // 2 / ln 2
    p.sk = (float)std::sqrt(k);
    p.inv_sk = (float)(1.0 / std::sqrt(k));
    p.c2k = (float)((double)gs.c * (double)gs.c * k);
    // (beyond x = 100 the density is 0 in float whatever the branch: larger g need no larger constants)
    const double g2 = std::fmax(std::fmin((double)gs.g2, 1.0e4), 1.0e-30), gr = std::sqrt(g2);
    p.vg2k = (float)(g2 * k);
    p.tk = (float)(2.0 * gr / std::sqrt(k));
    p.tc = (float)(2.0 * g2 + 1.0);
    const unsigned long long wgs = (unsigned long long)bt.B * p.groups * fg.tiles;
    if (wgs > 0x7fffffffULL) return hipErrorInvalidValue;
    // four wavefronts per workgroup by default: they share the tiles, so four times as many
    // wavefronts are resident for the same LDS (the kernel is bound by vector arithmetic and
    // needs them to keep the SIMDs busy)
    int nw = waves_per_tile == 0 ? 4 : waves_per_tile;
    if (tile_floats == 512 || out_is_double) nw = 1;
    if (nw > tile_floats / 512) nw = tile_floats / 512;
    const size_t lds_bytes = (size_t)kVecGroup * tile_floats * sizeof(float) + (size_t)nw * kTaskCap +
                             (4 + kVecGroup) * sizeof(int);
    const bool aligned = (gs.D % 4 == 0) && (((uintptr_t)out & 15u) == 0);
    const dim3 blk(64 * nw), grd((unsigned)wgs);
#define MG_VEC(Al, It, Nw, Ot)                                                                        \
    do {                                                                                              \
        if (gs.binary)                                                                                \
            hipExtLaunchKernelGGL((forward_vector_kernel<true, Al, It, Nw, Ot>), grd, blk,            \
                                  (uint32_t)lds_bytes, stream, ev.start, ev.stop, 0, p);              \
        else                                                                                          \
            hipExtLaunchKernelGGL((forward_vector_kernel<false, Al, It, Nw, Ot>), grd, blk,           \
                                  (uint32_t)lds_bytes, stream, ev.start, ev.stop, 0, p);              \
    } while (0)
#define MG_VEC_NW(Al, It, Ot) \
    if (nw == 1) MG_VEC(Al, It, 1, Ot); else MG_VEC(Al, It, 2, Ot)
    if (out_is_double) {
        if (aligned) MG_VEC(true, 1, 1, double); else MG_VEC(false, 1, 1, double);
    } else if (tile_floats == 512) {
        if (aligned) MG_VEC(true, 1, 1, float); else MG_VEC(false, 1, 1, float);
    } else if (tile_floats == 1024) {
        if (aligned) { MG_VEC_NW(true, 2, float); } else { MG_VEC_NW(false, 2, float); }
    } else if (nw == 4) {
        if (aligned) MG_VEC(true, 4, 4, float); else MG_VEC(false, 4, 4, float);
    } else {
        if (aligned) { MG_VEC_NW(true, 4, float); } else { MG_VEC_NW(false, 4, float); }
    }
#undef MG_VEC_NW
#undef MG_VEC
    return hipGetLastError();
}

// Small problems (index types into a float grid, no subgrids) in one launch: floats per
// tile (negative: its type's atoms are listed first), 0 where the prep kernel and its tables are quicker.
//   * up to 64 atoms, 2048 in the batch: 1024, one wavefront that looks at all of them in one round
//     (with 65 to 256 it needs several rounds: 8 x 256 atoms, 28 x 48^3 39 us against 27 by the tables);
//   * else, up to 2048 atoms: several wavefronts that first list the tile's type (find_atoms).
//     Tiles of about two x-planes, so that the atoms found need one round: 1024 (two wavefronts)
//     below 37 points a side, else 4096 (four); 2048 where that leaves less than three workgroups
//     per CU and a tile more than one plane.
//     Listing and placing the atoms per tile costs 3.5 us per 3.1 M voxels at 2040 atoms against the
//     10 us of the prep kernel: up to 8 M voxels, or 4096 of the small tiles (tiles, not
//     voxels: a channel of a few points a side is a tile all the same).
// Whole calls, one launch / prep kernel and tables, us, atoms at 0.076 per cubic Angstrom: 100 atoms, 4 x 24^3: 9.1 / 13.6;
// 2040 atoms, 28 x 48^3: 12.0 / 15.7, 14 x 48^3 9.2 / 15.7, 4 x 48^3 13 / 26, 1 x 48^3 20 / 39, 1 x 24^3 at 1 A 45 / 59;
// two of 28 x 48^3 14.7 / 18.7, three of 24 x 48^3 (8 M voxels) 17.4 / 21.1, four of 28 x 48^3 22.0 / 23.4; 14 x 64^3 11.6 / 17.2.
// Small tiles: 2000 of them are quicker in one launch (62 x 8 x 16^3 of 500 atoms 14.8 / 17.1, 10 x 14 x 24^3 11.7 / 13.7,
// 4 x 14 x 32^3 9.7 / 11.8; but 71 x 28 x 8^3 13.2 / 14.7, 142 x 14 x 8^3 of 2040 20.0 / 17.9), 3000 alike (93 x 8 x 16^3 of 500
// 19.5 / 19.1, 15 x 14 x 24^3 15.6 / 15.2, 6 x 14 x 32^3 12.3 / 12.4; 53 x 28 x 12^3 of 2040 21.2 / 22.8), 4000 slower
// (125 x 8 x 16^3 of 500 22.1 / 20.5, 20 x 14 x 24^3 18.6 / 16.3, 8 x 14 x 32^3 14.9 / 13.8; 71 x 28 x 12^3 of 2040 24.7 / 23.3).  The
// line was drawn when a sort was slower; it would lie at 3000 now.
constexpr int kSmallTotal = 2048;
static int single_launch_tile(const GridSpec &gs, const Batch &bt, bool out_is_double)
{
    if (bt.vec || out_is_double || bt.sub.count != 1 || bt.N > kFusedAtoms) return 0;
    const long long voxels = (long long)bt.B * bt.T * gs.D * gs.D * gs.D;
    const bool large = gs.D >= 37;
    if (bt.N <= 64) return (long long)bt.B * bt.N <= kSmallTotal ? 1024 : 0;
    if (!large) return (long long)bt.B * bt.T * forward_geometry(gs.D, 1024, tiles_shift(gs.D, 1024)).tiles <= 4096 ? -1024 : 0;
    if (voxels <= 8LL << 20) {
        const long long wgs = (long long)bt.B * bt.T * forward_geometry(gs.D, 4096).tiles;
        return wgs < 768 && gs.D < 64 ? -2048 : -4096;
    }
    return 0;
}

bool forward_takes_single_launch(const GridSpec &gs, const Batch &bt, bool out_is_double)
{
    return single_launch_tile(gs, bt, out_is_double) != 0;
}

hipError_t launch_forward(const GridSpec &gs, const Batch &bt, const Workspace &ws, void *out,
                          bool out_is_double, int tile_floats, int waves_per_tile, int xcd_run,
                          int lds_floor, int debug, int tile_order, int keep_alive, bool single_launch,
                          unsigned expect_tag, KernelEvents ev, hipStream_t stream, int keep_alive_stride)
{
    if (bt.vec)
        return launch_forward_vector(gs, bt, ws, out, out_is_double, tile_floats, waves_per_tile, expect_tag, ev,
                                     stream);
    if (tile_floats == 512) tile_floats = 1024;     // the smallest tile of these kernels
    if (waves_per_tile == 0) waves_per_tile = 1;
    bool find = false;          // single launch with find_atoms
    if (single_launch) {        // ids in order
        tile_floats = single_launch_tile(gs, bt, out_is_double);
        find = tile_floats < 0;
        if (find) tile_floats = -tile_floats;
        waves_per_tile = !find ? 1 : (tile_floats == 1024 ? 2 : 4);
        xcd_run = 0;
        tile_order = 0;
        keep_alive = 0;
        lds_floor = 0;
    }
    if (tile_floats == 0) {
        // 4 KB tiles unless a tile meets many records (then the fixed cost per tile counts for
        // more than the shorter life of a small tile): about N/T atoms per channel, of which
        // those within a cutoff sphere's width (taken as 6 A) of the tile's x-plane are read.
        // Measured: 48^3 at 0.5 A with 2040 atoms (20 per tile) 102 us against 111 us with 8 KB
        // tiles; 96^3 at 0.25 A with 8000 atoms (74 per tile) 275 us with 8 KB tiles against 297 us,
        // with 6000 atoms (56 per tile) 281 against 279 us, with 5000 (47) 285 against 275 us.
        const double groups = bt.vec ? 1.0 : (double)bt.T;
        const double planes = 6.0 / (double)gs.res + 1.0;
        const double per_tile = (double)bt.N / groups * (planes < gs.D ? planes / gs.D : 1.0);
        tile_floats = per_tile > 60.0 ? 2048 : 1024;
        if (waves_per_tile > tile_floats / 512) waves_per_tile = tile_floats / 512;
    }
    if (out_is_double) {        // 512 voxels = 4 KB of doubles per one-wavefront workgroup
        tile_floats = 512;
        waves_per_tile = 1;
    }
    const bool out16 = ((uintptr_t)out & 15u) == 0;
    const bool aligned = gs.D % 4 == 0 && out16;
    const bool shifted = out16 && tiles_shift(gs.D, tile_floats);
    const ForwardGeometry fg = forward_geometry(gs.D, tile_floats, shifted);
    FwdParams p;
    p.gs = gs;
    p.shifted = shifted ? 1u : 0u;
    p.rec = ws.rec;
    p.idx = ws.idx;
    p.range = ws.range;
    p.weights = bt.weights;
    p.radii = bt.radii;
    p.gcen = ws.gcen;
    p.chan_order = ws.chan_order;
    p.tag = ws.tag;
    p.expect_tag = single_launch ? 0u : expect_tag;
    p.groups = 0;
    p.raw = raw_inputs(bt);
    p.out = out;
    p.subgrids = bt.sub.count; p.N = bt.N; p.T = bt.T;
    p.tile_floats = fg.tile_floats;
    p.div_magic = ((1ULL << 40) + (unsigned long long)gs.D - 1ULL) / (unsigned long long)gs.D;
    const int iters = tile_floats / 512;
    int nw = waves_per_tile < iters ? waves_per_tile : iters;
    if (iters == 8 && nw < 2) nw = 2;           // 16 KB tiles are built for two or four wavefronts
    p.pos_major = tile_order == 1 ? 1u : 0u;
    p.tiles = p.pos_major ? (unsigned)bt.B * (unsigned)bt.T : (unsigned)fg.tiles;
    p.tiles_magic = magic64(p.tiles);
    p.t_magic = magic64((unsigned)bt.T);
    const unsigned long long groups = (unsigned long long)bt.B * bt.T * fg.tiles;
    p.xcd_shift = -1;
    p.n_remap = 0;
    for (int sh = 0; sh < 16; ++sh)
        if (xcd_run == (1 << sh)) p.xcd_shift = sh;
    if (p.xcd_shift >= 0) {
        const unsigned long long chunk = 8ull << p.xcd_shift;
        p.n_remap = (unsigned)(groups / chunk * chunk);
    }
    p.debug = debug;
    {   // the tables lie one after the other in the workspace, from the records to the grid centres
        const size_t bytes = (size_t)((const char *)(ws.gcen + (size_t)bt.B * 4) - (const char *)ws.rec);
        p.ka_chunks = 0;
        p.ka_last = 0;
        p.ka_skip = keep_alive_stride > 1 ? (unsigned)keep_alive_stride - 1u : 0u;
        // keep_alive: 0 = none, 1 = the default chunk, else the chunk in bytes (256, 512, 1024)
        const unsigned chunk = keep_alive == 1 ? kKeepAliveBytes : (unsigned)keep_alive;
        p.ka_shift = chunk == 1024u ? 10u : (chunk == 512u ? 9u : (chunk == 128u ? 7u : (chunk == 64u ? 6u : 8u)));
        // (vector types are bound by arithmetic and a grid of doubles by its own stores: measured no gain)
        if (keep_alive && !bt.vec && !out_is_double && bytes >= 1024 && bytes < (1ull << 31)) {
            p.ka_chunks = (unsigned)((bytes + chunk - 1) >> p.ka_shift);
            p.ka_last = (unsigned)(bytes - chunk);
        }
    }
    const double k = 2.8853900817779268;        // 2 / ln 2
    p.sk = (float)std::sqrt(k);
    p.inv_sk = (float)(1.0 / std::sqrt(k));
    p.g2k = (float)((double)gs.g2 * k);
    p.c2k = (float)((double)gs.c * (double)gs.c * k);
    p.sA = (float)std::sqrt((double)gs.A / k);
    p.cA = (float)((double)gs.c * std::sqrt((double)gs.A));
    // tile | marks of each wavefront | shared words; lds_floor raises the request to cap how
    // many tiles are resident on a CU
    size_t lds_bytes = (size_t)tile_floats * sizeof(float) + (size_t)nw * kTaskCap + 16;
    if (find) lds_bytes += (kFusedAtoms + 8) * sizeof(unsigned short);
    // 4 KB tiles, one wavefront each: 26 per CU (104 KB of stores in flight) instead of all 32
    // slots measured 98.2 us against 102.4 us on the 48^3 batch (22 to 30 per CU alike)
    if (lds_floor < 0) lds_floor = (tile_floats == 1024 && nw == 1 && !out_is_double && !bt.vec) ? 6144 : 0;
    if (lds_bytes < (size_t)lds_floor) lds_bytes = (size_t)lds_floor;
    const dim3 blk(64 * nw), grd((unsigned)groups);
#define MG_LAUNCH5(Bn, Al, It, Nw) \
    hipExtLaunchKernelGGL((forward_kernel<Bn, Al, It, Nw, float>), grd, blk, (uint32_t)lds_bytes, \
                          stream, ev.start, ev.stop, 0, p)
#define MG_LAUNCH(Bn, Al)                                                       \
    if (out_is_double) {                                                        \
        hipExtLaunchKernelGGL((forward_kernel<Bn, Al, 1, 1, double>), grd, blk,                    \
                              (uint32_t)lds_bytes, stream, ev.start, ev.stop, 0, p);               \
    } else switch (iters * 8 + nw) {                                            \
    case 2 * 8 + 1: MG_LAUNCH5(Bn, Al, 2, 1); break;                            \
    case 2 * 8 + 2: MG_LAUNCH5(Bn, Al, 2, 2); break;                            \
    case 4 * 8 + 1: MG_LAUNCH5(Bn, Al, 4, 1); break;                            \
    case 4 * 8 + 2: MG_LAUNCH5(Bn, Al, 4, 2); break;                            \
    case 4 * 8 + 4: MG_LAUNCH5(Bn, Al, 4, 4); break;                            \
    case 8 * 8 + 2: MG_LAUNCH5(Bn, Al, 8, 2); break;                            \
    case 8 * 8 + 4: MG_LAUNCH5(Bn, Al, 8, 4); break;                            \
    default: return hipErrorInvalidValue;                                       \
    }
    if (single_launch) {
#define MG_FUSED1(Bn, Al, It, Nw)                                                             \
    hipExtLaunchKernelGGL((forward_kernel<Bn, Al, It, Nw, float, true>), grd, blk,            \
                          (uint32_t)lds_bytes, stream, ev.start, ev.stop, 0, p)
#define MG_FUSED(Bn, Al)                                                                      \
    do {                                                                                      \
        if (nw == 1) MG_FUSED1(Bn, Al, 2, 1);                                                 \
        else if (nw == 2) MG_FUSED1(Bn, Al, 2, 2);                                            \
        else if (iters == 4) MG_FUSED1(Bn, Al, 4, 4);                                         \
        else MG_FUSED1(Bn, Al, 8, 4);                                                         \
    } while (0)
        if (gs.binary) { if (aligned) MG_FUSED(true, true); else MG_FUSED(true, false); }
        else           { if (aligned) MG_FUSED(false, true); else MG_FUSED(false, false); }
#undef MG_FUSED
#undef MG_FUSED1
    } else {
        if (gs.binary) { if (aligned) MG_LAUNCH(true, true) else MG_LAUNCH(true, false) }
        else           { if (aligned) MG_LAUNCH(false, true) else MG_LAUNCH(false, false) }
    }
#undef MG_LAUNCH
#undef MG_LAUNCH5
    return hipGetLastError();
}

}  // namespace mg
