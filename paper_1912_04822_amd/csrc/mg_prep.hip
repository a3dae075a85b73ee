// Steps 1 and 2 of the path: per-example coordinate transform, radius lookup,
// bounding-box culling, channel binning and x-plane binning.
//
// Transform (Transformations section of the paper): x' = R(q)(x - c) + c + t,
// q = (w,x,y,z) with (1,0,0,0) the identity.  The arithmetic is double in one
// fixed order (no fused multiply-add; the file is compiled with
// -ffp-contract=off) and the result is rounded once to float, so that the
// binary-occupancy decision downstream is reproducible bit for bit:
//   n  = ((w*w + x*x) + y*y) + z*z          s = 2/n   (n == 0: identity)
//   xs = x*s, ys = y*s, zs = z*s
//   R  = [ 1-(y*ys+z*zs)   x*ys-w*zs      x*zs+w*ys   ]
//        [ x*ys+w*zs       1-(x*xs+z*zs)  y*zs-w*xs   ]
//        [ x*zs-w*ys       y*zs+w*xs      1-(x*xs+y*ys) ]
//   x'_m = (((R_m0*u0 + R_m1*u1) + R_m2*u2) + c_m) + t_m,   u = x - c
//
// Culling is exact: the density is identically zero beyond c(grm)*r, so an
// atom whose cutoff cube misses the grid box contributes nothing.
//
// Usual sizes: one workgroup per example (512 threads up to 2048 atoms of index
// types, 1024 otherwise) does a counting sort of the example's atoms by (type, x-plane bin) in LDS (vector
// types: by bin, with a sort that is stable by itself, see prep_example_vector_kernel):
//   1. every atom: transform, cull, key = type * bins + bin (bins 0 and D+1 are
//      the atoms left / right of the grid, bin D+2 the culled ones), count;
//   2. exclusive scan of the counts = where each (type, bin) starts;
//   3. atoms are placed, each bin is put in atom order (so the order in which
//      the forward kernel sums is fixed), records are written bin by bin;
//   4. for every type and x-plane, the span of records that can reach it.
// Larger examples: several workgroups per example, each sorting its share of the keys
// (prep_range_kernel).
#include <algorithm>

#include "mg_common.h"
#include "mg_wave.h"
#include "mg_xform.h"

namespace mg {

namespace {


template <bool INVERSE>
__global__ __launch_bounds__(256) void transform_kernel(int B, int N, const float *coords,
                                                        const float *centers, const float *quats,
                                                        const float *translations, float *out)
{
    const int b = blockIdx.y;
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= N) return;
    Xform X;
    load_xform(X, b, centers, quats, translations);
    const size_t k = ((size_t)b * N + a) * 3;
    float o[3];
    if (INVERSE)
        apply_xform_inverse(X, coords + k, o);
    else
        apply_xform(X, coords + k, o);
    out[k + 0] = o[0];
    out[k + 1] = o[1];
    out[k + 2] = o[2];
}

// Exclusive prefix sum of `v` over the 64 lanes of the wavefront; *total gets the sum.
// (DPP row shifts and broadcasts: no trips through LDS.)
__device__ inline int wave_exclusive_scan(int v, int *total)
{
    const int incl = wave_inclusive_scan(v);
    *total = __builtin_amdgcn_readlane(incl, 63);
    return incl - v;
}

// The pose, the same in all lanes, in scalar registers: 30 vector registers less.
__device__ inline void keep_scalar(Xform &X)
{
    const auto uniform = [](double v) {
        const long long bits = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_readfirstlane((int)bits), hi = __builtin_amdgcn_readfirstlane((int)(bits >> 32));
        return __longlong_as_double((long long)hi << 32 | (unsigned)lo);
    };
    for (int m = 0; m < 9; ++m) X.R[m] = uniform(X.R[m]);
    for (int m = 0; m < 3; ++m) X.c[m] = uniform(X.c[m]);
    for (int m = 0; m < 3; ++m) X.t[m] = uniform(X.t[m]);
}

// The rotation's rows for the backward pass (with constant indices: an index by lane would keep the whole
// pose in scratch memory).
__device__ inline void store_rotation(const Xform &X, float *rot)
{
    *reinterpret_cast<float4 *>(rot) = make_float4((float)X.R[0], (float)X.R[1], (float)X.R[2], (float)X.R[3]);
    *reinterpret_cast<float4 *>(rot + 4) = make_float4((float)X.R[4], (float)X.R[5], (float)X.R[6], (float)X.R[7]);
    rot[8] = (float)X.R[8];
}

// Centre of the grid of virtual example b (source example bs); X holds bs's centre (a float
// widened to double, so narrowing it back is exact).
__device__ inline void grid_center(const Subgrids &sub, const Xform &X, int b, int bs, float *gc)
{
    for (int m = 0; m < 3; ++m) gc[m] = (float)X.c[m];
    if (sub.per_side > 1) {
        const int s = b - bs * sub.count;
        const int sxy = s / sub.per_side;
        const int sv[3] = {sxy / sub.per_side, sxy % sub.per_side, s % sub.per_side};
        for (int m = 0; m < 3; ++m) gc[m] = gc[m] + ((float)sv[m] - sub.mid) * sub.step;
    }
}

// Planes on each side of its own that an atom reaches, plus one (past the grid's own planes all are alike: the
// bound keeps the bin numbers made from it within the grid's for any radius).
__device__ inline int planes_reached(const GridSpec &gs, float reach)
{
    return (int)fminf(ceilf(reach * gs.inv_res + 1.0e-3f * gs.res), (float)(gs.D + 2)) + 1;
}

// Vector types: the reach of the widest channel (the lanes of a wavefront read the radii together).
__device__ inline float widest_reach(const GridSpec &gs, const Batch &bt)
{
    float widest = 0.0f;
    for (int k = (int)(threadIdx.x & 63u); k < bt.T; k += 64) widest = fmaxf(widest, gs.radius_scale * bt.radii[k]);
    widest = __int_as_float(bcast(wave_inclusive_max(__float_as_int(widest)), 63));     // (>= 0: ordered like ints)
    return gs.binary ? widest : widest * gs.c;
}

// Vector types: the channels of (virtual) example b in order of radius, for the kernels that
// take several channels of an atom together; called by one wavefront.  NaN and negative
// radii rank as 0, so the result is a permutation whatever the table holds.
__device__ inline void rank_channels(const Batch &bt, const Workspace &ws, int b)
{
    const int T = bt.T, lane = threadIdx.x & 63;
    for (int k0 = 0; k0 < T; k0 += 64) {
        const int k = k0 + lane;
        float mine = k < T ? bt.radii[k] : 0.0f;
        mine = mine > 0.0f ? mine : 0.0f;
        int rank = k;
        if (T <= kRankCap) {
            rank = 0;
            for (int j0 = 0; j0 < T; j0 += 64) {
                float theirs = j0 + lane < T ? bt.radii[j0 + lane] : 0.0f;
                theirs = theirs > 0.0f ? theirs : 0.0f;
                for (int j = 0; j < min(64, T - j0); ++j) {
                    const float other = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(theirs), j));
                    rank += (other < mine || (other == mine && j0 + j < k)) ? 1 : 0;
                }
            }
        }
        if (k < T) ws.chan_order[(size_t)b * T + rank] = k;
    }
}

// ---------------------------------------------------------------------------
// One workgroup per example: counting sort by (type, x-bin) in LDS.
// ---------------------------------------------------------------------------
constexpr int kExThreads = 1024;            // the larger of the two block sizes
constexpr int kExMaxAtoms = 8192;           // 8 atoms per thread (4 in the kernel for N <= 4096)
constexpr size_t kExMaxLds = 64 * 1024;     // two words per (type, bin) key, two per type and two bytes per atom

struct ExLayout {       // LDS, in ints
    int K, Tg, N;
    __host__ __device__ int cnt() const { return 0; }
    __host__ __device__ int pos() const { return K; }
    __host__ __device__ int rmax() const { return 2 * K; }
    __host__ __device__ int rad() const { return 2 * K + Tg; }                  // float[Tg]
    __host__ __device__ int part() const { return 2 * K + 2 * Tg; }
    __host__ __device__ int order() const { return 2 * K + 2 * Tg + 32; }       // ushort[N]
    __host__ __device__ int ints() const { return order() + (N + 1) / 2; }
};

template <int kPer, int NT>
__global__ __launch_bounds__(NT) void prep_example_kernel(GridSpec gs, Batch bt,
                                                                  Workspace ws, unsigned tag,
                                                                  int stop)
{
    extern __shared__ int s_mem[];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int bs = source_example(bt.sub.count, b);       // whose atoms and pose this (virtual) example reads
    const int N = bt.N, T = bt.T, D = gs.D;
    if (MG_STOP_IS(stop, 1)) return;
    const int Tg = T;                   // groups per example
    const int nb = D + 3;               // bins per group; bin D+2 holds the culled atoms
    ExLayout L;
    L.K = Tg * nb; L.Tg = Tg; L.N = N;
    const int K = L.K;
    int *s_cnt = s_mem + L.cnt();
    int *s_pos = s_mem + L.pos();
    int *s_rmax = s_mem + L.rmax();
    float *s_rad = reinterpret_cast<float *>(s_mem + L.rad());
    int *s_part = s_mem + L.part();
    unsigned short *s_order = reinterpret_cast<unsigned short *>(s_mem + L.order());

    // Everything this thread needs from HBM is requested before anything is waited for:
    // its atoms (thread tid owns atoms tid, tid + 1024, ...), the radii table, the pose.
    const int32_t *ty = bt.types + (size_t)bs * N;
    const float *crd = bt.coords + (size_t)bs * N * 3;          // 32-bit offsets from here on
    const float *rad_b = bt.radii + (!gs.radius_type_indexed ? (size_t)bs * N : 0);
    int my_t[kPer];
    float my_c[kPer][3], my_r[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int a = tid + u * NT;
        my_t[u] = -1;
        my_c[u][0] = 0.0f; my_c[u][1] = 0.0f; my_c[u][2] = 0.0f;
        my_r[u] = 0.0f;
        if (a < N) {
            my_t[u] = ty[a];
            my_c[u][0] = crd[a * 3];
            my_c[u][1] = crd[a * 3 + 1];
            my_c[u][2] = crd[a * 3 + 2];
            if (!gs.radius_type_indexed) my_r[u] = rad_b[a];
        }
    }
    // (the radius table too: this thread's entry now, into LDS once the loads have landed)
    const bool rad_table = gs.radius_type_indexed;
    float my_rad = 0.0f;
    if (rad_table && tid < Tg) my_rad = bt.radii[tid];
    int n = N;
    if (bt.natoms) {
        n = bt.natoms[bs];
        n = n < 0 ? 0 : (n > N ? N : n);
    }
    Xform X;
    load_xform(X, bs, bt.centers, bt.quats, bt.translations);
    if (tid == 0) store_rotation(X, ws.rot + b * 12);
    if (b == 0 && tid == 0) *ws.tag = tag;
    float org[3];                   // the grid's first point
    float gc[3];
    grid_center(bt.sub, X, b, bs, gc);
    if (tid == 0) *reinterpret_cast<float4 *>(ws.gcen + b * 4) = make_float4(gc[0], gc[1], gc[2], 0.0f);
    for (int m = 0; m < 3; ++m) org[m] = gc[m] - gs.half;

    if (rad_table) {
        if (tid < Tg) s_rad[tid] = my_rad;
        for (int k = tid + NT; k < Tg; k += NT) s_rad[k] = bt.radii[k];
    }
    if (MG_STOP_IS(stop, 2)) return;
    for (int k = tid; k < K; k += NT) s_cnt[k] = 0;
    for (int k = tid; k < Tg; k += NT) s_rmax[k] = 0;
    __syncthreads();

    // ---- 1. key and a slot inside its bin for every atom ----
    int my_key[kPer], my_slot[kPer];
    float my_p[kPer][3], my_w[kPer];        // transformed position, radius (0: culled)
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int a = tid + u * NT;
        my_key[u] = 0xFFFF;
        my_slot[u] = 0;
        my_w[u] = 0.0f;
        my_p[u][0] = 0.0f; my_p[u][1] = 0.0f; my_p[u][2] = 0.0f;
        if (a >= N) continue;
        const int tg = my_t[u];
        const bool member = a < n && tg >= 0 && tg < Tg;
        if (member) {
            apply_xform(X, my_c[u], my_p[u]);
            const float r = gs.radius_scale * (gs.radius_type_indexed ? s_rad[tg] : my_r[u]);
            const float reach = gs.binary ? r : r * gs.c;
            const bool live = meets_grid(gs, org, my_p[u], r, reach);
            int bin = D + 2;
            if (live) {
                const float f = floorf((my_p[u][0] - org[0]) * gs.inv_res);
                bin = f < 0.0f ? 0 : (f >= (float)D ? D + 1 : (int)f + 1);
                atomicMax(&s_rmax[tg], __float_as_int(r));      // r > 0: ordered like ints
                my_w[u] = r;
            }
            my_key[u] = tg * nb + bin;
            my_slot[u] = atomicAdd(&s_cnt[my_key[u]], 1);
            ws.alive[(size_t)b * N + a] = live ? 1 : 0;
        } else {
            ws.alive[(size_t)b * N + a] = 0;        // no group owns this atom
        }
    }
    __syncthreads();
    if (MG_STOP_IS(stop, 3)) return;

    // ---- 2. exclusive scan of the counts ----
    const int chunk = (K + NT - 1) / NT;
    const int k0 = min(K, tid * chunk), k1 = min(K, k0 + chunk);
    int mine = 0;
    for (int k = k0; k < k1; ++k) mine += s_cnt[k];
    int wtotal;
    int run = wave_exclusive_scan(mine, &wtotal);
    if ((tid & 63) == 0) s_part[tid >> 6] = wtotal;
    __syncthreads();
    if (tid < 64) {
        int t16;
        const int v = tid < NT / 64 ? s_part[tid] : 0;
        const int ex = wave_exclusive_scan(v, &t16);
        if (tid < NT / 64) s_part[tid] = ex;
        if (tid == 0) s_part[NT / 64] = t16;
    }
    __syncthreads();
    run += s_part[tid >> 6];
    const int total = s_part[NT / 64];      // atoms that belong to a group
    for (int k = k0; k < k1; ++k) {
        s_pos[k] = run;
        run += s_cnt[k];
    }
    __syncthreads();
    if (MG_STOP_IS(stop, 4)) return;

    // ---- 3. atoms into their bins in any order; group descriptors and spans meanwhile ----
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (my_key[u] != 0xFFFF) s_order[s_pos[my_key[u]] + my_slot[u]] = (unsigned short)(tid + u * NT);
    for (int tg = tid; tg < Tg; tg += NT) {
        const int first = s_pos[tg * nb];
        const int dead = s_pos[tg * nb + D + 2];
        const int end = tg + 1 < Tg ? s_pos[(tg + 1) * nb] : total;
        ws.meta[(size_t)b * T + tg] = make_int4(first, dead - first, end - first, 0);
    }
    for (int e = tid; e < Tg * D; e += NT) {
        const int tg = e / D, i = e - tg * D;
        // plane i is reached from bins [i - Rv, i + Rv + 1]
        const float rmax = __int_as_float(s_rmax[tg]) * (gs.binary ? 1.0f : gs.c);
        const int Rv = planes_reached(gs, rmax);
        const int lo = max(0, i - Rv), hi = min(D + 1, i + Rv + 1);
        ws.range[((size_t)b * T + tg) * D + i] = make_int2(s_pos[tg * nb + lo], s_pos[tg * nb + hi + 1]);
    }
    __syncthreads();
    if (MG_STOP_IS(stop, 5)) return;

    // ---- 4. every atom writes its record where its rank inside the bin puts it ----
    // (rank = how many atoms of the bin have a smaller index: the order in which the
    // forward kernel sums is fixed; the order of culled atoms does not matter)
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int key = my_key[u];
        if (key == 0xFFFF) continue;
        const int a = tid + u * NT;
        const int lo = s_pos[key];
        int rank = my_slot[u];
        if (key - (key / nb) * nb != D + 2) {
            const int cnt = s_cnt[key];
            rank = 0;
            for (int i = 0; i < cnt; ++i) rank += s_order[lo + i] < a ? 1 : 0;
        }
        ws.rec[(size_t)b * N + lo + rank] = make_float4(my_p[u][0], my_p[u][1], my_p[u][2], my_w[u]);
        ws.idx[(size_t)b * N + lo + rank] = a;
        ws.rchan[(size_t)b * N + lo + rank] = key / nb;
    }
}

// ---------------------------------------------------------------------------
// Vector types, one workgroup per example: counting sort by x-bin in LDS.  All atoms are in one group, so
// bins are long (34 atoms each on 2040 atoms and 48 planes), and putting every bin in atom order by
// counting (as for index types) was 7 of 18 us.  The sort is stable by itself instead: every wavefront has a
// run of consecutive atoms and its own count of every bin, looks at 64 atoms at a time and tells by
// ballots over the bits of the key which of its lanes hold the same bin; the counts are summed over bins
// and, within a bin, over wavefronts.
// ---------------------------------------------------------------------------
template <int kPer>
__global__ __launch_bounds__(kExThreads) void prep_example_vector_kernel(GridSpec gs, Batch bt, Workspace ws,
                                                                         unsigned tag, int stop)
{
    constexpr int NT = kExThreads, NW = NT / 64;
    extern __shared__ int s_mem[];
    __shared__ int s_part[NW + 1];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bs = source_example(bt.sub.count, b);       // whose atoms and pose this (virtual) example reads
    const int N = bt.N, D = gs.D;
    if (MG_STOP_IS(stop, 1)) return;
    const int nb = D + 3;               // bin D+2 holds the culled atoms
    unsigned short *s_cnt = reinterpret_cast<unsigned short *>(s_mem);     // [nb][NW], later where they begin

    // everything this thread needs from HBM is requested before anything is waited for
    const float *crd = bt.coords + (size_t)bs * N * 3;
    float my_c[kPer][3];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int a = (wave * kPer + u) * 64 + lane;
        my_c[u][0] = 0.0f; my_c[u][1] = 0.0f; my_c[u][2] = 0.0f;
        if (a < N) {
            my_c[u][0] = crd[a * 3];
            my_c[u][1] = crd[a * 3 + 1];
            my_c[u][2] = crd[a * 3 + 2];
        }
    }
    int n = N;
    if (bt.natoms) {
        n = bt.natoms[bs];
        n = n < 0 ? 0 : (n > N ? N : n);
    }
    Xform X;
    load_xform(X, bs, bt.centers, bt.quats, bt.translations);
    if (tid == 0) store_rotation(X, ws.rot + b * 12);
    if (b == 0 && tid == 0) *ws.tag = tag;
    const float reach = widest_reach(gs, bt);
    float org[3];                   // the grid's first point
    float gc[3];
    grid_center(bt.sub, X, b, bs, gc);
    if (tid == 0) *reinterpret_cast<float4 *>(ws.gcen + b * 4) = make_float4(gc[0], gc[1], gc[2], 0.0f);
    for (int m = 0; m < 3; ++m) org[m] = gc[m] - gs.half;
    for (int k = tid; k < (nb * NW + 1) / 2; k += NT) s_mem[k] = 0;
    __syncthreads();
    if (MG_STOP_IS(stop, 2)) return;

    // ---- 1. bin and place within (bin, wavefront) for every atom ----
    int my_key[kPer], my_slot[kPer];
    float my_p[kPer][3];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int a = (wave * kPer + u) * 64 + lane;
        const bool member = a < n;
        bool live = false;
        int key = 0;
        my_p[u][0] = my_p[u][1] = my_p[u][2] = 0.0f;
        if (member) {
            apply_xform(X, my_c[u], my_p[u]);
            live = meets_grid(gs, org, my_p[u], 1.0f, reach);
            const float f = floorf((my_p[u][0] - org[0]) * gs.inv_res);
            key = !live ? D + 2 : f < 0.0f ? 0 : (f >= (float)D ? D + 1 : (int)f + 1);
        }
        if (a < N) ws.alive[(size_t)b * N + a] = live ? 1 : 0;
        // the lanes with the same key
        unsigned long long same = __ballot(member);
        for (int bit = 1; bit < nb; bit <<= 1) {
            const bool set = (key & bit) != 0;
            const unsigned long long m = __ballot(set);
            same &= set ? m : ~m;
        }
        my_key[u] = member ? key : -1;
        my_slot[u] = 0;
        if (member) {
            const int before = (int)__builtin_popcountll(same & ((1ull << lane) - 1ull));
            unsigned short *c = &s_cnt[key * NW + wave];
            const int base = *c;
            my_slot[u] = base + before;
            lds_sync();
            if (before == 0) *c = (unsigned short)(base + (int)__builtin_popcountll(same));
        }
        lds_sync();
    }
    if (wave == NW - 1) rank_channels(bt, ws, b);       // (while the others wait)
    __syncthreads();
    if (MG_STOP_IS(stop, 3)) return;

    // ---- 2. exclusive scan of the counts ----
    const int K = nb * NW;
    const int chunk = (K + NT - 1) / NT;
    const int k0 = min(K, tid * chunk), k1 = min(K, k0 + chunk);
    int mine = 0;
    for (int k = k0; k < k1; ++k) mine += s_cnt[k];
    int wtotal;
    int run = wave_exclusive_scan(mine, &wtotal);
    if (lane == 0) s_part[wave] = wtotal;
    __syncthreads();
    if (wave == 0) {
        int t16;
        const int v = lane < NW ? s_part[lane] : 0;
        const int ex = wave_exclusive_scan(v, &t16);
        if (lane < NW) s_part[lane] = ex;
        if (lane == 0) s_part[NW] = t16;
    }
    __syncthreads();
    run += s_part[wave];
    for (int k = k0; k < k1; ++k) {
        const int c = s_cnt[k];
        s_cnt[k] = (unsigned short)run;
        run += c;
    }
    __syncthreads();
    if (MG_STOP_IS(stop, 4)) return;

    // ---- 3. records, group descriptor, spans ----
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (my_key[u] < 0) continue;
        const size_t at = (size_t)b * N + s_cnt[my_key[u] * NW + wave] + my_slot[u];
        ws.rec[at] = make_float4(my_p[u][0], my_p[u][1], my_p[u][2], my_key[u] == D + 2 ? 0.0f : 1.0f);
        ws.idx[at] = (wave * kPer + u) * 64 + lane;
    }
    const int total = s_part[NW];
    if (tid == 0) ws.meta[(size_t)b * bt.T] = make_int4(0, s_cnt[(D + 2) * NW], total, 0);
    const int Rv = planes_reached(gs, reach);
    for (int i = tid; i < D; i += NT) {             // plane i is reached from bins [i - Rv, i + Rv + 1]
        const int lo = max(0, i - Rv), hi = min(D + 1, i + Rv + 1);
        ws.range[(size_t)b * bt.T * D + i] = make_int2(s_cnt[lo * NW], s_cnt[(hi + 1) * NW]);
    }
}

// ---------------------------------------------------------------------------
// Large examples: P workgroups per example, no exchange between them.  Workgroup p looks at all
// atoms of the example but sorts and writes only its share of the keys: index types, the types
// [tA, tB) (the atoms of smaller types are counted on the way: where its records start; the
// coordinates of other types' atoms are not even read); vector types, a run of x-plane bins (all
// atoms are placed once, to count the other bins).
// The share's atoms are listed in LDS on the way.  Only those are placed after that, twice (which costs
// less than keeping their positions in registers): for the counts, and in order of bins for the
// records.  A share of more than kOwnAtoms atoms (one type of a large receptor) goes through all atoms again for
// the counts and leaves atom, key and place within the bin where its records will be (index types; vector types
// go through all atoms once more for the places), and its list in bin order sits in the workspace (rchan, whose
// final contents are written last): one example of 20000 atoms in two channels 71 us, 94 with a second pass over
// all atoms for the places, and 89 with two such passes and no list before them.
// Bound: trips to memory one after the other, and placing atoms in double precision.  Two examples of
// 20000 atoms and 18 channels as eight subgrids each: 27 us, 42 when all passes went through all
// atoms; one of 20000, 28 channels 17 / 31; 12000 in two channels 34 / 57; vector types, two of 20000 28 / 56.
// ---------------------------------------------------------------------------
constexpr int kRangeThreads = 1024;
constexpr int kRangeMaxKeys = 1700;     // keys of a workgroup: two words of LDS each
constexpr int kOwnAtoms = 12288;        // atoms of a share that are listed in LDS, twelve per thread
constexpr int kRankBin = 2048;          // longer bins are put in atom order by one wavefront, not by counting

template <bool VECTOR>
__global__ __launch_bounds__(kRangeThreads) void prep_range_kernel(GridSpec gs, Batch bt, Workspace ws,
                                                                  unsigned tag, int stop, int per, int keys_cap)
{
    constexpr int NT = kRangeThreads, U = 8;
    extern __shared__ int s_mem[];
    int *s_pos = s_mem;                         // [keys + 1] where a bin starts (from the first record of the share)
    int *s_cnt = s_mem + keys_cap + 1;          // [keys] count, then fill cursor
    int *s_rmax = s_cnt + keys_cap;             // [types of the share]
    __shared__ int s_part[NT / 64 + 1], s_less, s_found;
    __shared__ int s_own[kOwnAtoms];            // the share's atoms, later in order of bins
    unsigned short *s_mine = reinterpret_cast<unsigned short *>(s_own);        // ... of a round
    static_assert(kOwnAtoms * sizeof(int) >= NT * U * sizeof(unsigned short), "a round's atoms");
    const int p = blockIdx.y, b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bs = source_example(bt.sub.count, b);       // whose atoms and pose this (virtual) example reads
    const int N = bt.N, T = bt.T, D = gs.D, nb = D + 3;   // bin D+2 holds the culled atoms
    if (MG_STOP_IS(stop, 1)) return;
    int n = N;
    if (bt.natoms) {
        n = bt.natoms[bs];
        n = n < 0 ? 0 : (n > N ? N : n);
    }
    const int32_t *ty = VECTOR ? nullptr : bt.types + (size_t)bs * N;
    const int tA = VECTOR ? 0 : min(T, p * per), tB = VECTOR ? 1 : min(T, tA + per);
    const int Tg = tB - tA, K = Tg * nb;
    // keys of this share: all of its types' bins; vector types: bins [kA, kB) of the one group
    const int kA = VECTOR ? min(nb, p * per) : 0, kB = VECTOR ? min(nb, kA + per) : K;

    Xform X;
    load_xform(X, bs, bt.centers, bt.quats, bt.translations);
    keep_scalar(X);
    float vec_reach = 0.0f;         // reach of the widest channel, for vector types
    if (VECTOR) {
        vec_reach = widest_reach(gs, bt);
        if (p == 0 && wave == NT / 64 - 1) rank_channels(bt, ws, b);
    }
    float org[3];                   // the grid's first point
    float gc[3];
    grid_center(bt.sub, X, b, bs, gc);
    for (int m = 0; m < 3; ++m) org[m] = gc[m] - gs.half;
    if (p == 0) {
        if (tid == 0) store_rotation(X, ws.rot + b * 12);
        if (tid == 0) *reinterpret_cast<float4 *>(ws.gcen + b * 4) = make_float4(gc[0], gc[1], gc[2], 0.0f);
        if (b == 0 && tid == 0) *ws.tag = tag;
    }
    for (int k = tid; k < K; k += NT) s_cnt[k] = 0;
    for (int k = tid; k < Tg; k += NT) s_rmax[k] = 0;
    if (tid == 0) s_less = s_found = 0;
    __syncthreads();

    const float *crd = bt.coords + (size_t)bs * N * 3;
    const float *rad = bt.radii + ((!VECTOR && !gs.radius_type_indexed) ? (size_t)bs * N : 0);
    struct Raw {
        float c[3], r;
    };
    auto fetch = [&](int a, int t) {
        Raw w;
        w.c[0] = crd[(size_t)a * 3]; w.c[1] = crd[(size_t)a * 3 + 1]; w.c[2] = crd[(size_t)a * 3 + 2];
        w.r = VECTOR ? 1.0f : rad[gs.radius_type_indexed ? t : a];
        return w;
    };
    // key of an atom of type t (relative to the share's first type); pp, r: its record (r = 0: culled)
    auto place = [&](const Raw &w, int t, float (&pp)[3], float &r) {
        apply_xform(X, w.c, pp);
        r = VECTOR ? 1.0f : gs.radius_scale * w.r;
        const float reach = VECTOR ? vec_reach : (gs.binary ? r : r * gs.c);
        const bool live = meets_grid(gs, org, pp, r, reach);
        int bin = D + 2;
        if (live) {
            const float f = floorf((pp[0] - org[0]) * gs.inv_res);
            bin = f < 0.0f ? 0 : (f >= (float)D ? D + 1 : (int)f + 1);
        } else {
            r = 0.0f;
        }
        return (t - tA) * nb + bin;
    };
    // body(atom, type, Raw, number) for every atom of the share.  Index types: the share's atoms of a round (8192)
    // are gathered in LDS first, so that all lanes place atoms, and numbered; vector types: for all atoms.
    auto for_mine = [&](auto body) {
        int done = 0;
        for (int base = 0; base < N; base += NT * U) {
            int v[U], found = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int a = base + u * NT + tid;
                v[u] = a < n ? (VECTOR ? 0 : ty[a]) : -1;
            }
            if (!VECTOR) {
                if (tid == 0) s_found = 0;
                __syncthreads();
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int a = base + u * NT + tid;
                const bool own = v[u] >= tA && v[u] < tB;
                if (VECTOR) continue;
                const unsigned long long m = __ballot(own);
                int at = 0;
                if (lane == 0 && m) at = atomicAdd(&s_found, (int)__builtin_popcountll(m));
                at = bcast(at, 0) + (int)__builtin_popcountll(m & ((1ull << lane) - 1ull));
                if (own) s_mine[at] = (unsigned short)(a - base);
            }
            if (!VECTOR) {
                __syncthreads();
                found = s_found;
            }
            Raw w[U];
            int t[U], own_a[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                own_a[u] = -1;
                if (VECTOR) {
                    if (v[u] == 0) own_a[u] = base + u * NT + tid;
                } else if (u * NT + tid < found) {
                    own_a[u] = base + s_mine[u * NT + tid];
                }
                t[u] = own_a[u] < 0 || VECTOR ? 0 : ty[own_a[u]];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (own_a[u] >= 0) w[u] = fetch(own_a[u], t[u]);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (own_a[u] >= 0) body(own_a[u], t[u], w[u], done + u * NT + tid);
            done += found;
            if (!VECTOR) __syncthreads();       // s_mine is free again
        }
    };

    // ---- 0. the share's atoms; what it has to know of the others ----
    // Index types: how many atoms of smaller types there are.  Vector types: every atom is placed, those of
    // other bins are counted, and the share with the last bin writes the records of the culled atoms, from
    // the end of the example's records backwards.
    int less = 0;
    const bool last = VECTOR && kA < kB && kB == nb;
    for (int base = 0; base < N; base += NT * U) {
        int v[U];
        Raw w[VECTOR ? U : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int a = base + u * NT + tid;
            v[u] = a < n ? (VECTOR ? 0 : ty[a]) : -1;
            if (VECTOR && v[u] == 0) w[VECTOR ? u : 0] = fetch(a, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int a = base + u * NT + tid;
            bool own;
            if (VECTOR) {
                float pp[3], r = 0.0f;
                const int key = v[u] == 0 ? place(w[VECTOR ? u : 0], 0, pp, r) : -1;
                own = key >= kA && key < kB && key != D + 2;
                const unsigned long long culled = __ballot(key == D + 2);
                int base_c = 0;
                if (lane == 0 && culled) base_c = atomicAdd(&s_cnt[D + 2], (int)__builtin_popcountll(culled));
                base_c = bcast(base_c, 0);      // (here, where lane 0 is active: it need not be culled itself)
                if (key == D + 2) {
                    if (last) {
                        const int at = n - 1 - base_c - (int)__builtin_popcountll(culled & ((1ull << lane) - 1ull));
                        ws.rec[(size_t)b * N + at] = make_float4(pp[0], pp[1], pp[2], 0.0f);
                        ws.idx[(size_t)b * N + at] = a;
                        ws.alive[(size_t)b * N + a] = 0;
                    }
                } else if (key >= 0 && !own) {
                    atomicAdd(&s_cnt[key], 1);
                }
                if (p == 0 && a < N && v[u] < 0) ws.alive[(size_t)b * N + a] = 0;       // past natoms
            } else {
                own = v[u] >= tA && v[u] < tB;
                less += v[u] >= 0 && v[u] < tA ? 1 : 0;
                if (p == 0 && a < N && (v[u] < 0 || v[u] >= T)) ws.alive[(size_t)b * N + a] = 0;        // no group owns this atom
            }
            const unsigned long long m = __ballot(own);
            int at = 0;
            if (lane == 0 && m) at = atomicAdd(&s_found, (int)__builtin_popcountll(m));
            at = bcast(at, 0) + (int)__builtin_popcountll(m & ((1ull << lane) - 1ull));
            if (own && at < kOwnAtoms) s_own[at] = a;
        }
    }
    if (!VECTOR) {
        const int incl = wave_inclusive_scan(less);
        if (lane == 63 && incl > 0) atomicAdd(&s_less, incl);
    }
    __syncthreads();
    const int found = s_found;
    const bool kept = found <= kOwnAtoms;
    int4 *listed = VECTOR ? nullptr : reinterpret_cast<int4 *>(ws.rec + (size_t)b * N + s_less);       // (a share that is not kept)

    // ---- 1. atoms per key ----
    constexpr int kPer = kOwnAtoms / NT;
    int my_a[kPer], my_slot[kPer];      // slot: key << 14 | place within the bin
    static_assert(kOwnAtoms <= 1 << 14 && kRangeMaxKeys < 1 << 17, "packed into a word");
    // body(u, atom, type, Raw) for the kept atoms of this thread, four requested at a time
    const auto for_kept = [&](auto body) {
#pragma unroll
        for (int u0 = 0; u0 < kPer; u0 += 4) {
            if (u0 * NT >= found) break;
            int t[4];
            Raw w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = VECTOR || my_a[u0 + u] < 0 ? 0 : ty[my_a[u0 + u]];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (my_a[u0 + u] >= 0) w[u] = fetch(my_a[u0 + u], t[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (my_a[u0 + u] >= 0) body(u0 + u, my_a[u0 + u], t[u], w[u]);
        }
    };
    if (kept) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) my_a[u] = u * NT + tid < found ? s_own[u * NT + tid] : -1;
        for_kept([&](int u, int a, int t, const Raw &w) {
            float pp[3], r;
            const int key = place(w, t, pp, r);
            my_slot[u] = key << 14 | atomicAdd(&s_cnt[key], 1);
            if (!VECTOR && r > 0.0f) atomicMax(&s_rmax[t - tA], __float_as_int(r));         // r > 0: ordered like ints
            ws.alive[(size_t)b * N + a] = r > 0.0f ? 1 : 0;
        });
    } else {
        for (int k = tid; k < K; k += NT) s_cnt[k] = 0;
        __syncthreads();
        for_mine([&](int a, int t, const Raw &w, int at) {
            float pp[3], r;
            const int key = place(w, t, pp, r);
            if (VECTOR) atomicAdd(&s_cnt[key], 1);
            else listed[at] = make_int4(a, key, atomicAdd(&s_cnt[key], 1), 0);
            if (!VECTOR && r > 0.0f) atomicMax(&s_rmax[t - tA], __float_as_int(r));
            if (key >= kA && key < kB) ws.alive[(size_t)b * N + a] = r > 0.0f ? 1 : 0;
        });
    }
    __syncthreads();
    if (MG_STOP_IS(stop, 3)) return;

    // ---- 2. exclusive scan of the counts ----
    const int chunk = (K + NT - 1) / NT;
    const int k0 = min(K, tid * chunk), k1 = min(K, k0 + chunk);
    int mine = 0;
    for (int k = k0; k < k1; ++k) mine += s_cnt[k];
    int wtotal;
    int run = wave_exclusive_scan(mine, &wtotal);
    if (lane == 0) s_part[wave] = wtotal;
    __syncthreads();
    if (wave == 0) {
        int t16;
        const int v = lane < NT / 64 ? s_part[lane] : 0;
        const int ex = wave_exclusive_scan(v, &t16);
        if (lane < NT / 64) s_part[lane] = ex;
        if (lane == 0) s_part[NT / 64] = t16;
    }
    __syncthreads();
    run += s_part[wave];
    for (int k = k0; k < k1; ++k) {
        s_pos[k] = run;
        run += s_cnt[k];
        s_cnt[k] = 0;
    }
    if (tid == 0) s_pos[K] = s_part[NT / 64];
    __syncthreads();
    if (MG_STOP_IS(stop, 4)) return;

    // ---- 3. atoms into their bins in any order; group descriptors and spans meanwhile ----
    const int first = VECTOR ? 0 : s_less;
    float4 *rec = ws.rec + (size_t)b * N + first;
    int *idx = ws.idx + (size_t)b * N + first, *order = ws.rchan + (size_t)b * N + first;
    const int own0 = s_pos[kA];         // (vector types: the share's bins begin there)
    if (kept) {
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (my_a[u] >= 0) s_own[s_pos[my_slot[u] >> 14] - own0 + (my_slot[u] & 16383)] = my_a[u];
    } else if (!VECTOR) {
        for (int base = tid; base < found; base += 4 * NT) {
            int4 e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = base + u * NT < found ? listed[base + u * NT] : make_int4(-1, 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (e[u].x >= 0) order[s_pos[e[u].y] + e[u].z] = e[u].x;
        }
    } else {
        for_mine([&](int a, int t, const Raw &w, int) {
            float pp[3], r;
            const int key = place(w, t, pp, r);
            if (key >= kA && key < kB) order[s_pos[key] + atomicAdd(&s_cnt[key], 1)] = a;
        });
    }
    if (!VECTOR || p == 0) {
        for (int tg = tid; tg < Tg; tg += NT) {
            const int f = s_pos[tg * nb], dead = s_pos[tg * nb + D + 2], end = s_pos[(tg + 1) * nb];
            ws.meta[(size_t)b * T + tA + tg] = make_int4(first + f, dead - f, end - f, 0);
        }
        for (int e = tid; e < Tg * D; e += NT) {
            const int tg = e / D, i = e - tg * D;
            // plane i is reached from bins [i - Rv, i + Rv + 1]
            const float rmax = VECTOR ? vec_reach : __int_as_float(s_rmax[tg]) * (gs.binary ? 1.0f : gs.c);
            const int Rv = planes_reached(gs, rmax);
            const int lo = max(0, i - Rv), hi = min(D + 1, i + Rv + 1);
            ws.range[((size_t)b * T + tA + tg) * D + i] =
                make_int2(first + s_pos[tg * nb + lo], first + s_pos[tg * nb + hi + 1]);
        }
    }
    __syncthreads();
    if (MG_STOP_IS(stop, 5)) return;

    // ---- 4. records: the atoms of a bin in atom order (the order the forward kernel sums in) ----
    if (kept) {
        // in order of bins: the lanes of a wavefront compare with the same few atoms (33 -> 24 us for 9000
        // atoms of four types), and neighbours write next to each other
#pragma unroll
        for (int u = 0; u < kPer; ++u) my_a[u] = u * NT + tid < found ? s_own[u * NT + tid] : -1;
        for_kept([&](int u, int a, int t, const Raw &w) {
            float pp[3], r;
            const int key = place(w, t, pp, r), lo = s_pos[key], cnt = s_pos[key + 1] - lo;
            int at = own0 + u * NT + tid;               // culled atoms: where they are
            if (r > 0.0f) {
                if (cnt > kRankBin) return;             // below
                at = lo;
                int i = 0;
                for (; i + 4 <= cnt; i += 4) {
                    int o[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) o[k] = s_own[lo - own0 + i + k];
#pragma unroll
                    for (int k = 0; k < 4; ++k) at += o[k] < a ? 1 : 0;
                }
                for (; i < cnt; ++i) at += s_own[lo - own0 + i] < a ? 1 : 0;
            }
            rec[at] = make_float4(pp[0], pp[1], pp[2], r);
            idx[at] = a;
        });
    }
    const int e0 = s_pos[kA], e1 = s_pos[kB];
    for (int e = e0 + tid; !kept && e < e1; e += NT) {
        const int a = order[e], t = VECTOR ? 0 : ty[a];
        float pp[3], r;
        const int key = place(fetch(a, t), t, pp, r);
        const int lo = s_pos[key], cnt = s_pos[key + 1] - lo;
        int at = e;                             // culled atoms: where they are
        if (r > 0.0f) {
            if (cnt > kRankBin) continue;       // below
            int rank = 0, i = 0;
            for (; i + 4 <= cnt; i += 4) {
                int o[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) o[u] = order[lo + i + u];
#pragma unroll
                for (int u = 0; u < 4; ++u) rank += o[u] < a ? 1 : 0;
            }
            for (; i < cnt; ++i) rank += order[lo + i] < a ? 1 : 0;
            at = lo + rank;
        }
        rec[at] = make_float4(pp[0], pp[1], pp[2], r);
        idx[at] = a;
    }
    // bins with very many atoms: one wavefront goes through the example in atom order
    for (int k = kA + wave; k < kB; k += NT / 64) {
        const int tg = k / nb, lo = s_pos[k];
        if (s_pos[k + 1] - lo <= kRankBin || k - tg * nb == D + 2) continue;
        int at = lo;
        for (int base = 0; base < n; base += 64) {
            const int a = base + lane;
            float pp[3] = {0.0f, 0.0f, 0.0f}, r = 0.0f;
            const bool hit = a < n && (VECTOR || ty[a] == tA + tg) &&
                             place(fetch(a, tA + tg), tA + tg, pp, r) == k;
            const unsigned long long m = __ballot(hit);
            if (hit) {
                const int e = at + (int)__builtin_popcountll(m & ((1ull << lane) - 1ull));
                rec[e] = make_float4(pp[0], pp[1], pp[2], r);
                idx[e] = a;
            }
            at += (int)__builtin_popcountll(m);
        }
    }
    if (VECTOR) return;
    __syncthreads();                            // the list has been read by all
    for (int tg = wave; tg < Tg; tg += NT / 64) {
        const int e2 = s_pos[(tg + 1) * nb];
        for (int e = s_pos[tg * nb] + lane; e < e2; e += 64) order[e] = tA + tg;
    }
}

size_t align16(size_t v) { return (v + 15) / 16 * 16; }

}  // namespace

size_t workspace_bytes(const GridSpec &gs, int subgrid_count, int B, int N, int T)
{
    const size_t bn = (size_t)B * (size_t)N, bt = (size_t)B * (size_t)T;
    size_t bytes = bn * sizeof(float4);                     // rec
    bytes += align16(bn * sizeof(int));                     // idx
    bytes += bt * sizeof(int4);                             // meta
    bytes += align16(bt * (size_t)gs.D * sizeof(int2));     // range
    bytes += (size_t)B * 12 * sizeof(float);                // rot
    bytes += (size_t)B * 4 * sizeof(float);                 // gcen
    bytes += align16(bt * sizeof(int));                     // chan_order
    bytes += align16(bn);                                   // alive
    bytes += align16(bn * sizeof(int));                     // rchan
    bytes += 16;                                            // tag
    if (subgrid_count > 1) {
        bytes += align16(bn * 3 * sizeof(float));           // gtmp
        if (gs.radius_type_indexed) bytes += align16(bn * (size_t)T * sizeof(float));   // wtmp
    }
    return bytes;
}

Workspace carve_workspace(const GridSpec &gs, int subgrid_count, void *base, int B, int N, int T)
{
    const size_t bn = (size_t)B * (size_t)N, bt = (size_t)B * (size_t)T;
    char *p = (char *)base;
    Workspace ws;
    ws.rec = (float4 *)p;
    p += bn * sizeof(float4);
    ws.idx = (int *)p;
    p += align16(bn * sizeof(int));
    ws.meta = (int4 *)p;
    p += bt * sizeof(int4);
    ws.range = (int2 *)p;
    p += align16(bt * (size_t)gs.D * sizeof(int2));
    ws.rot = (float *)p;
    p += (size_t)B * 12 * sizeof(float);
    ws.gcen = (float *)p;
    p += (size_t)B * 4 * sizeof(float);
    ws.chan_order = (int *)p;
    p += align16(bt * sizeof(int));
    ws.alive = (unsigned char *)p;
    p += align16(bn);
    ws.rchan = (int *)p;
    p += align16(bn * sizeof(int));
    ws.tag = (unsigned *)p;
    p += 16;
    ws.gtmp = nullptr;
    ws.wtmp = nullptr;
    if (subgrid_count > 1) {
        ws.gtmp = (float *)p;
        p += align16(bn * 3 * sizeof(float));
        if (gs.radius_type_indexed) ws.wtmp = (float *)p;
    }
    return ws;
}

hipError_t launch_transform(int B, int N, const float *coords, const float *centers,
                            const float *quats, const float *translations, float *out,
                            bool inverse, hipStream_t stream)
{
    dim3 grid((N + 255) / 256, B);
    if (inverse)
        hipLaunchKernelGGL(transform_kernel<true>, grid, dim3(256), 0, stream, B, N, coords,
                           centers, quats, translations, out);
    else
        hipLaunchKernelGGL(transform_kernel<false>, grid, dim3(256), 0, stream, B, N, coords,
                           centers, quats, translations, out);
    return hipGetLastError();
}

// What the tables were made for, folded into one word (never 0): the kernels of a *_prepared
// call compare it with their own arguments and do nothing if the workspace holds something else.
unsigned workspace_tag(const GridSpec &gs, const Batch &bt)
{
    unsigned long long h = 0x9E3779B97F4A7C15ull;
    const unsigned words[] = {(unsigned)bt.B, (unsigned)bt.N, (unsigned)bt.T, (unsigned)gs.D,
                              (unsigned)bt.sub.per_side, bt.vec ? 1u : 0u, (unsigned)gs.binary,
                              (unsigned)gs.radius_type_indexed};
    for (unsigned w : words) {
        h ^= w;
        h *= 0x100000001B3ull;
        h ^= h >> 29;
    }
    const unsigned t = (unsigned)(h ^ (h >> 32));
    return t ? t : 1u;
}

hipError_t launch_prep(const GridSpec &gs, const Batch &bt, const Workspace &ws, int stop,
                       hipStream_t stream)
{
    const unsigned tag = workspace_tag(gs, bt);
    const bool vec = bt.vec;
    ExLayout L;
    L.Tg = bt.T;
    L.N = bt.N;
    const long long K = (long long)L.Tg * (gs.D + 3);
    // Index types of more than 4096 atoms: shares of the types for several workgroups while there are few
    // examples, else one workgroup per example.  Kernel, us, shares / one workgroup: 16 x 8192 atoms, 28 channels 13.5 / 19.1,
    // 1 x 8192 11.3 / 18.1, 32 x 8192 17.0 / 19.6, 48 x 8000 26 / 20, 64 x 8000 in eight channels 24 / 18, 12 x 8192 in two 34 / 49;
    // 16 x 4100 11.5 / 12.7, 32 x 4100 13.5 / 13.1; below 4096 atoms alike for few examples (20 x 3000 11 / 11), worse for many
    // (50 x 2040 18 / 10).
    // With few channels one share may hold nearly all atoms.  It sorts them in order of bins, which pays where atoms inside the
    // grid and culled ones are mixed or bins are long; not where nearly all are culled (up to five channels, grids of up to 14 A),
    // nor in up to three where all find room in the grid (0.08 per cubic Angstrom), up to 60 to a plane.  All atoms in one channel,
    // points a side at 0.5 A, call, us, shares / one workgroup: 8192 atoms 16 27.4 / 18.7, 24 27.8 / 24.0, 32 28.7 / 29.0, 48 32.7 / 41.1,
    // 96 47.2 / 48.7; eight of 5000 16 20.6 / 15.4, 48 26.2 / 33.2, 72 33.8 / 40.3, 96 32.0 / 28.7; 4100 24 19.0 / 14.5, 48 24.1 / 24.6,
    // 72 26.0 / 21.5, 48 at 1 A 31.8 / 34.1; in two of five channels 8192 16 19.4 / 14.8, eight of 5000 72 20.4 / 24.8.
    const float side = (float)gs.D * gs.res, room = side + 4.0f;        // 2 A on each side for the atoms' reach
    const bool culled = bt.T <= 5 && side <= 14.0f;
    const bool roomy = bt.T <= 3 && bt.N <= std::min(5500, 60 * gs.D) && 0.08f * room * room * room >= (float)bt.N;
    const bool shared = bt.N > 4096 && bt.B <= 32 && !culled && !roomy;
    const bool fits = !vec && !shared && bt.N <= kExMaxAtoms && (size_t)K * 2 * sizeof(int) <= kExMaxLds;
    L.K = fits ? (int)K : 0;
    const size_t lds_bytes = (size_t)L.ints() * sizeof(int);
    if (vec && bt.N <= kExMaxAtoms) {
        const dim3 grd(bt.B), blk(kExThreads);
        const size_t lds = ((size_t)(gs.D + 3) * (kExThreads / 64) + 1) / 2 * sizeof(int);
        if (bt.N <= 2 * kExThreads)
            hipLaunchKernelGGL(prep_example_vector_kernel<2>, grd, blk, lds, stream, gs, bt, ws, tag, stop);
        else if (bt.N <= 4 * kExThreads)
            hipLaunchKernelGGL(prep_example_vector_kernel<4>, grd, blk, lds, stream, gs, bt, ws, tag, stop);
        else
            hipLaunchKernelGGL(prep_example_vector_kernel<8>, grd, blk, lds, stream, gs, bt, ws, tag, stop);
        return hipGetLastError();
    }
    if (fits && lds_bytes <= kExMaxLds) {
        const dim3 grd(bt.B);
        // 512 threads while they still hold all the atoms four apiece: half as many wavefronts
        // behind every barrier (1 us less per call at 2040 atoms; 256 threads with eight atoms
        // apiece measured 4 us more)
        if (bt.N <= 4 * 512)
            hipLaunchKernelGGL((prep_example_kernel<4, 512>), grd, dim3(512), lds_bytes, stream, gs, bt, ws, tag, stop);
        else if (bt.N <= 4 * kExThreads)
            hipLaunchKernelGGL((prep_example_kernel<4, kExThreads>), grd, dim3(kExThreads), lds_bytes, stream, gs, bt, ws, tag, stop);
        else
            hipLaunchKernelGGL((prep_example_kernel<8, kExThreads>), grd, dim3(kExThreads), lds_bytes, stream, gs, bt, ws, tag, stop);
        return hipGetLastError();
    }
    // Shares per example, at most kRangeMaxKeys keys each: as many workgroups as the chip holds at a time (one per
    // CU).  A few more would run alone after the others: kernel, us, 256 / B shares at most / rounded up: index types, 28 examples of
    // 4100 atoms and 28 channels 14.1 / 15.9, 20 of 5000 and 25 channels 13.8 / 15.2; vector types, 20 of 20000 32.3 / 53.6,
    // 100 of 9000 28.1 / 42.7 (but index types, 40 of 9000 and 28 channels 21.8 / 20.8).  Where that leaves index types
    // fewer than five shares (more than 51 examples) one is longer than the list, as types are uneven, and a
    // second wave costs less: 60 of 20000 atoms, five channels 85.5 / 47.9, 86 of 9000, 28 channels 37.2 / 32.9.
    // The grid runs over the examples first: the XCDs take workgroups in turn, and with the shares first the longest
    // share of every example lay on the same ones (32 examples of 16000 atoms, all in one of two channels, 96 points a side, 129 us,
    // 156 with the shares first; 24 of 20000 147 / 173; 70 of 20000 and 18 channels 52 / 104).
    const int nb = gs.D + 3, units = vec ? nb : bt.T;
    int want = 256 / bt.B;
    if (!vec && want < 5) want = (256 + bt.B - 1) / bt.B;
    want = std::max(1, std::min(units, want));
    int per = (units + want - 1) / want;
    if (!vec) per = std::min(per, std::max(1, kRangeMaxKeys / nb));
    const int shares = (units + per - 1) / per;
    const int keys = vec ? nb : per * nb;
    const size_t lds = (size_t)(2 * keys + 1 + (vec ? 1 : per)) * sizeof(int);
    const dim3 grd(bt.B, shares), blk(kRangeThreads);       // (at most 65535 types)
    if (vec) hipLaunchKernelGGL(prep_range_kernel<true>, grd, blk, lds, stream, gs, bt, ws, tag, stop, per, keys);
    else hipLaunchKernelGGL(prep_range_kernel<false>, grd, blk, lds, stream, gs, bt, ws, tag, stop, per, keys);
    return hipGetLastError();
}

}  // namespace mg
