// Step kernels that march along z: a block keeps a column of the lattice and works through its planes one by
// one, so that what a node passes on to its neighbours goes through LDS and registers instead of memory.
//
// Each thread owns one (x, y) column.  Of the nineteen post-collision populations of its node of plane z,
// the sixteen that change column go to the neighbours through LDS, one value per population and node; the three that
// stay in the column are handed on in registers.  A plane's level and upward populations wait in registers until
// the plane they are needed on, one and two planes later, so LDS holds one plane's worth only:
// at iteration k the block has the post-collision state of plane k and completes the pull of plane k - 1.
//
//   KIND_PAIR  FP32 populations, projected operator, points that stay where they are: TWO steps in one launch.  The
//              first collides every node of plane k with populations pulled from memory, the second every
//              node of plane k - 1 with populations pulled from the first, so two steps read and write the
//              state once: 76 instead of 152 B per node and step.
//   KIND_MOM   moment storage, one step: the populations are rebuilt once per node from its ten pieces
//              and pulled from LDS, where the gather from memory needs 91 values of 18 neighbours per node.
//
// Planes of at most 1024 nodes are taken whole (the column's neighbours wrap round inside the block); larger
// ones are cut into 64 x 8 or 64 x 12 output nodes with a rim of one node, whose first step is repeated by
// every block that shares it (29 or 20 % more of it; which one is left to the cost model).  A block makes zc planes and repeats one below and above.  The inner
// nodes of a cut row are one wave's, the two outer columns the last wave's: loads start on a cache line, and
// the waves of the rim skip the second half (256^3: 297 -> 268 us a step, moment storage 307 -> 258, against threads
// in the order of the 66 x 10 nodes; cuts of 32 x 8 or 32 x 16, two blocks per compute unit, 387 and 430).
//
// What bounds it: the two barriers a plane and the arithmetic between them, with one or two blocks of 8 to 16 waves per
// compute unit (42 KB of LDS for the populations, 72 to 117 registers); the memory side is at three quarters of
// the copy rate (256^3: 262 us a step, 76 B a node, 4.9 TB/s; 440 us and 5.8 TB/s one step at a time; moment
// storage 236 us, 80 B, 5.7 TB/s).
//
// Points stay outside: a block has all points of its column, one plane after another, so that work per point
// in it is serial (2000 points within 32^3 nodes of 128^3 with moment storage: 899 us a step with records staged and
// velocities summed here, 85 so, 78 in the kernel of one node per thread).  launch_force_field lays the force
// density out in the list tiles that have points, once for fixed points and before every step otherwise; the kernel
// reads it there with the plane before (elsewhere the counter-force stands) and leaves the velocity there, which
// launch_partials sums per point.  Every iteration issues the same loads for it, needed or not: on a path with
// fewer loads in flight a wait for one is a wait for all that came after it too (256^3 with 1000 colloids and
// moment storage: 350 us a step with loads where needed, 290 so).  Runs without points have kernels of their own.
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "lbm_collide.h"
#include "lbm_device.h"
#include "lbm_internal.h"

namespace lbm {

namespace {

enum Kind { KIND_PAIR = 0, KIND_MOM = 1 };

constexpr int MX = 64, EX = MX + 2;        // output nodes of a block along x where planes are cut, ... with the rim
constexpr int NE_MAX = 1024;               // nodes of the largest plane taken whole
constexpr int LY = 2, LX = 6;              // point-list tiles of cut planes: 64 x 4 x 1 nodes (base-2 logarithms)
constexpr unsigned NOWHERE = 1u << 31;     // offset past every descriptor's range: loads give 0, stores are dropped

// populations that change column, and their place in LDS
constexpr bool moves(int i) { return cvel(i, 0) != 0 || cvel(i, 1) != 0; }
constexpr int place(int i)
{
    int n = 0;
    for (int j = 0; j < i; ++j) n += moves(j) ? 1 : 0;
    return n;
}
constexpr int NP = place(NQ);
static_assert(NP == 16, "populations through LDS");

struct MarchArgs {
    int zc, nbx, nby, nchunk;      // planes per block; blocks along x, y, z
    const float* src;
    float* dst;
    const BoxDev* boxes;
    const int* toff;
    const unsigned* groups;        // per list tile: which of its 32 groups of eight nodes along x points reach
    const float* field;            // force density, [box][z][y][component][x], in those groups
    float *vel0, *vel1;            // velocity of the (first, second) step there, or NULL
};

// NE nodes of a block and plane; MY: output rows of a cut plane (0: planes taken whole)
template <int KIND, int COLL, int NE, int MY, bool LISTS>
__global__ __launch_bounds__((NE + 63) / 64 * 64) void k_march(const Geom G, const MarchArgs A)
{
    constexpr bool CUT = MY > 0;
    constexpr int EY = MY + 2;
    constexpr int NV = KIND == KIND_PAIR ? NQ : MP_N;   // values a thread loads per plane
    __shared__ float pops[NP][NE];

    // block -> (columns, chunk of planes, box); neighbours on one XCD
    int b = xcd_tile(int(blockIdx.x), int(gridDim.x));
    const int bx = b % A.nbx;
    b /= A.nbx;
    const int by = b % A.nby;
    b /= A.nby;
    const int ch = b % A.nchunk, box = b / A.nchunk;
    const int x0 = CUT ? bx * MX : 0, y0 = CUT ? by * MY : 0, z0 = ch * A.zc, nzc = min(A.zc, G.nz - z0);
    const int tid = threadIdx.x, lane = tid & 63;

    // The thread's column, whether it makes output, and where its values (e) and those of its neighbours lie in LDS.
    // Of a cut plane each wave takes the inner nodes of one row, so that its loads start on a line, and the last
    // wave the two outer columns; only the waves of output rows take part in the second half of an iteration.
    const int ne = CUT ? NE : G.nx * G.ny;
    int x, y, e = min(tid, ne - 1), at = 0;
    bool out;
    if constexpr (CUT) {
        const int rim = min(max(tid - MX * EY, 0), 2 * EY - 1);
        const int ex = tid < MX * EY ? 1 + tid % MX : (rim & 1) * (EX - 1), ey = tid < MX * EY ? tid / MX : rim >> 1;
        e = ex + EX * ey;
        x = (x0 - 1 + ex + G.nx) % G.nx;
        y = (y0 - 1 + ey + G.ny) % G.ny;
        out = tid < MX * EY && ey >= 1 && ey <= MY && x0 + ex - 1 < G.nx && y0 + ey - 1 < G.ny;
        at = min(max(e, EX + 1), NE - EX - 2);     // threads of the rim: some place inside
    } else {
        x = e % G.nx;
        y = e / G.nx;
        out = tid < ne;
    }
    const bool active = !CUT || __any(out);
    const int xm = x == 0 ? G.nx - 1 : x - 1, xp = x + 1 == G.nx ? 0 : x + 1;
    const int ym = y == 0 ? G.ny - 1 : y - 1, yp = y + 1 == G.ny ? 0 : y + 1;
    auto from = [&](int i) {                       // column x - c_i
        if constexpr (CUT) return at - cvel(i, 0) - cvel(i, 1) * EX;
        const int cx = cvel(i, 0), cy = cvel(i, 1);
        return (cx > 0 ? xm : cx < 0 ? xp : x) + G.nx * (cy > 0 ? ym : cy < 0 ? yp : y);
    };

    const BoxDev& B = A.boxes[box];
    const Rates<float> R = rates_of<COLL, float>(G, B);
    const float gc[3] = {float(B.gc[0]), float(B.gc[1]), float(B.gc[2])};

    // memory: a descriptor per z plane, lane offset of a node, plane offset of a value
    const unsigned rbb = unsigned(G.rb) * 4u, kp = unsigned(G.kp) * 4u, pbytes = unsigned(G.ny) * rbb;
    const unsigned own = unsigned(y) * rbb + unsigned(x) * 4u, dest = out ? own : NOWHERE;
    const char* sb = reinterpret_cast<const char*>(A.src + (long long)box * G.sbox);
    char* db = reinterpret_cast<char*>(A.dst + (long long)box * G.sbox);
    auto plane = [&](int z) { return z < 0 ? z + G.nz : (z >= G.nz ? z - G.nz : z); };
    auto load = [&](int k, float (&p)[NV]) {       // what iteration k starts from
        const unsigned size = k <= nzc ? pbytes : 0u;   // past the last iteration: nothing
        if constexpr (KIND == KIND_PAIR) {
            const rsrc_t r[3] = {plane_rsrc(sb + (unsigned long long)plane(z0 + k + 1) * pbytes, size),
                                 plane_rsrc(sb + (unsigned long long)plane(z0 + k) * pbytes, size),
                                 plane_rsrc(sb + (unsigned long long)plane(z0 + k - 1) * pbytes, size)};
            const unsigned ro[3] = {unsigned(yp) * rbb, unsigned(y) * rbb, unsigned(ym) * rbb};
            const unsigned xo[3] = {unsigned(xp) * 4u, unsigned(x) * 4u, unsigned(xm) * 4u};
#pragma unroll
            for (int i = 0; i < NQ; ++i)
                p[i] = bload<float, 0>(r[cvel(i, 2) + 1], ro[cvel(i, 1) + 1] + xo[cvel(i, 0) + 1], unsigned(i) * kp);
        } else {
            const rsrc_t r = plane_rsrc(sb + (unsigned long long)plane(z0 + k) * pbytes, size);
#pragma unroll
            for (int q = 0; q < MP_N; ++q) p[q] = bload<float, 0>(r, own, unsigned(q) * kp);
        }
    };

    // The list tiles the block needs, one per lane (the same in every wave): those of its output nodes (all of a whole
    // plane) and, where the first of two steps collides the rim too, those around them.
    auto tile_of = [&](int px, int py) { return CUT ? (py >> LY) * G.ntx + (px >> LX) : py >> G.lty; };
    constexpr int TW = KIND == KIND_PAIR ? 3 : 1, TN = CUT ? TW * ((MY >> LY) + TW - 1) : 0;
    static_assert(MY % (1 << LY) == 0 && TN <= 16, "list tiles of a block");
    int mytile = -1;
    if constexpr (!CUT) {
        if (lane < G.nty) mytile = lane;           // a tile spans the rows
    } else {
        if (lane < TN) {
            const int tx = ((x0 >> LX) + lane % TW - TW / 2 + G.ntx) % G.ntx;
            const int ty = ((y0 >> LY) + lane / TW - TW / 2 + G.nty) % G.nty;
            mytile = ty * G.ntx + tx;
        }
        for (int l = 0; l < TN - 1; ++l)           // a tile met twice round a narrow box counts once
            if (lane > l && lane < TN && mytile == __builtin_amdgcn_readlane(mytile, l)) mytile = -1;
    }
    // the lane that has the thread's own tile (one without any where the block does not need it)
    const int nodetile = tile_of(x, y);
    int slot = 63;
    for (int l = 0; l < 16; ++l)
        if (__builtin_amdgcn_readlane(mytile, l) == nodetile) slot = l;

    const int group = CUT ? ((y & ((1 << LY) - 1)) << LX | (x & ((1 << LX) - 1))) >> 3
                          : ((y & (G.ty - 1)) << G.ltx | x) >> 3;

    struct List {
        int a, c;        // this lane's tile: entries a .. c - 1
        unsigned g;      // ... and the groups of nodes they reach, if there are any
    };
    const rsrc_t rtoff = plane_rsrc(A.toff, A.toff ? unsigned(G.ntiles + 1) * 4u : 0u);
    const rsrc_t rgroups = plane_rsrc(A.groups, A.toff ? unsigned(G.ntiles) * 4u : 0u);
    const unsigned tiles_at = mytile >= 0 ? unsigned(mytile) * 4u : NOWHERE;
    auto entries = [&](int k) {                    // of plane z0 + k (none past the last plane)
        typedef int i32x2 __attribute__((ext_vector_type(2)));
        const unsigned first = unsigned((box * G.ntz + plane(z0 + k)) * G.nty * G.ntx) * 4u;
        const unsigned at = tiles_at | (k <= nzc ? 0u : NOWHERE);
        const i32x2 v = __builtin_bit_cast(i32x2, __builtin_amdgcn_raw_buffer_load_b64(rtoff, at, first, 0));
        return List{v.x, v.y, bload<unsigned, 0>(rgroups, at, first)};
    };
    // the lanes whose nodes points reach
    auto reached = [&](const List& l) {
        return __ballot((unsigned(__shfl(int(l.c > l.a ? l.g : 0u), slot)) >> group & 1u) != 0);
    };
    // the force field and the velocities at the thread's node of plane z0 + k, if points reach it
    const unsigned frow = unsigned(G.nx) * 4u, fsize = unsigned(G.ny) * 3u * frow;
    const unsigned fown = unsigned(y) * 3u * frow + unsigned(x) * 4u;
    auto field_plane = [&](const float* f, int k) {
        return plane_rsrc(reinterpret_cast<const char*>(f) + (unsigned long long)(box * G.nz + plane(z0 + k)) * fsize, fsize);
    };
    auto mine = [&](unsigned long long lanes) { return unsigned(lanes >> lane) & 1u; };
    // (offsets past the range by a bit, not by a choice: the compiler makes a branch of a choice, and with it
    // vector registers of what both sides compute)
    auto force = [&](int k, unsigned long long lanes, float (&g)[3]) {
        const rsrc_t r = field_plane(A.field, k);
        const unsigned at = fown | ((mine(lanes) ^ 1u) << 31);
#pragma unroll
        for (int q = 0; q < 3; ++q) g[q] = bload<float, 0>(r, at, unsigned(q) * frow);
    };
    auto keep = [&](float* vel, int k, unsigned long long lanes, const float (&u)[3]) {
        if (!vel || lanes == 0) return;
        const rsrc_t r = field_plane(vel, k);
        const unsigned at = fown | ((mine(lanes) ^ 1u) << 31) | (out ? 0u : NOWHERE);
#pragma unroll
        for (int q = 0; q < 3; ++q) bstore<float, 0>(u[q], r, at, unsigned(q) * frow);
    };

    // nxt: what the next iteration starts from; lev: level populations of the plane before; up1, up2: upward ones of
    // the plane before and the one before it
    float nxt[NV], lev[NQ], up1[NQ], up2[NQ], gp[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < NQ; ++i) lev[i] = up1[i] = up2[i] = 0.0f;
    bool bad = false;
    // lanes whose nodes points reach in plane k - 1 (m1) and k (m0); la: the lists of plane k + 1
    List la{0, 0, 0};
    unsigned long long m0 = 0, m1 = 0;
    float gn[3];                               // the next plane's force density
    if constexpr (LISTS) {
        m0 = reached(entries(-1));
        la = entries(0);
        force(-1, m0, gn);
    }
    load(-1, nxt);
    for (int k = -1; k <= nzc; ++k) {
        float cur[NQ], u[3];
        if constexpr (KIND == KIND_PAIR) {
#pragma unroll
            for (int i = 0; i < NQ; ++i) cur[i] = nxt[i];
        } else {
            float p[MP_N];
#pragma unroll
            for (int q = 0; q < MP_N; ++q) p[q] = nxt[q];
            cur[0] = p[MP_R0];
#pragma unroll
            for (int i = 1; i < NQ; i += 2) rebuild_pair(p, i, cur[i], cur[i + 1]);
        }
        float g[3] = {gc[0], gc[1], gc[2]};
        unsigned long long ma = 0;
        if constexpr (LISTS) {
            // plane k + 1's forces and plane k + 2's lists, the same loads in every iteration
#pragma unroll
            for (int q = 0; q < 3; ++q) g[q] = mine(m0) ? gn[q] : gc[q];
            ma = reached(la);
            la = entries(k + 2);
            force(k + 1, ma, gn);
        }
        load(k + 1, nxt);
        if constexpr (KIND == KIND_PAIR) {
            // the first step's collision of plane k
            const Node<float> m = moments_of(cur);
            float p[MP_N];
            pieces_of<0>(m, g, R, p, u);
            if (out && k >= 0 && k < nzc) bad = bad || !finite_node(m, g);
            populations_of(p, cur);
            if (LISTS && k >= 0 && k < nzc) keep(A.vel0, k, m0, u);
        }

        // pull of plane k - 1 and its collision
        if (tid < ne) {
#pragma unroll
            for (int i = 1; i < NQ; ++i)
                if (moves(i)) pops[place(i)][e] = cvel(i, 2) > 0 ? up2[i] : (cvel(i, 2) == 0 ? lev[i] : cur[i]);
        }
        __syncthreads();
        if (active && k >= 1) {
            float f[NQ];
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                if (moves(i))
                    f[i] = pops[place(i)][from(i)];
                else
                    f[i] = cvel(i, 2) > 0 ? up2[i] : (cvel(i, 2) == 0 ? lev[i] : cur[i]);
            }
            const rsrc_t r = plane_rsrc(db + (unsigned long long)(z0 + k - 1) * pbytes, pbytes);
            float p[MP_N];
            if constexpr (KIND == KIND_PAIR) {
                const Node<float> m = moments_of(f);
                pieces_of<0>(m, gp, R, p, u);
                bad = bad || (out && !finite_node(m, gp));
                bstore<float, 2>(float(wgt(0)) * p[MP_R0], r, dest, 0u);
#pragma unroll
                for (int i = 1; i < NQ; i += 2) {
                    float bp, bm;
                    rebuild_pair(p, i, bp, bm);
                    bstore<float, 2>(float(wgt(i)) * bp, r, dest, unsigned(i) * kp);
                    bstore<float, 2>(float(wgt(i)) * bm, r, dest, unsigned(i + 1) * kp);
                }
            } else {
                // f are brackets f*_i / w_i: the weights 12, 2, 1 (times 1/36) go on the sums
                float q[NQ];
#pragma unroll
                for (int i = 0; i < NQ; ++i) q[i] = float(wgt(i)) * f[i];
                const Node<float> m = moments_of(q);
                pieces_of<COLL>(m, gp, R, p, u);
                bad = bad || (out && !finite_node(m, gp));
#pragma unroll
                for (int v = 0; v < MP_N; ++v) bstore<float, 2>(p[v], r, dest, unsigned(v) * kp);
            }
            if constexpr (LISTS) keep(KIND == KIND_PAIR ? A.vel1 : A.vel0, k - 1, m1, u);
        }
        __syncthreads();

#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            up2[i] = up1[i];
            up1[i] = cur[i];
            lev[i] = cur[i];
        }
        gp[0] = g[0];
        gp[1] = g[1];
        gp[2] = g[2];
        m1 = m0;
        m0 = ma;
    }
    if (__any(bad) && lane == 0) atomicOr(&G.nf[box], 1);
    if (blockIdx.x == 0 && tid == 0) *G.rebin = 0;   // as the other step kernels
}

}  // namespace

// Force density (counter-force and points, the sums of the single-step kernel, in its order) near points, for the
// marching kernels.  Of a tile's 256 nodes only the groups of eight along x that a stencil reaches are written (and read): a
// tenth of them where points are spread out (256^3, FP32, 10^4 points and their velocities 317 -> 297 us a step, 512 boxes
// of 32^3 with 5900 298 -> 277).  A wave looks through FT tiles, one per lane; their entries are consecutive in the lists.
// Where they are few (WPT), the wave fetches all their records at once and takes the reached groups of each tile, eight at a
// time, a node per lane: two chains of loads for FT tiles (256^3 with 10^4 colloids and moment storage 383 -> 343 us a
// step against a block per FT tiles; FT = 8 352).  Where they are many, the block takes the tiles one by one, a node
// per thread, with the records staged RPT at a time.  (The waves of a block have tiles far apart, so that points in one
// place are many blocks'.)
constexpr int FT = 4, RW = int(sizeof(PRec<float>) / 16), RPT = BLOCK / RW, WPT = 128 / RW;

// the groups of tile (tx, ty) that a stencil starting at (bx, by) reaches
__device__ __forceinline__ unsigned stencil_groups(const Geom& G, int bx, int by, int tx, int ty)
{
    unsigned row = 0, near = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int sx = bx + i - (bx + i >= G.nx ? G.nx : 0);
        row |= unsigned(sx >> G.ltx == tx) << ((sx & (G.tx - 1)) >> 3);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int sy = by + j - (by + j >= G.ny ? G.ny : 0);
        near |= (sy >> G.lty == ty ? row : 0u) << ((sy & (G.ty - 1)) << (G.ltx - 3));
    }
    return near;
}

__global__ __launch_bounds__(BLOCK) void k_force_field(const Geom G, const BoxDev* __restrict__ boxes,
                                                       const int* __restrict__ toff, const int* __restrict__ tlist,
                                                       const PRec<float>* __restrict__ rec, unsigned* __restrict__ groups,
                                                       float* __restrict__ field)
{
    constexpr int NW = BLOCK / 64;
    __shared__ uint4 sraw[RPT * RW];
    __shared__ uint4 wraw[NW][128];
    __shared__ int many[NW];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    auto first_of = [&](int w) { return ((long long)w * gridDim.x + blockIdx.x) * FT; };
    struct Tile {
        int tx, ty, z, box;
    };
    auto tile_at = [&](unsigned t) {
        return Tile{int(t % G.ntx), int(t / G.ntx % G.nty), int(t / unsigned(G.ntx * G.nty) % G.ntz),
                    int(t / G.tiles_per_box)};
    };
    auto reaches = [&](int z, int bz) {
        const int dz = z - bz + (z < bz ? G.nz : 0);
        return dz <= 3;
    };
    auto store = [&](const Tile& T, int x, int y, const float (&g)[3]) {
        float* f = field + (((long long)T.box * G.nz + T.z) * G.ny + y) * 3 * G.nx + x;
        for (int q = 0; q < 3; ++q) f[q * G.nx] = g[q];
    };

    // the wave's tiles
    const long long first = first_of(wave);
    const bool has = lane < FT && first + lane < G.ntiles;
    const int a = has ? toff[first + lane] : 0, c = has ? toff[first + lane + 1] : 0;
    const unsigned long long tiles = __ballot(c > a);
    const int e0 = tiles ? __builtin_amdgcn_readlane(a, __ffsll(tiles) - 1) : 0;
    const int n = tiles ? __builtin_amdgcn_readlane(c, 63 - __builtin_clzll(tiles)) - e0 : 0;
    if (lane == 0) many[wave] = n > WPT;
    if (n > 0 && n <= WPT) {
        const PRec<float>* staged = reinterpret_cast<const PRec<float>*>(wraw[wave]);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int word = lane + 64 * i, sp = word / RW, sw = word - sp * RW;
            if (sp < n) wraw[wave][word] = reinterpret_cast<const uint4*>(rec + pk_point(tlist[e0 + sp]))[sw];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        int4 h{};
        if (lane < n) h = __builtin_bit_cast(int4, wraw[wave][lane * RW]);
        for (unsigned long long m = tiles; m; m &= m - 1) {
            const int l = __ffsll(m) - 1;
            const unsigned t = unsigned(first + l);
            const Tile T = tile_at(t);
            const bool hit = lane >= __builtin_amdgcn_readlane(a, l) - e0 && lane < __builtin_amdgcn_readlane(c, l) - e0 &&
                             reaches(T.z, h.z);
            const unsigned near = wave_or(hit ? stencil_groups(G, h.x, h.y, T.tx, T.ty) : 0u);
            const unsigned long long hits = __ballot(hit);
            if (lane == 0) groups[t] = near;
            const BoxDev& B = boxes[T.box];
            for (unsigned left = near; left;) {
                // lane -> node of the eight next groups
                int group = -1;
                for (int j = 0; j < 8 && left; ++j, left &= left - 1)
                    if (lane >> 3 == j) group = __ffs(left) - 1;
                const int node = max(group, 0) * 8 + (lane & 7);
                const int x = (T.tx << G.ltx) + (node & (G.tx - 1)), y = (T.ty << G.lty) + (node >> G.ltx);
                float g[3] = {float(B.gc[0]), float(B.gc[1]), float(B.gc[2])};
                for (unsigned long long q = hits; q; q &= q - 1) {
                    const int p = __ffsll(q) - 1;
                    add_point(G, __builtin_amdgcn_readlane(h.x, p), __builtin_amdgcn_readlane(h.y, p),
                              __builtin_amdgcn_readlane(h.z, p), staged[p], x, y, T.z, g[0], g[1], g[2]);
                }
                if (group >= 0 && x < G.nx && y < G.ny) store(T, x, y, g);
            }
        }
    }
    __syncthreads();

    // tiles with many entries
    const PRec<float>* staged = reinterpret_cast<const PRec<float>*>(sraw);
    const int sp = int(threadIdx.x) / RW, sw = int(threadIdx.x) - sp * RW;
    for (int w = 0; w < NW; ++w) {
        if (!many[w]) continue;
        const long long f0 = first_of(w);
        const bool in = lane < FT && f0 + lane < G.ntiles;
        const int ta = in ? toff[f0 + lane] : 0, tc = in ? toff[f0 + lane + 1] : 0;
        const unsigned long long some = __ballot(tc > ta);
        const int end = __builtin_amdgcn_readlane(tc, 63 - __builtin_clzll(some));   // past the last tile's entries
        int s0 = 0, s1 = 0;                                                          // entries staged
        for (unsigned long long m = some; m; m &= m - 1) {
            const int l = __ffsll(m) - 1;
            const unsigned t = unsigned(f0 + l);
            const Tile T = tile_at(t);
            const int x = (T.tx << G.ltx) + (threadIdx.x & (G.tx - 1)), y = (T.ty << G.lty) + (threadIdx.x >> G.ltx);
            const BoxDev& B = boxes[T.box];
            float g[3] = {float(B.gc[0]), float(B.gc[1]), float(B.gc[2])};
            unsigned near = 0;
            for (int k = __builtin_amdgcn_readlane(ta, l), k1 = __builtin_amdgcn_readlane(tc, l); k < k1;) {
                if (k >= s1) {
                    s0 = k;
                    s1 = min(k + RPT, end);
                    __syncthreads();   // every wave has read the records before
                    if (sp < s1 - s0)
                        sraw[threadIdx.x] = reinterpret_cast<const uint4*>(rec + pk_point(tlist[s0 + sp]))[sw];
                    __syncthreads();
                }
                // a lane looks at each staged point: those that reach the plane (and the row, where a wave has one)
                // are added
                const int np = min(k1, s1) - k;
                int4 h{};
                bool hit = false;
                if (lane < np) {
                    h = __builtin_bit_cast(int4, sraw[(k - s0 + lane) * RW]);
                    int dy = y - h.y;
                    if (dy < 0) dy += G.ny;
                    hit = reaches(T.z, h.z);
                    near |= hit ? stencil_groups(G, h.x, h.y, T.tx, T.ty) : 0u;
                    hit = hit && (dy <= 3 || G.tx < 64);
                }
                for (unsigned long long q = __ballot(hit); q; q &= q - 1) {
                    const int p = __ffsll(q) - 1;
                    add_point(G, __builtin_amdgcn_readlane(h.x, p), __builtin_amdgcn_readlane(h.y, p),
                              __builtin_amdgcn_readlane(h.z, p), staged[k - s0 + p], x, y, T.z, g[0], g[1], g[2]);
                }
                k += np;
            }
            near = wave_or(near);
            if (threadIdx.x == 0) groups[t] = near;
            if (x < G.nx && y < G.ny && (near >> (threadIdx.x >> 3) & 1u)) store(T, x, y, g);
        }
    }
}

void launch_force_field(const Geom& G, const BoxDev* boxes, const int* toff, const int* tlist, const void* rec, unsigned* groups,
                        float* field, hipStream_t s)
{
    hipLaunchKernelGGL(k_force_field, dim3((unsigned)((G.ntiles + FT * (BLOCK / 64) - 1) / (FT * (BLOCK / 64)))),
                       dim3(BLOCK), 0, s, G, boxes, toff, tlist,
                       (const PRec<float>*)rec, groups, field);
}

bool march_whole(int nx, int ny) { return nx <= 64 && ny <= 64 && nx * ny <= NE_MAX; }

void march_tile(int nx, int ny, int& tx, int& ty)
{
    tx = march_whole(nx, ny) && nx <= 32 ? (nx <= 16 ? 16 : 32) : 64;
    ty = BLOCK / tx;
}

void launch_march(int storage, const Geom& G, int my, int zc, const void* src, void* dst, const BoxDev* boxes, const int* toff,
                  const unsigned* groups, const float* field, float* vel0, float* vel1, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    MarchArgs A;
    A.zc = zc;
    A.nbx = my == 0 ? 1 : (G.nx + MX - 1) / MX;
    A.nby = my == 0 ? 1 : (G.ny + my - 1) / my;
    A.nchunk = (G.nz + zc - 1) / zc;
    A.src = (const float*)src;
    A.dst = (float*)dst;
    A.boxes = boxes;
    A.toff = toff;
    A.groups = groups;
    A.field = field;
    A.vel0 = vel0;
    A.vel1 = vel1;
    const dim3 grid((unsigned)((long long)A.nbx * A.nby * A.nchunk * G.nboxes));
    auto go = [&](auto kern, int nodes) {
        const dim3 block((nodes + 63) / 64 * 64);
        if (ev0 && ev1)
            hipExtLaunchKernelGGL(kern, grid, block, 0, s, ev0, ev1, 0, G, A);
        else
            hipLaunchKernelGGL(kern, grid, block, 0, s, G, A);
    };
    const int n = G.nx * G.ny;
    auto by_size = [&](auto kind, auto coll, auto lists) {
        constexpr int KIND = decltype(kind)::value, COLL = decltype(coll)::value;
        constexpr bool LISTS = decltype(lists)::value;
        if (my == 8) go(k_march<KIND, COLL, EX * 10, 8, LISTS>, EX * 10);
        else if (my == 12) go(k_march<KIND, COLL, EX * 14, 12, LISTS>, EX * 14);
        else if (n <= 256) go(k_march<KIND, COLL, 256, 0, LISTS>, n);
        else if (n <= 576) go(k_march<KIND, COLL, 576, 0, LISTS>, n);
        else go(k_march<KIND, COLL, NE_MAX, 0, LISTS>, n);
    };
    auto by_kind = [&](auto lists) {
        using std::integral_constant;
        if (storage == ST_FP32) by_size(integral_constant<int, KIND_PAIR>{}, integral_constant<int, 0>{}, lists);
        else if (G.coll) by_size(integral_constant<int, KIND_MOM>{}, integral_constant<int, 1>{}, lists);
        else by_size(integral_constant<int, KIND_MOM>{}, integral_constant<int, 0>{}, lists);
    };
    if (toff) by_kind(std::true_type{});
    else by_kind(std::false_type{});
}

}  // namespace lbm
