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
// ones are cut into MX x MY output nodes with a rim of one node, whose first step is repeated by
// every block that shares it (29 % more of it).  A block makes zc planes and repeats one below and above.  The inner
// nodes of a cut row are one wave's, the two outer columns the last wave's: loads start on a cache line, and
// the waves of the rim skip the second half (256^3: 297 -> 268 us a step, moment storage 307 -> 258, against threads
// in the order of the 66 x 10 nodes; cuts of 32 x 8 or 32 x 16, two blocks per compute unit, 387 and 430).
//
// What bounds it: the two barriers a plane and the arithmetic between them, with one block of 11 or 16 waves per compute
// unit (42 KB of LDS for the populations, 24 B a node for velocities, 128 to 140 registers); the memory side is at
// three quarters of the copy rate (256^3: 259 us a step, 76 B a node, 4.9 TB/s, without points; 440 us and
// 5.8 TB/s one step at a time; moment storage 236 us, 80 B, 5.7 TB/s).
//
// Points: the entries of a plane in the point lists are looked up, fetched and staged in LDS over the planes before
// it; more than RPT of them at once are fetched in rounds.  Every iteration issues the same loads for them,
// needed or not: on a path with fewer loads in flight a wait for one is a wait for all that came after it too (256^3
// with 1000 colloids and moment storage: 350 us a step with loads where needed, 290 so).  Where two steps are taken of
// cut planes, whose rim touches the lists of twelve tiles, the force density is laid out once as a field instead
// (launch_force_field) and read with the plane before it where the lists have points near the block (128^3 with 600
// points: 60.8 -> 42 us a step; 512 whole boxes of 32^3 lose with it, 255 -> 277, to its three registers), and only
// velocities that are wanted need the records.  Interpolation partials are taken after the plane's last barrier, beside the
// next plane.  Runs without points have kernels of their own (256^3: 274 -> 259, moment storage 259 -> 236).
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "lbm_collide.h"
#include "lbm_device.h"
#include "lbm_internal.h"

namespace lbm {

namespace {

enum Kind { KIND_PAIR = 0, KIND_MOM = 1 };

constexpr int MX = 64, MY = 8;             // output nodes of a block and plane where planes are cut
constexpr int EX = MX + 2, EY = MY + 2;    // ... with the rim
constexpr int NE_CUT = EX * EY;
constexpr int NE_MAX = 1024;               // nodes of the largest plane taken whole
constexpr int LY = 2, LX = 6;              // point-list tiles of cut planes: 64 x 4 x 1 nodes (base-2 logarithms)
constexpr unsigned NOWHERE = 1u << 31;     // offset past every descriptor's range: loads give 0, stores are dropped
constexpr int RW = int(sizeof(PRec<float>) / 16), RPT = 48;   // staged records of a plane

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
    const int *toff, *tlist;
    const PRec<float>* rec;
    const float* field;            // two steps of cut planes: force density of the fixed points, [box][z][y][component][x]
    float *part0, *part1;          // interpolation partials of the (first, second) step, or NULL
};

template <int KIND, int COLL, int NE, bool CUT, bool LISTS>
__global__ __launch_bounds__((NE + 63) / 64 * 64) void k_march(const Geom G, const MarchArgs A)
{
    constexpr int NV = KIND == KIND_PAIR ? NQ : MP_N;   // values a thread loads per plane
    constexpr int NU = KIND == KIND_PAIR ? 2 : 1;       // velocities per iteration
    constexpr bool FIELD = KIND == KIND_PAIR && CUT;    // forces from the laid-out field
    constexpr bool EARLY = KIND == KIND_PAIR && !CUT;   // a plane's records are needed at its first collision
    __shared__ float pops[NP][NE];
    __shared__ float su[2][NU][3][NE];
    __shared__ uint4 sraw[3][RPT * RW];
    __shared__ int sent[3][RPT], stile[3][RPT];

    // block -> (columns, chunk of planes, box); neighbours on one XCD
    int b = xcd_tile(int(blockIdx.x), int(gridDim.x));
    const int bx = b % A.nbx;
    b /= A.nbx;
    const int by = b % A.nby;
    b /= A.nby;
    const int ch = b % A.nchunk, box = b / A.nchunk;
    const int x0 = CUT ? bx * MX : 0, y0 = CUT ? by * MY : 0, z0 = ch * A.zc, nzc = min(A.zc, G.nz - z0);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;

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

    // The list tiles the block needs, one per lane (the same in every wave): those of its output nodes (own0, own1,
    // or all of a whole plane) and, where the first of two steps collides the rim too, those around them.
    auto tile_of = [&](int px, int py) { return CUT ? (py >> LY) * G.ntx + (px >> LX) : py >> G.lty; };
    const int own0 = tile_of(x0, y0);
    const int own1 = CUT && (y0 >> LY) + 1 < G.nty ? own0 + G.ntx : own0;
    int mytile = -1;
    if constexpr (!CUT) {
        if (lane < G.nty) mytile = lane;           // a tile spans the rows
    } else if constexpr (KIND == KIND_MOM) {
        if (lane == 0 || (lane == 1 && own1 != own0)) mytile = lane == 0 ? own0 : own1;
    } else {
        if (lane < 12) {
            const int tx = ((x0 >> LX) + lane % 3 - 1 + G.ntx) % G.ntx, ty = ((y0 >> LY) + lane / 3 - 1 + G.nty) % G.nty;
            mytile = ty * G.ntx + tx;
        }
        for (int l = 0; l < 11; ++l)               // a tile met twice round a narrow box counts once
            if (lane > l && lane < 12 && mytile == __builtin_amdgcn_readlane(mytile, l)) mytile = -1;
    }
    const int nodetile = tile_of(x, y);
    auto mine = [&](int t) { return !CUT || t == own0 || t == own1; };
    // whether points' records are needed: for spreading without a field, for velocities in any case
    const bool stages = !FIELD || A.part0;

    struct List {
        int a, c;        // this lane's tile: entries a .. c - 1
    };
    const rsrc_t rtoff = plane_rsrc(A.toff, A.toff ? unsigned(G.ntiles + 1) * 4u : 0u);
    const rsrc_t rlist = plane_rsrc(A.tlist, NOWHERE), rrec = plane_rsrc(A.rec, NOWHERE);   // (offsets from the lists)
    auto entries = [&](int k) {                    // of plane z0 + k (none past the last plane)
        typedef int i32x2 __attribute__((ext_vector_type(2)));
        const unsigned t = unsigned((box * G.ntz + plane(z0 + k)) * G.nty * G.ntx + mytile);
        const i32x2 v = __builtin_bit_cast(
            i32x2, __builtin_amdgcn_raw_buffer_load_b64(rtoff, mytile >= 0 && k <= nzc ? t * 4u : NOWHERE, 0, 0));
        return List{v.x, v.y};
    };
    // force density of plane z0 + k at the thread's node, where the lists have points near the block: from the field
    // that launch_force_field left
    auto force = [&](int k, bool any, float (&g)[3]) {
        const unsigned row = unsigned(G.nx) * 4u, size = unsigned(G.ny) * 3u * row;
        const rsrc_t r = plane_rsrc(reinterpret_cast<const char*>(A.field) +
                                        (unsigned long long)(box * G.nz + plane(z0 + k)) * size, size);
        const unsigned off = any ? unsigned(y) * 3u * row + unsigned(x) * 4u : NOWHERE;
#pragma unroll
        for (int q = 0; q < 3; ++q) g[q] = bload<float, 0>(r, off, unsigned(q) * row);
    };
    // the thread's word of the plane's staged records: entry index and tile (or -1), and how many there are
    const int sp = tid / RW, sw = tid - sp * RW;
    auto assign = [&](const List& l, int& idx, int& tile) {
        int total = 0;
        idx = -1;
        tile = -1;
        for (unsigned long long m = __ballot(l.c > l.a && mine(mytile)); m; m &= m - 1) {
            const int q = __ffsll(m) - 1, e0 = __builtin_amdgcn_readlane(l.a, q);
            const int n = __builtin_amdgcn_readlane(l.c, q) - e0;
            if (sp >= total && sp < total + n) {
                idx = e0 + sp - total;
                tile = __builtin_amdgcn_readlane(mytile, q);
            }
            total += n;
        }
        if (sp >= RPT) idx = -1;
        return total;
    };
    auto entry = [&](int idx) { return bload<int, 0>(rlist, idx >= 0 ? unsigned(idx) * 4u : NOWHERE); };
    auto record = [&](int idx, int ent) {
        const unsigned at = unsigned(pk_point(ent)) * unsigned(sizeof(PRec<float>)) + unsigned(sw) * 16u;
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rrec, idx >= 0 ? at : NOWHERE, 0, 0));
    };
    auto put = [&](int buf, int idx, int ent, int tile, const uint4& w) {
        if (idx >= 0) {
            sraw[buf][tid] = w;
            if (sw == 0) {
                sent[buf][sp] = ent;
                stile[buf][sp] = tile;
            }
        }
    };
    auto staged = [&](int buf, int p) -> const PRec<float>& { return reinterpret_cast<const PRec<float>*>(sraw[buf])[p]; };
    // f(record, entry, tile, number) for every entry of a plane whose records are not all staged
    auto in_rounds = [&](int buf, const List& l, auto f) {
        for (unsigned long long m = __ballot(l.c > l.a && mine(mytile)); m; m &= m - 1) {
            const int q = __ffsll(m) - 1, e0 = __builtin_amdgcn_readlane(l.a, q), e1 = __builtin_amdgcn_readlane(l.c, q);
            const int tile = __builtin_amdgcn_readlane(mytile, q);
            for (int kb = e0; kb < e1; kb += RPT) {
                const int n = min(RPT, e1 - kb);
                __syncthreads();
                if (sp < n) {
                    const int ent = entry(kb + sp);
                    put(buf, kb + sp, ent, tile, record(kb + sp, ent));
                }
                __syncthreads();
                for (int p = 0; p < n; ++p) f(staged(buf, p), sent[buf][p], tile, p);
            }
        }
    };
    // force density of the plane's points at this node
    auto spread = [&](int buf, const List& l, int total, int z, float (&g)[3]) {
        auto add = [&](const PRec<float>& r, int, int tile, int) {
            if (tile == nodetile) add_point(G, r, x, y, z, g[0], g[1], g[2]);
        };
        if (total > RPT)
            in_rounds(buf, l, add);
        else
            for (int p = 0; p < total; ++p) add(staged(buf, p), 0, stile[buf][p], p);
    };
    // partial sums of the plane's velocity for the points of the output tiles, one wave per point (all 64 stencil
    // nodes, those of other planes and tiles with weight zero: the sums of the single-step kernel, in its order)
    auto interpolate = [&](int buf, const List& l, int total, int z, const float (&v)[3][NE], float* part) {
        const int dx = lane & 3, dy = (lane >> 2) & 3, dz = lane >> 4;
        auto sum = [&](const PRec<float>& r, int ent, int tile, int p) {
            if (p % nw != wave) return;
            int px = r.bx + dx, py = r.by + dy, pz = r.bz + dz;
            if (px >= G.nx) px -= G.nx;
            if (py >= G.ny) py -= G.ny;
            if (pz >= G.nz) pz -= G.nz;
            const bool in = pz == z && tile_of(px, py) == tile;
            const int li = in ? (CUT ? px - x0 + 1 + EX * (py - y0 + 1) : px + G.nx * py) : 0;
            const float w = in ? r.wx[dx] * r.wy[dy] * r.wz[dz] : 0.0f;
            const float sx = wave_sum(v[0][li] * w), sy = wave_sum(v[1][li] * w), sz = wave_sum(v[2][li] * w);
            float* o = part + ((long long)pk_point(ent) * G.maxp + pk_slot(ent)) * 3;
            if (lane == 0) {
                o[0] = sx;
                o[1] = sy;
                o[2] = sz;
            }
        };
        if (total > RPT)
            in_rounds(buf, l, sum);
        else
            for (int p = wave; p < total; p += nw) sum(staged(buf, p), sent[buf][p], stile[buf][p], p);
    };
    auto keep = [&](float (&v)[3][NE], const float (&u)[3]) {
        if (tid < ne) {
            v[0][e] = u[0];
            v[1][e] = u[1];
            v[2][e] = u[2];
        }
    };

    // nxt: what the next iteration starts from; lev: level populations of the plane before; up1, up2: upward ones of
    // the plane before and the one before it
    float nxt[NV], lev[NQ], up1[NQ], up2[NQ], gp[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < NQ; ++i) lev[i] = up1[i] = up2[i] = 0.0f;
    bool bad = false;
    // lists: l0, l1 of planes k and k - 1 with t0, t1 entries (staged in buffers b0, b1), la of plane k + 1
    List l0 = LISTS ? entries(-1) : List{0, 0}, l1{0, 0}, la = LISTS ? entries(0) : List{0, 0};
    int t0 = 0, t1 = 0, b0 = 0, b1 = 2;
    auto look = [&](const List& l, int& idx, int& tile) {
        const int total = stages ? assign(l, idx, tile) : 0;
        if (!stages || total > RPT) idx = -1;
        return total;
    };
    int idx = -1, tile = -1, ent = 0;          // the thread's word: its entry's index, tile and value
    if constexpr (LISTS) {
        t0 = look(l0, idx, tile);
        ent = entry(idx);
        if constexpr (EARLY) put(b0, idx, ent, tile, record(idx, ent));
    }
    float gn[3];                               // plane k + 1's force density (from the field), if there is any
    bool any = __ballot(l0.c > l0.a) != 0;
    if constexpr (FIELD && LISTS) force(-1, any, gn);
    load(-1, nxt);
    __syncthreads();
    for (int k = -1; k <= nzc; ++k) {
        // Point lists: the records of plane k, whose entries are here (EARLY: those of plane k + 1 at the end), the
        // entries of plane k + 1, the tile offsets of plane k + 2.
        const int idx0 = idx, tile0 = tile, ent0 = ent;
        uint4 word{};
        const List lc = la;
        int ta = 0;
        if constexpr (LISTS) {
            if constexpr (!EARLY) word = record(idx0, ent0);
            ta = look(lc, idx, tile);
            if (!EARLY || ta > 0) ent = entry(idx);
            la = entries(k + 2);
        }

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
        if constexpr (FIELD) {
#pragma unroll
            for (int q = 0; q < 3; ++q) g[q] = LISTS && any ? gn[q] : gc[q];
            if constexpr (LISTS) {
                any = __ballot(lc.c > lc.a) != 0;
                force(k + 1, any, gn);
            }
        }
        load(k + 1, nxt);
        if constexpr (KIND == KIND_PAIR) {
            // the first step's collision of plane k
            if constexpr (!FIELD) spread(b0, l0, t0, plane(z0 + k), g);
            const Node<float> m = moments_of(cur);
            float p[MP_N];
            pieces_of<0>(m, g, R, p, u);
            if (out && k >= 0 && k < nzc) bad = bad || !finite_node(m, g);
            populations_of(p, cur);
            if (A.part0 && t0 > 0) keep(su[k & 1][0], u);
        }

        // pull of plane k - 1 and its collision
        if (tid < ne) {
#pragma unroll
            for (int i = 1; i < NQ; ++i)
                if (moves(i)) pops[place(i)][e] = cvel(i, 2) > 0 ? up2[i] : (cvel(i, 2) == 0 ? lev[i] : cur[i]);
        }
        __syncthreads();
        if constexpr (KIND == KIND_MOM) spread(b1, l1, t1, z0 + k - 1, g);
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
                pieces_of<COLL>(m, g, R, p, u);
                bad = bad || (out && !finite_node(m, g));
#pragma unroll
                for (int v = 0; v < MP_N; ++v) bstore<float, 2>(p[v], r, dest, unsigned(v) * kp);
            }
            if ((KIND == KIND_PAIR ? A.part1 : A.part0) && t1 > 0) keep(su[k & 1][NU - 1], u);
        }
        const int bn = 3 - b0 - b1;                // the third buffer
        if constexpr (EARLY) {
            if (ta > 0) put(bn, idx, ent, tile, record(idx, ent));
        } else {
            put(b0, idx0, ent0, tile0, word);
        }
        __syncthreads();
        if constexpr (KIND == KIND_PAIR) {
            if (A.part0 && t0 > 0 && k >= 0 && k < nzc) interpolate(b0, l0, t0, z0 + k, su[k & 1][0], A.part0);
            if (A.part1 && t1 > 0 && k >= 1) interpolate(b1, l1, t1, z0 + k - 1, su[k & 1][1], A.part1);
        } else {
            if (A.part0 && t1 > 0 && k >= 1) interpolate(b1, l1, t1, z0 + k - 1, su[k & 1][0], A.part0);
        }

#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            up2[i] = up1[i];
            up1[i] = cur[i];
            lev[i] = cur[i];
        }
        gp[0] = g[0];
        gp[1] = g[1];
        gp[2] = g[2];
        l1 = l0;
        l0 = lc;
        t1 = t0;
        t0 = ta;
        b1 = b0;
        b0 = bn;
    }
    if (__any(bad) && lane == 0) atomicOr(&G.nf[box], 1);
    if (blockIdx.x == 0 && tid == 0) *G.rebin = 0;   // as the other step kernels
}

}  // namespace

// Force density of fixed points and counter-force at every node, for the two-step kernel: the sums of the
// single-step kernel, in its order, once per change of the points.  One block per list tile.
__global__ __launch_bounds__(BLOCK) void k_force_field(const Geom G, const BoxDev* __restrict__ boxes,
                                                       const int* __restrict__ toff, const int* __restrict__ tlist,
                                                       const PRec<float>* __restrict__ rec, float* __restrict__ field)
{
    const long long t = blockIdx.x;
    const int tx = int(t % G.ntx), ty = int(t / G.ntx % G.nty), box = int(t / G.tiles_per_box);
    const int z = int(t / ((long long)G.ntx * G.nty) % G.ntz);
    const int x = (tx << LX) + (threadIdx.x & 63), y = (ty << LY) + (threadIdx.x >> 6);
    if (x >= G.nx || y >= G.ny) return;
    const BoxDev& B = boxes[box];
    float g[3] = {float(B.gc[0]), float(B.gc[1]), float(B.gc[2])};
    for (int k = toff[t]; k < toff[t + 1]; ++k) add_point(G, rec[pk_point(tlist[k])], x, y, z, g[0], g[1], g[2]);
    float* f = field + (((long long)box * G.nz + z) * G.ny + y) * 3 * G.nx + x;
    for (int q = 0; q < 3; ++q) f[q * G.nx] = g[q];
}

void launch_force_field(const Geom& G, const BoxDev* boxes, const int* toff, const int* tlist, const void* rec, float* field,
                        hipStream_t s)
{
    hipLaunchKernelGGL(k_force_field, dim3((unsigned)G.ntiles), dim3(BLOCK), 0, s, G, boxes, toff, tlist,
                       (const PRec<float>*)rec, field);
}

bool march_whole(int nx, int ny) { return nx <= 64 && ny <= 64 && nx * ny <= NE_MAX; }

void march_tile(int nx, int ny, int& tx, int& ty)
{
    tx = march_whole(nx, ny) && nx <= 32 ? (nx <= 16 ? 16 : 32) : 64;
    ty = BLOCK / tx;
}

void launch_march(int storage, const Geom& G, int zc, const void* src, void* dst, const BoxDev* boxes, const int* toff,
                  const int* tlist, const void* rec, const float* field, void* part0, void* part1, hipStream_t s,
                  hipEvent_t ev0, hipEvent_t ev1)
{
    const bool whole = march_whole(G.nx, G.ny);
    MarchArgs A;
    A.zc = zc;
    A.nbx = whole ? 1 : (G.nx + MX - 1) / MX;
    A.nby = whole ? 1 : (G.ny + MY - 1) / MY;
    A.nchunk = (G.nz + zc - 1) / zc;
    A.src = (const float*)src;
    A.dst = (float*)dst;
    A.boxes = boxes;
    A.toff = toff;
    A.tlist = tlist;
    A.rec = (const PRec<float>*)rec;
    A.field = field;
    A.part0 = (float*)part0;
    A.part1 = (float*)part1;
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
        if (!whole) go(k_march<KIND, COLL, NE_CUT, true, LISTS>, NE_CUT);
        else if (n <= 256) go(k_march<KIND, COLL, 256, false, LISTS>, std::max(n, RPT * RW));
        else if (n <= 576) go(k_march<KIND, COLL, 576, false, LISTS>, n);
        else go(k_march<KIND, COLL, NE_MAX, false, LISTS>, n);
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
