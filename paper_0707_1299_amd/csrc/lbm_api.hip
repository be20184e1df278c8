// liblbm host runtime: the C ABI declared in include/lbm.h.
//
// The context owns no device memory: it carves the caller's workspace into
// the two population copies (pull scheme, A/B), per-box parameters, the
// per-point records, the tile bins and the scratch of the reductions, and
// enqueues every kernel on the caller's stream.  Repeated steps are captured
// once per (parity, force-set generation, length) into HIP graphs of 2, 4,
// ..., 128 steps and replayed.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "../../include/lbm.h"
#include "lbm_device.h"
#include "lbm_internal.h"

using namespace lbm;

namespace {

constexpr size_t ALIGN = 256;

size_t align_up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

// Multiplier and shift for n / d with n < 2^31 (d >= 1): s = 31 + ceil(log2 d), m = ceil(2^s / d)
// (below 2^32 for every d >= 1); then n / d = (n * m) >> s exactly.
void set_div_magic(int d, unsigned& m, int& s)
{
    int l = 0;
    while ((1LL << l) < d) ++l;
    s = 31 + l;
    m = unsigned(((1ULL << s) + (unsigned long long)d - 1) / (unsigned long long)d);
}

size_t storage_bytes(int st) { return st == LB_STORAGE_FP64 ? 8 : (st == LB_STORAGE_FP16 ? 2 : 4); }

size_t rec_bytes(int st) { return st == LB_STORAGE_FP64 ? sizeof(PRec<double>) : sizeof(PRec<float>); }

// most tiles of extent t met by the binning window of a point (5 consecutive nodes, periodic)
int max_axis_tiles(int n, int t)
{
    constexpr int WIN = 5;
    int best = 0;
    for (int b = 0; b < n; ++b) {
        int seen[WIN], cnt = 0;
        for (int k = 0; k < WIN; ++k) {
            const int tile = ((b + k) % n) / t;
            bool dup = false;
            for (int j = 0; j < cnt; ++j) dup |= seen[j] == tile;
            if (!dup) seen[cnt++] = tile;
        }
        best = std::max(best, cnt);
    }
    return best;
}

struct Layout {
    size_t pop[2], boxes, rec, psum, count, cursor, toff, bsum, tlist, tlist_tmp, partial, fpart, pmax, tmax, smax, ticket,
        tctr,
        err, nf, rebin, rebox, win,
        diag, diagout, field, vel[2], groups;
    size_t total;
};

struct Plan {
    Geom G;            // the geometry in use: Gp, or Gm while the marching kernels may take the steps (see set_geometry)
    Geom Gp, Gm;
    Geom Gr;           // that of reads without points (see read_geometry)
    Layout L;
    int chunks;
    long long cap;
    int march;         // z planes per block of the marching step kernels (see choose_march); 0: none
    int march_rows;    // ... and rows of a plane (0: all)
    double march_us, other_us;   // estimated time of a step without points: marching, other kernels (moment storage)
    int variant;       // the step kernel's variant bits (the caller's, or choose_default's)
    int plain[3];      // the tile that checkpoints name: the caller's, or plain_tile's for a caller who named none
    long long plain_tiles;
};

// Tile of a caller who names a variant but no tile, and the one that checkpoints name for every caller who named no
// tile: it follows from the box and the storage alone, where choose_default's goes by noise, operator and max_points too, and
// the marching kernels' by the registered sets.
void plain_tile(const lb_params* p, int& tx, int& ty, int& tz)
{
    const double box_bytes = double(p->nx) * p->ny * p->nz * planes_of(p->storage) * storage_bytes(p->storage);
    if (p->storage == LB_STORAGE_MOM32 && p->nx >= 128) {
        tx = 128; ty = 1; tz = 2;   // long x rows: the gathered pieces are re-read from L1
    } else if (box_bytes >= 4.0e9) {
        tx = 128; ty = 2; tz = 1;   // a whole wave on one row (also with two FP16 nodes per lane)
    } else if (p->nx >= 64) {
        tx = 64; ty = 2; tz = 2;
    } else if (p->nx >= 32) {
        tx = 32; ty = 4; tz = 2;
    } else {
        tx = 16; ty = 4; tz = 4;
    }
}

// Tile and variant of a caller who names neither.  Measured per step on one MI355X (us; the plain tile with variant 0 first
// where nothing else is said).  "Dense": room for a point per 1024 nodes.
//  - Tiles.  A tile row of 128 nodes where nx fills it (65 .. 128): fewer blocks share a misaligned row
//    (101 x 75 x 62 FP32 35.4 -> 31.9).  Sparse FP32 rows of 192 and more: one row per block (256^3 with 10^4
//    points 496 -> 429; 64 x 2 x 2 with the same variant 448), unless its last tile is mostly empty
//    (300 nodes: 41.9 -> 44.8); many points per node want compact tiles (65536 chain markers at 256^3: 590 ->
//    565, one row per block 940).  33 .. 63 nodes: one 64-node tile instead of two of 32 (100 boxes of
//    48^3: 458 -> 283), but for small dense lattices whose points are read one by one and that fill most of it (58^3 FP32
//    general with a point per 128 nodes 20.5 / 22.3; larger: 20 boxes of 45^3 with 2603 points 92 -> 56).  17 .. 31
//    nodes: 32-node tiles (40 boxes of 25^3 with 10416 55 -> 38; 17^3 FP64 with noise and room for 5000 points 33 -> 14, filled
//    with them 12.8 / 14.6).  Two FP16 nodes per lane: a whole wave per row from 128 nodes on (256^3: 292 -> 240; 64 x 2 x 2 250), small
//    dense ones only where the rows fill it (180 x 22 x 12 with 675 points 35 / 48), and with noise or small and general not where half a
//    tile stays idle (140 x 100 x 100 with noise 45 / 57; 130 x 60 x 30 11.7 / 12.5).  Moment storage: rows of a
//    z plane together (256^3: 524 -> 460), up to 70 MB (both copies) 64 x 2 x 2 if that needs 5 % fewer blocks (64 x 50 x 100
//    10.1 -> 9.0; 108 x 9 x 45 5.0 -> 4.0; 81^3 23.3 / 20.7).  FP64 with noise: 32-node tiles (130 x 146 x 202 498 -> 412,
//    70 x 60 x 60 56 -> 35), but where the last one holds 1 to 6 nodes 64-node ones up to 63 nodes (36^3 30.5 -> 16.6) and
//    beyond if they are fewer (98 x 14 x 36 18 / 31, 100 x 33 x 48 27 / 29; 66^3 66 -> 40).
//  - Block order.  Tile rows on one XCD (bit 64) except for lattices near the L2s' 32 MB.  Both copies up to 70 MB, in FP16
//    without noise 50 MB, narrow rows off the lines 48 MB: the orders cross between 60 and 75 MB in FP32 and FP64
//    with every operator (contiguous runs / tile rows: FP32 70^3, 52 MB, 13.6 / 14.0; 75^3, 64 MB, 16.6 / 16.4; 79^3, 75
//    MB, 20.6 / 18.0; 60 x 60 x 128, 70 MB, 13.9 / 14.1; 64 x 80 x 100, 78 MB, 15.3 / 14.5; with noise 79^3 26.8 / 23.3; FP64
//    57^3, 56 MB, 12.6 / 13.4; 63^3, 76 MB, 15.5 / 15.4; 79^3, 150 MB, 36.2 / 32.1) and at 45 in FP16 (85^3, 47 MB, 18.1 / 17.9;
//    90^3, 55 MB, 24.9 / 22.4; with noise 90^3 27.6 / 27.6, 95^3, 65 MB, 30.1 / 30.6).
//    Where the tiles of a row are no power of two, bit 64 means launch order.  In the projected FP64 step that pays from 110 MB
//    on (130 x 60 x 30, 71 MB, 18.0 / 19.0; 180 x 60 x 30, 98 MB, 22.1 / 22.4; 130 x 60 x 60, 142 MB, 35.7 / 33.1), otherwise as
//    above (FP32 137 x 41 x 122, 104 MB, 38.6 / 31.5, general 177 x 17 x 208, 95 MB, 27.6 / 25.5, FP16 149 x 64 x 143 46 /
//    42).  Contiguous runs come back with 64-node tiles of rows off the 32-byte sectors and large planes (FP32
//    151^3, 523 MB, 153 / 136, 158^3 173 / 194; 132 x 162 x 198, 644 MB, 209 / 196; 300 x 100 x 100, 456 MB, 100.0 / 98.8; FP64
//    130^3, 668 MB, 161 / 149; 154^3 262 / 282; on the sectors FP32 152^3 153 / 141, FP64 152^3 218 / 193).
//    Points crowded in one place would like them too (FP64 general, 2926 in one of 512 boxes of 16 x 44 x 5, 787 / 964), as
//    many spread out do not (130^3 with 3138 165 / 146).
//  - Loads.  Cached (bit 2) where neighbouring rows are read again after more than the L2 has passed (planes
//    over 2.6 MB: 256^3 455 -> 448; 128^3 67.5 -> 66.6 the other way) or where rows do not
//    start on a cache line, so that two rows share one (300 x 60 x 40: 47.6 -> 41.1; boxes of 16^3: 75 -> 65; 90^3 FP32
//    27.1 -> 24.5), unless the L2s hold them all the same: in FP64 up to 100 MB (2 boxes of 60 x 50 x 52, 95 MB, 20.6 ->
//    19.7 the other way; 70^3, 104 MB, 24.7 -> 24.2; 77^3 31.6 -> 30.2), rows of up to 64 nodes 140 MB (45 x 43 x 207, 122 MB, 50.6 ->
//    52.3); and in
//    the smallest lattices (20^3 FP32 10.0 -> 9.8; off the lines in FP16 up to 32 MB or 63 nodes: 100 boxes of 16^3 13.4 -> 11.0,
//    70^3 general 14.8 -> 13.1; 80^3, 39 MB, 17.0 -> 18.4).
//  - The kernel for one tile per block (bit 128) where its missing tile loop saves registers: FP16, moment
//    storage, the general and thermal operators, many points, small lattices; the FP32 and FP64 projected
//    step is memory bound and faster with the loop (256^3 FP32: 429 against 447), FP64 with noise on other tiles than 32-node
//    ones too when they are more than the 256 compute units (300 boxes of 14^3 114 / 156; one of 15^3 9.9 -> 8.6;
//    tiles an eighth full up to 320, 73 boxes of 5^3 30 -> 17, 83 42 / 43).
//    FP16 with one node per lane, sparse and with narrow rows likewise, and with cached loads (18 boxes of 31^3: 25.2 -> 23.4, 40 of 25^3 32.1 -> 27.5).
// Batches of FP16 boxes keep the plain tile: their checkpoints hold a maximum per tile.
void choose_default(const lb_params* p, int& tx, int& ty, int& tz, int& variant)
{
    const double esz = double(storage_bytes(p->storage)), planes = planes_of(p->storage);
    const double N = double(p->nx) * p->ny * p->nz, nodes = N * p->nboxes;
    const double box_bytes = N * planes * esz, copies = 2.0 * box_bytes * p->nboxes;
    const bool fp64 = p->storage == LB_STORAGE_FP64, fp16 = p->storage == LB_STORAGE_FP16, mom = p->storage == LB_STORAGE_MOM32;
    const bool noise = p->kT > 0.0, general = noise || p->collision != LB_COLLISION_PROJECTED;
    const bool pairs = fp16 && p->nx % 2 == 0;
    const bool dense = double(p->max_points) * 1024.0 > nodes;
    const auto tiles = [&](int a, int b, int c) {
        return double((p->nx + a - 1) / a) * ((p->ny + b - 1) / b) * ((p->nz + c - 1) / c);
    };
    plain_tile(p, tx, ty, tz);
    if (fp16 && p->nboxes > 1) {
    } else if (p->nx > 16 && p->nx < 32) {
        tx = 32; ty = 4; tz = 2;
    } else if (fp64 && noise && p->nx > 32) {
        const int last = p->nx % 32;
        if (last > 0 && last < 7 && (p->nx < 64 || tiles(64, 2, 2) < tiles(32, 4, 2))) { tx = 64; ty = 2; tz = 2; }
        else { tx = 32; ty = 4; tz = 2; }
    } else if (mom) {
        if (p->nx >= 64 && !(copies <= 70.0e6 && tiles(64, 2, 2) < 0.95 * tiles(64, 4, 1))) { tx = 64; ty = 4; tz = 1; }
        else if (p->nx > 32) { tx = 64; ty = 2; tz = 2; }
    } else if (pairs) {
        if (p->nx >= 128) {
            const bool idle = (p->nx + 63) / 64 % 2 != 0;     // half a tile of each row
            if (!(dense && p->nx % 128 != 0 && copies <= 25.0e6) && !(idle && (noise || (general && copies <= 32.0e6)))) { tx = 128; ty = 2; tz = 1; }
        } else if (p->nx > 32 && p->nx < 64 && !(dense && general && p->nx >= 48)) {
            tx = 64; ty = 2; tz = 2;
        }
    } else if (p->nx > 64 && p->nx <= 128 && !dense && !noise) {
        tx = 128; ty = 2; tz = 1;
    } else if (p->storage == LB_STORAGE_FP32 && p->nx >= 192 && !dense && !general &&
               3 * ((p->nx + 255) / 256 * 256) <= 4 * p->nx) {
        tx = 256; ty = 1; tz = 1;
    } else if (p->nx > 32 && p->nx < 64 && !(dense && general && p->nx > 48 && copies <= 70.0e6)) {
        tx = 64; ty = 2; tz = 2;
    }
    const int ntx = (p->nx + tx - 1) / tx;
    const bool rows = (ntx & (ntx - 1)) == 0;
    const bool aligned = (long long)(p->nx * esz) % 128 == 0, narrow = !aligned && p->nx < 32 && !mom;
    // two rows share a line that is read again
    const bool shared = !aligned && (esz < 8.0 || narrow || copies > (p->nx > 64 ? 100.0e6 : 140.0e6));
    if (copies <= (narrow ? 48.0e6 : fp64 && !general && !rows ? 110.0e6 : fp16 && !noise ? 50.0e6 : 70.0e6)) {
        variant = fp16 && !pairs && !general && p->nx < 64 && !dense ? 2 : 128;
        if (copies <= 9.0e6 || (fp16 && !aligned && (copies <= 32.0e6 || p->nx < 64))) variant |= 2;
    } else {
        const double plane = double(p->nx) * p->ny * planes * esz;
        const bool runs = !rows && tx == 64 && (long long)(p->nx * esz) % 32 != 0 && !fp16 && !mom && copies > (fp64 ? 1040.0e6 : 590.0e6) &&
                          plane > (fp64 ? 2.9e6 : 1.85e6);
        variant = runs ? 0 : 64;
        if (shared || (plane > 2.6e6 && !dense)) variant |= 2;
        if (fp16 || mom || general || dense) variant |= 128;
    }
    if (fp64 && noise && !(tx == 32 && rows && copies > 70.0e6)) {
        const double blocks = tiles(tx, ty, tz) * p->nboxes;
        variant = tx == 32 || blocks <= (nodes < 0.15 * BLOCK * blocks ? 320.0 : 256.0) ? 128 : 0;
        if (copies <= 9.0e6) variant |= 2;
    }
}

// Geometry of the lattice with tiles of tx x ty x tz (checked against the storage, the box size and cap points).
int fill_geometry(const lb_params* p, int variant, long long cap, int tx, int ty, int tz, Geom& G, std::string& why)
{
    memset(&G, 0, sizeof(G));
    G.nx = p->nx; G.ny = p->ny; G.nz = p->nz; G.nboxes = p->nboxes;
    G.tx = tx; G.ty = ty; G.tz = tz;
    G.ltx = __builtin_ctz(tx); G.lty = __builtin_ctz(ty); G.ltz = __builtin_ctz(tz);
    G.ntx = (p->nx + tx - 1) / tx;
    G.nty = (p->ny + ty - 1) / ty;
    G.ntz = (p->nz + tz - 1) / tz;
    set_div_magic(G.ntx, G.mtx, G.stx);
    set_div_magic(G.nty, G.mty, G.sty);
    set_div_magic(G.ntz, G.mtz, G.stz);
    G.N = (long long)p->nx * p->ny * p->nz;
    G.kp = p->nx;
    G.rb = (long long)planes_of(p->storage) * p->nx;
    G.sbox = ((long long)p->ny * p->nz * G.rb + 255) / 256 * 256 + 64;
    {
        // lanes along x of one tile row: a wave on one row addresses each row block from
        // its own descriptor; narrower rows of lanes address the box from one descriptor
        // with 32-bit offsets
        const bool pairs = p->storage == LB_STORAGE_FP16 && p->nx % 2 == 0 && !((variant >> 5) & 1);
        const int lanes_x = pairs ? tx / 2 : tx;
        if (lanes_x < 64 && (unsigned long long)G.sbox * storage_bytes(p->storage) >= (1ULL << 32)) {
            why = "tiles with fewer than 64 lanes along x (64 nodes, or 128 with two FP16 nodes per lane) need a "
                  "box of under 4 GiB";
            return LB_ERR_ARG;
        }
        // two FP16 nodes per lane on whole-wave rows address each z plane of rows from one descriptor
        if (pairs && lanes_x >= 64 && (unsigned long long)p->ny * G.rb * storage_bytes(p->storage) >= (1ULL << 32)) {
            why = "two FP16 nodes per lane need a z plane (ny * nx nodes) of under 4 GiB";
            return LB_ERR_SIZE;
        }
    }
    G.tiles_per_box = (long long)G.ntx * G.nty * G.ntz;
    G.ntiles = G.tiles_per_box * p->nboxes;
    G.rho0 = p->rho0 > 0.0 ? p->rho0 : 1.0;
    G.maxp = max_axis_tiles(p->nx, tx) * max_axis_tiles(p->ny, ty) * max_axis_tiles(p->nz, tz);
    // one block of BLOCK threads per tile: a launch of 2^32 threads and more would leave tiles out
    if (G.ntiles >= (1LL << 32) / BLOCK) { why = "too many tiles"; return LB_ERR_SIZE; }
    if (cap * G.maxp >= (1LL << 31) - 1 || cap >= (1LL << (31 - PK_SHIFT))) {
        why = "max_points too large";
        return LB_ERR_SIZE;
    }
    if (G.maxp > (1 << PK_BITS)) { why = "tile too small for the stencil"; return LB_ERR_ARG; }
    G.bchunks = int(std::min<long long>(256, (G.tiles_per_box + 255) / 256));
    G.tpb = 1 << ((variant >> 2) & 3);
    G.order = (variant >> 4) & 1;
    G.lgrp = 0;
    if ((variant >> 6) & 1) {
        // the runs of one tile row on one XCD: needs a power-of-two count of whole runs per row
        // (otherwise launch order)
        G.order = 1;
        if (G.ntx % G.tpb == 0 && ((G.ntx / G.tpb) & (G.ntx / G.tpb - 1)) == 0) {
            G.order = 2;
            G.lgrp = __builtin_ctz(unsigned(G.ntx / G.tpb));
        }
    }
    G.pairs = p->storage == LB_STORAGE_FP16 && p->nx % 2 == 0 && !((variant >> 5) & 1);
    G.coll = p->kT > 0.0 ? 2 : (p->collision != LB_COLLISION_PROJECTED ? 1 : 0);
    G.seed_lo = uint32_t(p->seed);
    G.seed_hi = uint32_t(p->seed >> 32);
    G.one = 1.0f;
    return LB_OK;
}

// Tiles of shape t that cover the lattice.
long long tiles_of(const Geom& G, const int (&t)[3])
{
    return (long long)((G.nx + t[0] - 1) / t[0]) * ((G.ny + t[1] - 1) / t[1]) * ((G.nz + t[2] - 1) / t[2]) * G.nboxes;
}

// Planes per block of the marching kernels (lbm_march.hip), or 0 where the kernels of one node per thread are
// faster.  A launch takes as many rounds as its blocks fill the chip; a round costs the block's planes and two
// repeated ones; the planes per block are chosen for the fewest.  Time of one plane of a block, measured: 7.2 us for
// whole planes of up to 1024 nodes, 5.4 up to 576, 5.3 up to 256 (three blocks per compute unit), 4.1 for a cut of
// 64 x 8 nodes with rim, 5.3 for one of 64 x 12; half of it with moment storage.  The other kernels: 4 us and 40 nodes
// per ns, by their tiles' lanes for whole planes, 1.3 (cut planes 1.15) times as long where rows do not fill cache lines.
// (us per step, other kernels -> two FP32 steps per launch: 512 boxes of 32^3 404 -> 264, of 24^3 323 -> 138, of 16^3
// 65.5 -> 52, 200 of 25 x 30 x 20 157 -> 82; 128^3 with 149 points 55.8 -> 42.0, 256^3 with 1000 439 -> 260; left
// alone: 64^3 9.0 / 10.6, one box of 32^3 4.3 / 9.0; 64 x 12 against 64 x 8 nodes: 96^3 24.1 (not marching) -> 17.9,
// 192^3 124 -> 114, 128^3 37.1 / 38.4, 256^3 266 / 284.  Moment storage without points: 128^3
// 53.5 -> 37, 256^3 415 -> 236, 512 boxes of 32^3 495 -> 286, of 16^3 112 -> 50; with a few colloids the estimate
// is short by a tenth: left alone 250 x 60 x 33 26.2 / 26.9.)
int choose_march(const lb_params* p, Plan& P)
{
    const Geom& G = P.Gp;
    const bool fp32 = p->storage == LB_STORAGE_FP32 && p->collision == LB_COLLISION_PROJECTED && !(p->kT > 0.0);
    const bool mom = p->storage == LB_STORAGE_MOM32;
    const double nodes = double(G.N) * G.nboxes;
    // (a plane is addressed with 31-bit byte offsets; lattices near the memory's size have no room for the fields)
    if (!(fp32 || mom) || double(G.ny) * G.rb * 4.0 >= 2.0e9 || double(p->max_points) * 1024.0 > nodes || nodes > 1.1e9) return 0;
    const bool whole = march_whole(G.nx, G.ny);
    const int plane = G.nx * G.ny;
    const double slots = whole && plane <= 256 ? 768 : 256;
    int best = 0;
    double t = 0;
    for (int my : {8, 12}) {
        const double cols = whole ? 1.0 : double((G.nx + 63) / 64) * ((G.ny + my - 1) / my);
        const double unit = (whole ? (plane > 576 ? 7.2 : plane > 256 ? 5.4 : 5.3) : my == 8 ? 4.1 : 5.3) * (mom ? 0.5 : 1.0);
        for (int n = 1; n <= (G.nz + 3) / 4; ++n) {
            const int zc = (G.nz + n - 1) / n;
            const double blocks = cols * ((G.nz + zc - 1) / zc) * G.nboxes, cost = ceil(blocks / slots) * (zc + 2) * unit;
            if (blocks < 2.0e9 && (best == 0 || cost < t)) {
                best = zc;
                P.march_rows = whole ? 0 : my;
                t = cost;
            }
        }
    }
    const bool aligned = (long long)G.nx * 4 % 128 == 0;
    const double lanes = whole ? double(G.ntiles) * BLOCK * (aligned ? 1.0 : 1.3) : nodes * (aligned ? 1.0 : 1.15);
    const double other = (4.0 + lanes / 40.0e3) * (mom ? 1.0 : 2.0);
    P.march_us = t;
    P.other_us = other;
    return best > 0 && t < (mom && !whole ? 0.85 : 0.93) * other ? best : 0;
}

int make_plan(const lb_params* p, Plan& P, std::string& why)
{
    if (!p) { why = "params is NULL"; return LB_ERR_ARG; }
    if (p->nx < 4 || p->ny < 4 || p->nz < 4) { why = "each of nx, ny, nz must be >= 4"; return LB_ERR_ARG; }
    if (p->nboxes < 1) { why = "nboxes must be >= 1"; return LB_ERR_ARG; }
    if (p->storage < LB_STORAGE_FP64 || p->storage > LB_STORAGE_MOM32) { why = "unknown storage"; return LB_ERR_ARG; }
    if (p->max_points < 0) { why = "max_points must be >= 0"; return LB_ERR_ARG; }
    if (!(p->rho0 >= 0.0) || !isfinite(p->rho0)) { why = "rho0 must be finite and >= 0"; return LB_ERR_ARG; }
    if (p->variant < 0 || p->variant > 255) { why = "unknown kernel variant"; return LB_ERR_ARG; }
    if ((p->variant & 128) && ((p->variant >> 2) & 3)) { why = "variant 128 needs one tile per block"; return LB_ERR_ARG; }
    if (p->collision < LB_COLLISION_PROJECTED || p->collision > LB_COLLISION_MRT) {
        why = "unknown collision operator";
        return LB_ERR_ARG;
    }
    if (p->collision == LB_COLLISION_MRT && !(p->ghost_rate > 0.0 && p->ghost_rate <= 4.0)) {
        why = "ghost_rate must be in (0, 4]";
        return LB_ERR_ARG;
    }
    if (p->storage == LB_STORAGE_MOM32 &&
        (p->collision == LB_COLLISION_BGK || (p->collision == LB_COLLISION_MRT && p->ghost_rate != 2.0))) {
        why = "moment storage keeps no ghost moments: the collision must project them out";
        return LB_ERR_ARG;
    }
    if (!(p->kT >= 0.0) || !isfinite(p->kT)) { why = "kT must be finite and >= 0"; return LB_ERR_ARG; }
    if (p->fp16_exponent < -100 || p->fp16_exponent > 120) {
        why = "fp16_exponent must lie in [-100, 120] (the range the scale exponent is kept in)";
        return LB_ERR_ARG;
    }
    if (p->storage == LB_STORAGE_MOM32 && p->kT > 0.0) {
        why = "moment storage keeps no ghost moments: thermal noise needs population storage";
        return LB_ERR_ARG;
    }
    int tx, ty, tz;
    plain_tile(p, P.plain[0], P.plain[1], P.plain[2]);
    P.variant = p->variant;
    if (p->tile_x > 0) {
        tx = p->tile_x;
        ty = p->tile_y;
        tz = p->tile_z;
        P.plain[0] = tx; P.plain[1] = ty; P.plain[2] = tz;
    } else if (p->variant == 0) {
        choose_default(p, tx, ty, tz, P.variant);
    } else {
        tx = P.plain[0]; ty = P.plain[1]; tz = P.plain[2];
    }
    if (!tile_supported(tx, ty, tz)) { why = "unsupported tile shape"; return LB_ERR_ARG; }
    P.cap = p->max_points;
    int r = fill_geometry(p, P.variant, P.cap, tx, ty, tz, P.Gp, why);
    if (r && p->tile_x <= 0 && p->variant == 0) {
        // choose_default goes by speed; what its tile does not serve (a box of 4 GiB and more on narrow rows of lanes,
        // rows of 256 k + 1 ... 3 nodes on 256-node tiles, whose windows meet 75 tiles) takes the plain tile
        P.variant = 0;
        r = fill_geometry(p, 0, P.cap, P.plain[0], P.plain[1], P.plain[2], P.Gp, why);
    }
    if (r) return r;
    P.march_us = P.other_us = 0.0;
    P.march_rows = 0;
    P.march = p->tile_x == 0 && p->variant == 0 ? choose_march(p, P) : 0;
    std::string none;
    int mx, my;
    march_tile(p->nx, p->ny, mx, my);
    if (P.march > 0 && fill_geometry(p, P.variant, P.cap, mx, my, 1, P.Gm, none)) P.march = 0;
    if (P.march == 0) P.Gm = P.Gp;
    P.Gr = P.Gp;
    if (p->storage == LB_STORAGE_FP16 && P.Gp.tx == 128 && p->nx % 128 != 0 && P.variant != p->variant &&
        fill_geometry(p, 0, P.cap, P.plain[0], P.plain[1], P.plain[2], P.Gr, none))
        P.Gr = P.Gp;
    P.G = P.Gp;
    const Geom& G = P.Gp;
    const long long ntiles = std::max(P.Gp.ntiles, P.Gm.ntiles);     // the lists serve both geometries
    const long long maxp = std::max(P.Gp.maxp, P.Gm.maxp);
    P.plain_tiles = tiles_of(G, P.plain);
    P.chunks = std::max(P.Gp.bchunks, P.Gm.bchunks);
    Layout& L = P.L;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o = align_up(o + std::max<size_t>(bytes, 1)); return at; };
    const size_t popb = (size_t)G.sbox * p->nboxes * storage_bytes(p->storage);
    L.pop[0] = take(popb);
    L.pop[1] = take(popb);
    L.boxes = take(sizeof(BoxDev) * p->nboxes);
    L.rec = take(rec_bytes(p->storage) * P.cap);
    L.psum = take(sizeof(double) * 3 * (prep_blocks(P.cap) + LB_MAX_SETS));
    L.count = take(sizeof(int) * ntiles);
    L.cursor = take(sizeof(int) * ntiles);
    L.toff = take(sizeof(int) * (ntiles + 1));
    L.bsum = take(sizeof(int) * scan_blocks(ntiles));
    L.tlist = take(sizeof(int) * P.cap * maxp);
    L.tlist_tmp = take(sizeof(int) * P.cap * maxp);
    L.partial = take(sizeof(double) * 3 * P.cap * maxp);
    L.fpart = take(sizeof(double) * 3 * p->nboxes * P.chunks);
    L.pmax = take(sizeof(float) * p->nboxes * P.chunks);
    L.tmax = take(sizeof(float) * std::max(ntiles, P.plain_tiles));   // (zeros but for batches of FP16 boxes)
    L.smax = take(sizeof(unsigned) * SMAX_SLOTS * SMAX_STRIDE);
    L.ticket = take(sizeof(unsigned) * p->nboxes);
    L.tctr = take(2 * sizeof(unsigned long long));
    L.err = take(sizeof(int) * 4);
    L.nf = take(sizeof(int) * p->nboxes);
    L.rebin = take(sizeof(int));
    L.rebox = take(sizeof(int) * p->nboxes);
    L.win = take(sizeof(int4) * P.cap);
    L.diag = take(sizeof(double) * LBD_N * std::max(ntiles, P.Gr.ntiles));
    L.diagout = take(sizeof(double) * LBD_N * p->nboxes);
    // the marching kernels' force density and velocities (of one step or two) near points
    const size_t field = P.march > 0 && P.cap > 0 ? sizeof(float) * 3 * G.N * p->nboxes : 0;
    L.groups = take(field ? sizeof(unsigned) * P.Gm.ntiles : 0);
    L.field = take(field);
    L.vel[0] = take(field);
    L.vel[1] = take(p->storage == LB_STORAGE_FP32 ? field : 0);
    L.total = o;
    return LB_OK;
}

// set kind of marker sets (curves and surfaces); the public kinds are 0..2
constexpr int KIND_ELASTIC = 100;

struct Set {
    long long n;
    const double* pos;
    const double* frc;
    const int* box;
    int kind;
    lb_point_model model;
    bool has_model;
    lb_elastic el;   // KIND_ELASTIC only
};

// longest captured chunk of steps (a power of two; graphs of 2, 4, ..., GRAPH_MAX steps)
constexpr int GRAPH_MAX = 128;

// Header of a checkpoint (see lb_checkpoint_save): what the state was taken from, and where each
// section starts in the blob.
struct CkptHeader {
    char magic[8];
    int32_t nx, ny, nz, nboxes, storage, collision, tx, ty, tz, pad;
    int64_t steps, npoints, pop_bytes, tiles, total;
    int64_t off_pop, off_boxes, off_tmax, off_smax, off_tctr, off_nf, off_win;
};
constexpr char CKPT_MAGIC[8] = {'l', 'b', 'c', 'k', 'p', 't', '0', '1'};

struct GraphEntry {
    int parity;
    unsigned long long gen;
    int len;
    hipGraph_t graph;
    hipGraphExec_t exec;
};

}  // namespace

struct lb_ctx {
    lb_params p;
    std::vector<double> tau;
    Plan P;
    char* ws;
    hipStream_t stream;
    hipStream_t cap_stream;
    int cur;
    std::vector<Set> sets;
    unsigned long long gen;
    unsigned long long binned_gen;   // gen the tile lists were last forced to rebuild for
    bool bins_valid;
    bool gc_valid;   // counter-force sums current for the registered static sets
    bool field_valid;   // ... and the marching kernels' force field
    std::vector<GraphEntry> graphs;
    bool timing;
    std::vector<hipEvent_t> ev;
    size_t ev_used;
    double timed_ms;
    long long timed_launches;
    long long steps;
    CkptHeader ckpt;   // header of the last checkpoint taken (read by its stream-ordered copy)
    std::vector<BoxDev> hboxes;
    std::string err;

    void* pop(int k) const { return ws + P.L.pop[k]; }
    BoxDev* boxes() const { return (BoxDev*)(ws + P.L.boxes); }
    void* rec() const { return ws + P.L.rec; }
    double* psum() const { return (double*)(ws + P.L.psum); }
    int* count() const { return (int*)(ws + P.L.count); }
    int* cursor() const { return (int*)(ws + P.L.cursor); }
    int* toff() const { return (int*)(ws + P.L.toff); }
    int* bsum() const { return (int*)(ws + P.L.bsum); }
    int* tlist() const { return (int*)(ws + P.L.tlist); }
    int* tlist_tmp() const { return (int*)(ws + P.L.tlist_tmp); }
    double* partial() const { return (double*)(ws + P.L.partial); }
    double* fpart() const { return (double*)(ws + P.L.fpart); }
    float* pmax() const { return (float*)(ws + P.L.pmax); }
    float* tmax() const { return (float*)(ws + P.L.tmax); }
    unsigned* smax() const { return (unsigned*)(ws + P.L.smax); }
    unsigned* ticket() const { return (unsigned*)(ws + P.L.ticket); }
    unsigned long long* tctr() const { return (unsigned long long*)(ws + P.L.tctr); }
    int* errw() const { return (int*)(ws + P.L.err); }
    int* nf() const { return (int*)(ws + P.L.nf); }
    int* rebin() const { return (int*)(ws + P.L.rebin); }
    int* rebox() const { return (int*)(ws + P.L.rebox); }
    int4* win() const { return (int4*)(ws + P.L.win); }
    double* diag() const { return (double*)(ws + P.L.diag); }
    double* diagout() const { return (double*)(ws + P.L.diagout); }
    unsigned* groups() const { return (unsigned*)(ws + P.L.groups); }
    float* field() const { return (float*)(ws + P.L.field); }
    float* vel(int k) const { return (float*)(ws + P.L.vel[k]); }
};

namespace {

thread_local std::string g_err;  // message of the last failure without a context

int fail(lb_ctx* c, int code, const std::string& msg)
{
    if (c)
        c->err = msg;
    else
        g_err = msg;
    return code;
}

// Launch errors are read with hipGetLastError after our own launches; drop
// any error an earlier, unrelated runtime call left behind first.
void clear_stale_error() { (void)hipGetLastError(); }

int hip_check(lb_ctx* c, hipError_t e, const char* what)
{
    if (e == hipSuccess) return LB_OK;
    return fail(c, LB_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

long long total_points(const lb_ctx* c)
{
    long long n = 0;
    for (auto& s : c->sets) n += s.n;
    return n;
}

bool has_kind(const lb_ctx* c, int kind)
{
    for (auto& s : c->sets)
        if (s.kind == kind) return true;
    return false;
}

// Whether a set takes its points' velocities from a step: to move them or to hand them out.
bool takes_velocity(const Set& st)
{
    return st.kind == LB_COLLOIDS || st.kind == KIND_ELASTIC ||
           (st.has_model && (st.model.d_vel_out || st.model.d_vel_sum));
}

bool wants_velocity(const lb_ctx* c)
{
    for (auto& st : c->sets)
        if (takes_velocity(st)) return true;
    return false;
}

// Whether the marching kernels take the steps of the registered sets: two FP32 steps per launch where no point
// moves, moment storage with any sets.  Velocities at fixed points cost a launch more, which lattices just large enough
// to march do not win back: cut planes only from 23 us (moment storage) and 28 us (two FP32 steps) on with the other
// kernels, whole planes of moment storage above 256 nodes from 27 us on (other kernels / marching, left alone: moment
// storage 115 x 28 x 144 17.6 / 23.4, 27 boxes of 29 x 28 x 28 22.5 / 26.3, FP32 127 x 67 x 38 17.3 / 20.8; marching: moment
// storage 93^3 39 -> 32, FP32 80 x 112 x 80 26.3 / 27.8).  Moving points, whose forces change too, cost two launches a
// step (15 to 25 us by the planes) and 6 ns a point (the other kernels: 12 us): only where that leaves a gain (71 boxes of
// 5 x 22 x 18 with 68 23.6 / 26.4).  Below 256 nodes a plane 2 us less from 60 MB (both copies) on, where the other kernels
// no longer find them in the caches (380 boxes of 16 x 7 x 44 106 -> 71, 557 of 12^3 58 -> 52; 413 of 12^3 44 / 46, 319 35 /
// 40).  Up to the bound of
// choose_march the others gain with any number of points, spread out or in one place (us per step, other kernels ->
// marching; fixed points: FP32 256^3 with 16000 425 -> 267, 128^3 with 2000 57 -> 39, 512 boxes of 32^3 with 512 and their
// velocities 410 -> 259, all in one box 411 -> 259; moment storage 128^3 with 100 56 -> 41; colloids: moment storage
// 256^3 with 1000 432 -> 302, 10^4 437 -> 343, 10^4 within 32^3 nodes 503 -> 372, 16000 440 -> 363, 192^3 with 6000 197 ->
// 170, 300 x 200 x 100 with 9 197 -> 132, 512 boxes of 24^3 with 2000 327 -> 173; left alone: 128^3 with 500 65 / 67, 40 boxes of 25^3 29 / 38).
bool marches(const Plan& P, int storage, long long points, bool velocities, bool moving)
{
    if (P.march == 0) return false;
    const bool mom = storage == LB_STORAGE_MOM32;
    const bool cut = P.march_rows > 0, large = P.Gm.nx * P.Gm.ny > 256;
    if (!moving) return !velocities || P.other_us >= (cut ? (mom ? 23.0 : 28.0) : mom && large ? 27.0 : 0.0);
    if (!mom) return false;
    const double more = cut ? 25.0 : large ? 22.0 : double(P.Gm.N) * P.Gm.nboxes > 0.75e6 ? 15.0 : 17.0;
    return P.march_us + more + 0.006 * double(points) < 0.93 * (P.other_us + 12.0);
}

bool marches(const lb_ctx* c)
{
    return marches(c->P, c->p.storage, total_points(c), wants_velocity(c), has_kind(c, LB_COLLOIDS) || has_kind(c, KIND_ELASTIC));
}

// The geometry (tiles of the point lists) for the registered sets; called when they change, which also
// makes the lists be built again.
// FP32 steps that do not pair (calls of one to three, the rest of a call by fours, timing) run the one-node kernel on the
// marching kernels' list tile.  Without points, where they could take their own, that gives no gain: 300 x 200 x 100 270 us
// on the list tile, 276 on their own, 256^3 436 / 441, 96^3 27 / 24.
void set_geometry(lb_ctx* c) { c->P.G = marches(c) ? c->P.Gm : c->P.Gp; }

// Geometry of the moments and the diagnostics between steps.  Without points any tile serves: that of single steps, or the
// plain one in FP16 where a read's one node per lane would leave lanes of a 128-node tile idle (moments of 160^3 56 ->
// 45 us); the diagnostics, bound by arithmetic, keep the marching kernels' tile, which leaves none idle (192^3
// FP32 159 against 193).  Block order of a caller who leaves the choice to the library (choose_default's is for steps):
// contiguous runs per XCD, as with variant 0, but for the moments of populations on whole cache lines from 400 MB a
// copy on and for moment storage on whole lines or narrow rows.  (Tile rows on one XCD -> contiguous runs: moments FP32
// 300 x 200 x 100 133 -> 117 us, 160^3 79 -> 70, 300 boxes of 24^3 92 -> 78, FP16 300 x 64 x 60 19 -> 16.5; left: FP32 192^3
// with 4000 points 123 / 129, 256^3 302 / 324, moment storage 256^3 397 / 433, 100 boxes of 48^3 305 / 318.
// Diagnostics FP64 192^3 254 -> 225, FP32 1000 boxes of 16^3 132 -> 119; left: moment storage 512^3 3091 / 3300.)
Geom read_geometry(const lb_ctx* c, bool diagnostics)
{
    const lb_params& p = c->p;
    Geom G = total_points(c) > 0 || (diagnostics && c->P.march > 0) ? c->P.G : c->P.Gr;
    G.tpb = 1;
    if (p.tile_x > 0 || p.variant != 0) return G;
    const bool mom = p.storage == LB_STORAGE_MOM32;
    const bool lines = (long long)(G.nx * storage_bytes(p.storage)) % 128 == 0;
    const double copy = double(G.sbox) * G.nboxes * storage_bytes(p.storage);
    if (mom ? !lines && G.nx > 64 : diagnostics || !lines || copy < 400.0e6) {
        G.order = 0;
        G.lgrp = 0;
    }
    return G;
}

// After the sets change, the next list build must run whatever the positions:
// raise the rebuild flag once per change.  Enqueued eagerly, never into a
// captured graph (a graph replays every node it holds).
void force_rebin(lb_ctx* c, hipStream_t s)
{
    if (c->binned_gen == c->gen) return;
    launch_fill_u32(c->rebin(), 1, 1u, s);
    launch_fill_u32(c->rebox(), c->p.nboxes, 1u, s);
    c->binned_gen = c->gen;
}

// blocks of point-force sums the records kernel writes (one box only; see k_prep)
long long npsum(const lb_ctx* c)
{
    long long nb = 0;
    for (auto& s : c->sets) nb += prep_blocks(s.n);
    return nb;
}

// tile bins for the points' records (the kernels rebuild the lists only while the rebuild flag is set)
void build_lists(lb_ctx* c, hipStream_t s)
{
    launch_bins(c->p.storage, c->P.G, total_points(c), c->rec(), c->count(), c->bsum(), c->toff(), c->cursor(), c->tlist(),
                c->tlist_tmp(), c->errw(), s);
}

// records + tile bins for the current point positions
void build_points(lb_ctx* c, hipStream_t s)
{
    const Geom& G = c->P.G;
    long long off = 0, blk = 0;
    for (auto& st : c->sets) {
        double* ps = G.nboxes == 1 ? c->psum() + 3 * blk : nullptr;
        launch_prep(c->p.storage, G, st.n, off, st.pos, st.frc, st.box, c->rec(), c->errw(), ps, s);
        off += st.n;
        blk += prep_blocks(st.n);
    }
    build_lists(c, s);
    c->gc_valid = false;
    c->field_valid = false;
}

// per-box work before a step or a read: the counter-force sums (only when the
// point records may have changed since they were last taken) and the FP16
// exponent of the coming step
void box_update(lb_ctx* c, hipStream_t s, bool fp16_exp)
{
    const bool sums = c->p.zero_net_force != 0 && !c->gc_valid;
    const bool fp16 = fp16_exp && c->p.storage == LB_STORAGE_FP16;
    if (!sums && !fp16) return;
    const bool one = c->P.G.nboxes == 1;
    launch_box_update(c->p.storage, c->P.G, c->rec(), total_points(c) > 0 ? c->toff() : nullptr, c->tlist(),
                      one ? c->psum() : nullptr, one ? npsum(c) : 0, c->tmax(), c->fpart(), c->pmax(), c->ticket(),
                      c->boxes(), sums ? 1 : 0, fp16 ? 1 : 0, s);
    if (sums) c->gc_valid = true;
}

// marker forces of the curve and surface sets from their current configuration
void elastic_forces(lb_ctx* c, hipStream_t s)
{
    const Geom& G = c->P.G;
    for (auto& st : c->sets)
        if (st.kind == KIND_ELASTIC) {
            ElasticLaunch e;
            e.kind = st.el.kind;
            e.chain_len = st.el.chain_len;
            e.n = st.n;
            e.pos = st.pos;
            e.ext = st.el.d_ext;
            e.frc = st.el.d_force;
            e.k_spring = st.el.k_spring;
            e.l0 = st.el.l0;
            e.tension = st.el.tension;
            e.tri = st.el.d_tri;
            e.vt_off = st.el.d_vt_off;
            e.vt_idx = st.el.d_vt_idx;
            launch_elastic_forces(G, e, s);
        }
}

// Whether the steps of one call hand over from one to the next: the move kernel of a step then writes the
// points' records of the step that follows (and one box's FP16 exponent), so that a step is three launches
// instead of five: step kernel, move, list check.  Forces are the caller's arrays, the same throughout a call,
// so their sums stand; the markers of curves and surfaces get new forces every step from their
// neighbours' positions, which no single kernel has.  48^3 with 321 colloids:
// 18.4 -> 14.8 us a step, 128^3 with 1000 Brownian ones 75.0 -> 70.8.
bool hands_over(const lb_ctx* c)
{
    return has_kind(c, LB_COLLOIDS) && !has_kind(c, KIND_ELASTIC) && !has_kind(c, LB_FORCES_NEXT_STEP);
}

// Outputs and moves of the sets' points from a step's interpolation partials; before and fp16_exp as in
// enqueue_step.
void move_points(lb_ctx* c, hipStream_t s, void* partial, const unsigned long long* tin, bool before, bool fp16_exp)
{
    const Geom& G = c->P.G;
    long long off = 0;
    for (auto& st : c->sets) {
        const bool adv = st.kind == LB_COLLOIDS || st.kind == KIND_ELASTIC;
        if (takes_velocity(st)) {
            AdvectLaunch a;
            memset(&a, 0, sizeof(a));
            a.n = st.n;
            a.off = off;
            a.frc = st.frc;
            a.pos = (double*)st.pos;
            a.boxid = st.box;
            a.advect = adv ? 1 : 0;
            a.tin = st.kind == LB_COLLOIDS ? tin : nullptr;   // markers of curves and surfaces: no zeta'

            if (st.has_model) {
                a.vel_out = st.model.d_vel_out;
                a.vel_sum = st.model.d_vel_sum;
                a.inv_a = st.model.inv_a;
                a.inv_aL = st.model.inv_aL;
                a.mlp = st.model.d_mlp;
                for (int k = 0; k < 4; ++k) {
                    a.in_shift[k] = st.model.in_shift[k];
                    a.in_scale[k] = st.model.in_scale[k];
                }
                a.out_scale = st.model.out_scale;
            }
            if (before && st.kind == LB_COLLOIDS) {
                a.rec = c->rec();
                a.err = c->errw();
                a.fp16_exp = fp16_exp ? 1 : 0;
                fp16_exp = false;
            }
            launch_advect(c->p.storage, G, a, c->boxes(), partial, s);
        }
        off += st.n;
    }
}

// one step on stream s; flips c->cur.  after: the step before it in this call handed over; before: this
// one hands over to another
void enqueue_step(lb_ctx* c, hipStream_t s, bool rebuild, bool after = false, bool before = false)
{
    const Geom& G = c->P.G;
    const long long npts = total_points(c);
    const bool one_box_fp16 = c->p.storage == LB_STORAGE_FP16 && G.nboxes == 1;
    elastic_forces(c, s);
    if (after)
        build_lists(c, s);
    else if (npts > 0 && rebuild)
        build_points(c, s);
    if (!(after && one_box_fp16)) box_update(c, s, true);
    bool fp16_exp = before && one_box_fp16;   // the first colloid set's kernel takes it
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (c->timing) {
        if (c->ev_used + 2 > c->ev.size()) {
            for (int k = 0; k < 256; ++k) {
                hipEvent_t e;
                (void)hipEventCreate(&e);
                c->ev.push_back(e);
            }
        }
        e0 = c->ev[c->ev_used++];
        e1 = c->ev[c->ev_used++];
        c->timed_launches++;
    }
    unsigned long long* tin = G.coll == 2 ? c->tctr() + c->cur : nullptr;
    unsigned long long* tout = G.coll == 2 ? c->tctr() + (c->cur ^ 1) : nullptr;
    const int* toff = npts > 0 ? c->toff() : nullptr;
    if (c->p.storage == LB_STORAGE_MOM32 && marches(c)) {
        float* v = npts > 0 && wants_velocity(c) ? c->vel(0) : nullptr;
        if (npts > 0 && rebuild) launch_force_field(G, c->boxes(), toff, c->tlist(), c->rec(), c->groups(), c->field(), s);
        launch_march(c->p.storage, G, c->P.march_rows, c->P.march, c->pop(c->cur), c->pop(c->cur ^ 1), c->boxes(), toff, c->groups(), c->field(), v, nullptr,
                     s, e0, e1);
        if (v) launch_partials(G, npts, c->rec(), v, nullptr, (float*)c->partial(), nullptr, s);
    } else
        launch_lattice(c->p.storage, G, 0, c->P.variant, c->pop(c->cur), c->pop(c->cur ^ 1), c->boxes(), toff, c->tlist(),
                       c->rec(), c->partial(), (double*)c->tmax(), tin, tout, s, e0, e1);
    move_points(c, s, c->partial(), tin, before, fp16_exp);
    c->cur ^= 1;
}

// n steps.  FP32 runs that the marching kernel takes go two steps a launch, by fours, so that calls end on the
// population copy they always ended on (which captured graphs, the caller's too, rely on).
void enqueue_steps(lb_ctx* c, hipStream_t s, bool rebuild, int n)
{
    if (c->p.storage == LB_STORAGE_FP32 && !c->timing && marches(c)) {
        // the partials of the second step behind those of the first (the workspace holds FP64's)
        const long long npts = total_points(c);
        const int* toff = npts > 0 ? c->toff() : nullptr;
        float* p0 = wants_velocity(c) ? (float*)c->partial() : nullptr;
        float* p1 = p0 ? p0 + 3 * c->P.cap * c->P.G.maxp : nullptr;
        float *v0 = p0 ? c->vel(0) : nullptr, *v1 = p0 ? c->vel(1) : nullptr;
        for (int pairs = n / 4 * 2; pairs > 0; --pairs) {
            box_update(c, s, true);
            launch_march(c->p.storage, c->P.G, c->P.march_rows, c->P.march, c->pop(c->cur), c->pop(c->cur ^ 1), c->boxes(), toff, c->groups(), c->field(), v0,
                         v1, s);
            if (p0) {
                launch_partials(c->P.G, npts, c->rec(), v0, v1, p0, p1, s);
                move_points(c, s, p0, nullptr, false, false);
                move_points(c, s, p1, nullptr, false, false);
            }
            c->cur ^= 1;
        }
        n %= 4;
    }
    const bool over = rebuild && hands_over(c);
    for (int k = 0; k < n; ++k) enqueue_step(c, s, rebuild, over && k > 0, over && k + 1 < n);
}

void drop_graphs(lb_ctx* c)
{
    for (auto& g : c->graphs) {
        (void)hipGraphExecDestroy(g.exec);
        (void)hipGraphDestroy(g.graph);
    }
    c->graphs.clear();
}

// graph of len (even) steps from the current parity; captured on first use
int get_graph(lb_ctx* c, bool rebuild, int len, hipGraphExec_t* out)
{
    for (auto& g : c->graphs)
        if (g.parity == c->cur && g.gen == c->gen && g.len == len) {
            *out = g.exec;
            return LB_OK;
        }
    if (!c->cap_stream) {
        int r = hip_check(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking), "hipStreamCreate");
        if (r) return r;
    }
    const int parity = c->cur;
    int r = hip_check(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed), "hipStreamBeginCapture");
    if (r) return r;
    enqueue_steps(c, c->cap_stream, rebuild, len);   // len even: parity restored
    hipGraph_t graph;
    r = hip_check(c, hipStreamEndCapture(c->cap_stream, &graph), "hipStreamEndCapture");
    if (r) return r;
    hipGraphExec_t exec;
    r = hip_check(c, hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0), "hipGraphInstantiate");
    if (r) {
        (void)hipGraphDestroy(graph);
        return r;
    }
    c->graphs.push_back({parity, c->gen, len, graph, exec});
    *out = exec;
    return LB_OK;
}

int check_async(lb_ctx* c)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, LB_ERR_HIP, std::string("launch failed: ") + hipGetErrorString(e));
    return LB_OK;
}

}  // namespace

extern "C" {

int lb_workspace_bytes(const lb_params* p, size_t* bytes)
{
    if (!bytes) return fail(nullptr, LB_ERR_ARG, "bytes is NULL");
    Plan P;
    std::string why;
    const int r = make_plan(p, P, why);
    if (r) return fail(nullptr, r, why);
    *bytes = P.L.total;
    return LB_OK;
}

int lb_plan(const lb_params* p, int64_t npoints, int32_t velocities, lb_plan_info* out)
{
    if (!out) return fail(nullptr, LB_ERR_ARG, "out is NULL");
    if (npoints < 0 || velocities < 0 || velocities > 2) return fail(nullptr, LB_ERR_ARG, "npoints or velocities out of range");
    Plan P;
    std::string why;
    const int r = make_plan(p, P, why);
    if (r) return fail(nullptr, r, why);
    const bool m = marches(P, p->storage, npoints, npoints > 0 && velocities > 0, npoints > 0 && velocities == 2);
    const Geom& G = m ? P.Gm : P.Gp;
    out->tile_x = G.tx;
    out->tile_y = G.ty;
    out->tile_z = G.tz;
    out->variant = P.variant;
    out->march_planes = m ? P.march : 0;
    out->march_rows = m ? P.march_rows : 0;
    return LB_OK;
}

int lb_init(const lb_params* p, void* d_workspace, size_t bytes, void* hip_stream, lb_ctx** out)
{
    if (!out) return fail(nullptr, LB_ERR_ARG, "out is NULL");
    *out = nullptr;
    clear_stale_error();
    Plan P;
    std::string why;
    int r = make_plan(p, P, why);
    if (r) return fail(nullptr, r, why);
    if (!p->tau) return fail(nullptr, LB_ERR_ARG, "tau is NULL");
    for (int b = 0; b < p->nboxes; ++b)
        if (!(p->tau[b] > 0.0) || !isfinite(p->tau[b])) return fail(nullptr, LB_ERR_ARG, "tau must be finite and > 0");
    if (p->collision == LB_COLLISION_MRT && p->tau_bulk)
        for (int b = 0; b < p->nboxes; ++b)
            if (!(p->tau_bulk[b] > 0.0) || !isfinite(p->tau_bulk[b]))
                return fail(nullptr, LB_ERR_ARG, "tau_bulk must be finite and > 0");
    if (!d_workspace || ((uintptr_t)d_workspace % ALIGN) != 0)
        return fail(nullptr, LB_ERR_ARG, "workspace NULL or not 256-byte aligned");
    if (bytes < P.L.total) return fail(nullptr, LB_ERR_SIZE, "workspace too small");
    lb_ctx* c = new lb_ctx();
    c->p = *p;
    c->tau.assign(p->tau, p->tau + p->nboxes);
    c->p.tau = c->tau.data();
    c->p.tau_bulk = nullptr;   // read below, not kept
    c->P = P;
    c->ws = (char*)d_workspace;
    for (Geom* g : {&c->P.Gp, &c->P.Gm, &c->P.Gr}) {
        g->nf = c->nf();
        g->rebin = c->rebin();
        g->rebox = c->rebox();
        g->win = c->win();
        g->smax = (p->storage == LB_STORAGE_FP16 && p->nboxes == 1) ? c->smax() : nullptr;
    }
    set_geometry(c);
    c->stream = (hipStream_t)hip_stream;
    c->cap_stream = nullptr;
    c->cur = 0;
    c->gen = 1;
    c->binned_gen = 0;
    c->bins_valid = false;
    c->gc_valid = false;
    c->field_valid = false;
    c->timing = false;
    c->ev_used = 0;
    c->timed_ms = 0.0;
    c->timed_launches = 0;
    c->steps = 0;
    int e0 = p->fp16_exponent != 0 ? p->fp16_exponent : 30;
    if (p->fp16_exponent == 0 && p->kT > 0.0) {
        // thermal populations from the first step on: per population the noise of the 15 modes
        // has standard deviation at most sqrt(mu rho / w_i) <= 6 sqrt(mu rho) in units of w_i
        // (completeness of the mode basis); keep 6 of those deviations under 2^14
        const double amp = 36.0 * sqrt(3.0 * p->kT * P.G.rho0);
        e0 = std::min(30, int(floor(log2(16384.0 / amp))));
    }
    c->hboxes.resize(p->nboxes);
    for (int b = 0; b < p->nboxes; ++b) {
        BoxDev& B = c->hboxes[b];
        memset(&B, 0, sizeof(B));
        B.tau = p->tau[b];
        B.omega = 1.0 / (p->tau[b] + 0.5);
        B.tau_b = (p->collision == LB_COLLISION_MRT && p->tau_bulk) ? p->tau_bulk[b] : p->tau[b];
        B.omega_b = 1.0 / (B.tau_b + 0.5);
        // eigenvalue r of a ghost mode: the moment is multiplied by (1 - r/2) / (1 + r/2)
        const double r = p->collision == LB_COLLISION_BGK ? 1.0 / p->tau[b]
                         : p->collision == LB_COLLISION_MRT ? p->ghost_rate : 2.0;
        B.kappa_g = (1.0 - 0.5 * r) / (1.0 + 0.5 * r);
        // thermal noise: a mode whose non-equilibrium part is multiplied by gamma receives
        // variance mu rho b (1 - gamma^2), mu = kT / cs^2
        const double mu = 3.0 * p->kT;
        const double gb = 1.0 - B.omega_b, gs = 1.0 - B.omega, gg = B.kappa_g;
        B.nz_b = sqrt(mu * (1.0 - gb * gb));
        B.nz_s = sqrt(mu * (1.0 - gs * gs));
        B.nz_g = sqrt(mu * (1.0 - gg * gg));
        const double eta = P.G.rho0 * p->tau[b] / 3.0;
        B.pn = p->kT / (3.0 * M_PI * eta);
        B.inv6pe = 1.0 / (6.0 * M_PI * eta);
        B.e_data = e0;
        B.s_in = ldexpf(1.0f, -e0);
        B.s_out = ldexpf(1.0f, e0);
    }
    hipStream_t s = c->stream;
    const Geom& G = c->P.G;
    const size_t popb = (size_t)G.sbox * p->nboxes * storage_bytes(p->storage);
    launch_fill_u32(c->pop(0), (long long)(popb / 4), 0u, s);
    launch_fill_u32(c->pop(1), (long long)(popb / 4), 0u, s);
    const long long ntiles = std::max(c->P.Gp.ntiles, c->P.Gm.ntiles);
    launch_fill_u32(c->count(), ntiles, 0u, s);
    launch_fill_u32(c->cursor(), ntiles, 0u, s);
    launch_fill_u32(c->toff(), ntiles + 1, 0u, s);
    launch_fill_u32(c->ticket(), p->nboxes, 0u, s);
    launch_fill_u32(c->tctr(), 4, 0u, s);
    launch_fill_u32(c->tmax(), std::max(ntiles, c->P.plain_tiles), 0u, s);
    launch_fill_u32(c->smax(), SMAX_SLOTS * SMAX_STRIDE, 0u, s);
    launch_fill_u32(c->errw(), 4, 0u, s);
    launch_fill_u32(c->nf(), p->nboxes, 0u, s);
    launch_fill_u32(c->rebin(), 1, 1u, s);
    launch_fill_u32(c->rebox(), p->nboxes, 1u, s);
    launch_fill_u32(c->win(), 4 * c->P.cap, 0u, s);
    r = hip_check(c, hipMemcpyAsync(c->boxes(), c->hboxes.data(), sizeof(BoxDev) * p->nboxes, hipMemcpyHostToDevice, s),
                  "hipMemcpyAsync");
    if (!r) r = check_async(c);
    if (r) {
        g_err = c->err;
        delete c;
        return r;
    }
    *out = c;
    return LB_OK;
}

int lb_set_stream(lb_ctx* c, void* hip_stream)
{
    if (!c) return LB_ERR_ARG;
    c->stream = (hipStream_t)hip_stream;
    return LB_OK;
}

int lb_set_equilibrium(lb_ctx* c, const double* d_rho, const double* d_u)
{
    if (!c) return LB_ERR_ARG;
    clear_stale_error();
    if (!d_rho || !d_u) return fail(c, LB_ERR_ARG, "lb_set_equilibrium: NULL field");
    launch_equilibrium(c->p.storage, c->P.G, c->pop(c->cur), c->boxes(), d_rho, d_u, c->stream);
    return check_async(c);
}

int lb_add_point_forces(lb_ctx* c, int64_t n, const double* d_pos, const double* d_force, const int32_t* d_box,
                        int kind, const lb_point_model* model)
{
    if (!c) return LB_ERR_ARG;
    if (n < 0) return fail(c, LB_ERR_ARG, "n < 0");
    if (n > 0 && (!d_pos || !d_force)) return fail(c, LB_ERR_ARG, "NULL positions or forces");
    if (kind != LB_FORCES_NEXT_STEP && kind != LB_FORCES_STATIC && kind != LB_COLLOIDS)
        return fail(c, LB_ERR_ARG, "unknown kind");
    if (kind == LB_COLLOIDS) {
        if (!model) return fail(c, LB_ERR_ARG, "colloids need a model (a, a_L)");
        if (!(model->inv_a > model->inv_aL) || !isfinite(model->inv_a) || !isfinite(model->inv_aL))
            return fail(c, LB_ERR_ARG, "need 1/a > 1/a_L (a < a_L) for a positive renormalised radius");
    }
    if ((int)c->sets.size() >= LB_MAX_SETS) return fail(c, LB_ERR_CAPACITY, "too many sets");
    if (total_points(c) + n > c->P.cap) return fail(c, LB_ERR_CAPACITY, "more points than max_points");
    if (n == 0) return LB_OK;
    Set s;
    s.n = n;
    s.pos = d_pos;
    s.frc = d_force;
    s.box = (const int*)d_box;
    s.kind = kind;
    s.has_model = model != nullptr;
    if (model)
        s.model = *model;
    else
        memset(&s.model, 0, sizeof(s.model));
    c->sets.push_back(s);
    set_geometry(c);
    c->gen++;
    c->bins_valid = false;
    c->gc_valid = false;
    c->field_valid = false;
    return LB_OK;
}

int lb_add_elastic(lb_ctx* c, const lb_elastic* e)
{
    if (!c) return LB_ERR_ARG;
    if (!e) return fail(c, LB_ERR_ARG, "lb_add_elastic: set is NULL");
    if (e->kind != LB_ELASTIC_CHAIN && e->kind != LB_ELASTIC_SURFACE) return fail(c, LB_ERR_ARG, "unknown elastic kind");
    if (e->n <= 0 || !e->d_pos || !e->d_force) return fail(c, LB_ERR_ARG, "elastic set: n <= 0 or NULL arrays");
    if (e->kind == LB_ELASTIC_CHAIN) {
        if (e->chain_len < 2 || e->n % e->chain_len != 0)
            return fail(c, LB_ERR_ARG, "chain: chain_len >= 2 and n a multiple of it");
        if (!isfinite(e->k_spring) || !isfinite(e->l0) || e->l0 < 0.0)
            return fail(c, LB_ERR_ARG, "chain: finite k_spring and l0 >= 0");
    } else {
        if (e->ntri <= 0 || !e->d_tri || !e->d_vt_off || !e->d_vt_idx)
            return fail(c, LB_ERR_ARG, "surface: ntri > 0 and the triangle and incidence arrays");
        if (!isfinite(e->tension)) return fail(c, LB_ERR_ARG, "surface: finite tension");
        if (e->n > INT32_MAX) return fail(c, LB_ERR_ARG, "surface: too many vertices");
    }
    if ((int)c->sets.size() >= LB_MAX_SETS) return fail(c, LB_ERR_CAPACITY, "too many sets");
    if (total_points(c) + e->n > c->P.cap) return fail(c, LB_ERR_CAPACITY, "more points than max_points");
    Set s;
    s.n = e->n;
    s.pos = e->d_pos;
    s.frc = e->d_force;
    s.box = (const int*)e->d_box;
    s.kind = KIND_ELASTIC;
    memset(&s.model, 0, sizeof(s.model));
    s.model.d_vel_out = e->d_vel_out;
    s.has_model = true;   // inv_a = inv_aL = 0: the markers move with U alone
    s.el = *e;
    c->sets.push_back(s);
    set_geometry(c);
    c->gen++;
    c->bins_valid = false;
    c->gc_valid = false;
    c->field_valid = false;
    return LB_OK;
}

int lb_clear_forces(lb_ctx* c)
{
    if (!c) return LB_ERR_ARG;
    c->sets.clear();
    set_geometry(c);
    c->gen++;
    c->bins_valid = false;
    c->gc_valid = false;
    c->field_valid = false;
    return LB_OK;
}

int lb_step(lb_ctx* c, int32_t nsteps)
{
    if (!c) return LB_ERR_ARG;
    clear_stale_error();
    if (nsteps < 0) return fail(c, LB_ERR_ARG, "nsteps < 0");
    if (nsteps == 0) return LB_OK;
    int left = nsteps;
    force_rebin(c, c->stream);
    if (has_kind(c, LB_FORCES_NEXT_STEP)) {
        enqueue_step(c, c->stream, true);
        c->sets.erase(std::remove_if(c->sets.begin(), c->sets.end(),
                                     [](const Set& s) { return s.kind == LB_FORCES_NEXT_STEP; }),
                      c->sets.end());
        set_geometry(c);
        c->gen++;
        c->bins_valid = false;
        c->gc_valid = false;
        c->field_valid = false;
        c->steps++;
        left--;
        force_rebin(c, c->stream);
    }
    const bool moving = has_kind(c, LB_COLLOIDS) || has_kind(c, KIND_ELASTIC);
    const bool pts = total_points(c) > 0;
    if (left > 0 && pts && !moving && !c->bins_valid) {
        build_points(c, c->stream);
        c->bins_valid = true;
    }
    if (left > 0 && !moving) {
        // static sums and the force field outside any captured graph
        box_update(c, c->stream, false);
        if (pts && marches(c) && !c->field_valid &&
            (c->p.storage == LB_STORAGE_MOM32 || (left >= 4 && !c->timing))) {
            launch_force_field(c->P.G, c->boxes(), c->toff(), c->tlist(), c->rec(), c->groups(), c->field(), c->stream);
            c->field_valid = true;
        }
    }
    const bool rebuild = moving;
    if (c->timing || left < 4) {
        enqueue_steps(c, c->stream, rebuild, left);
    } else {
        // the longest power-of-two chunks first
        int rest = left;
        while (rest >= 2) {
            int len = GRAPH_MAX;
            while (len > rest) len >>= 1;
            hipGraphExec_t exec;
            int r = get_graph(c, rebuild, len, &exec);
            if (r) return r;
            for (; rest >= len; rest -= len) {
                r = hip_check(c, hipGraphLaunch(exec, c->stream), "hipGraphLaunch");
                if (r) return r;
            }
        }
        if (rest) enqueue_step(c, c->stream, rebuild);
    }
    c->steps += left;
    return check_async(c);
}

int lb_prepare_steps(lb_ctx* c, int32_t nsteps)
{
    if (!c) return LB_ERR_ARG;
    clear_stale_error();
    if (nsteps < 0) return fail(c, LB_ERR_ARG, "nsteps < 0");
    // the same chunks as lb_step; a pending next-step set changes the sets after the first step
    if (has_kind(c, LB_FORCES_NEXT_STEP) || c->timing || nsteps < 4) return LB_OK;
    const bool rebuild = has_kind(c, LB_COLLOIDS) || has_kind(c, KIND_ELASTIC);
    int rest = nsteps;
    while (rest >= 2) {
        int len = GRAPH_MAX;
        while (len > rest) len >>= 1;
        hipGraphExec_t exec;
        const int r = get_graph(c, rebuild, len, &exec);
        if (r) return r;
        while (rest >= len) rest -= len;
    }
    return LB_OK;
}

static int prepare_fields(lb_ctx* c)
{
    if (total_points(c) > 0) {
        force_rebin(c, c->stream);
        elastic_forces(c, c->stream);
        build_points(c, c->stream);
        if (!has_kind(c, LB_COLLOIDS) && !has_kind(c, KIND_ELASTIC)) c->bins_valid = true;
    }
    box_update(c, c->stream, false);
    return LB_OK;
}

int lb_moments(lb_ctx* c, double* d_rho, double* d_u)
{
    if (!c) return LB_ERR_ARG;
    clear_stale_error();
    if (!d_u) return fail(c, LB_ERR_ARG, "lb_moments: d_u is NULL");
    prepare_fields(c);
    launch_lattice(c->p.storage, read_geometry(c, false), 1, 0, c->pop(c->cur), nullptr, c->boxes(),
                   total_points(c) > 0 ? c->toff() : nullptr, c->tlist(), c->rec(), d_rho, d_u, nullptr, nullptr,
                   c->stream);
    return check_async(c);
}

int lb_interp_velocity(lb_ctx* c, int64_t n, const double* d_pos, const int32_t* d_box, double* d_u_out)
{
    if (!c) return LB_ERR_ARG;
    clear_stale_error();
    if (n < 0) return fail(c, LB_ERR_ARG, "n < 0");
    if (n == 0) return LB_OK;
    if (!d_pos || !d_u_out) return fail(c, LB_ERR_ARG, "NULL positions or output");
    prepare_fields(c);
    launch_interp_points(c->p.storage, c->P.G, n, d_pos, (const int*)d_box, d_u_out, c->pop(c->cur), c->boxes(),
                         total_points(c) > 0 ? c->toff() : nullptr, c->tlist(), c->rec(), c->stream);
    return check_async(c);
}

static int read_flags(lb_ctx* c)
{
    int errw[4];
    int r = hip_check(c, hipMemcpyAsync(errw, c->errw(), sizeof(errw), hipMemcpyDeviceToHost, c->stream), "hipMemcpy");
    if (r) return r;
    std::vector<int> nf(c->p.nboxes);
    r = hip_check(c, hipMemcpyAsync(nf.data(), c->nf(), sizeof(int) * c->p.nboxes, hipMemcpyDeviceToHost, c->stream),
                  "hipMemcpy");
    if (r) return r;
    r = hip_check(c, hipStreamSynchronize(c->stream), "hipStreamSynchronize");
    if (r) return r;
    if (errw[0] & 1) {
        launch_fill_u32(c->errw(), 4, 0u, c->stream);
        return fail(c, LB_ERR_ARG, "a point names a box id out of range");
    }
    if (errw[0] & 2) {
        launch_fill_u32(c->errw(), 4, 0u, c->stream);
        return fail(c, LB_ERR_NONFINITE, "non-finite point position or force");
    }
    if (errw[0] & 4) {
        launch_fill_u32(c->errw(), 4, 0u, c->stream);
        return fail(c, LB_ERR_STATE, "tile-list rebuild: a grid barrier wait ran out (lists may be incomplete)");
    }
    for (int b = 0; b < c->p.nboxes; ++b)
        if (nf[b]) return fail(c, LB_ERR_NONFINITE, "non-finite value or FP16 overflow in box " + std::to_string(b));
    return LB_OK;
}

int lb_diagnostics(lb_ctx* c, double* h_out)
{
    if (!c) return LB_ERR_ARG;
    clear_stale_error();
    if (!h_out) return fail(c, LB_ERR_ARG, "h_out is NULL");
    prepare_fields(c);
    const Geom G = read_geometry(c, true);
    launch_lattice(c->p.storage, G, 2, 0, c->pop(c->cur), nullptr, c->boxes(), total_points(c) > 0 ? c->toff() : nullptr,
                   c->tlist(), c->rec(), c->diag(), nullptr, nullptr, nullptr, c->stream);
    launch_diag_reduce(G, c->diag(), c->diagout(), c->stream);
    int r = check_async(c);
    if (r) return r;
    r = hip_check(c,
                  hipMemcpyAsync(h_out, c->diagout(), sizeof(double) * LBD_N * c->p.nboxes, hipMemcpyDeviceToHost,
                                 c->stream),
                  "hipMemcpy");
    if (r) return r;
    r = read_flags(c);   // waits for the copy
    if (r) return r;
    for (int b = 0; b < c->p.nboxes; ++b)
        if (h_out[(size_t)b * LBD_N + 12] > 0.0)
            return fail(c, LB_ERR_NEGATIVE_DENSITY, "non-positive density in box " + std::to_string(b));
    return LB_OK;
}

int lb_sync(lb_ctx* c)
{
    if (!c) return LB_ERR_ARG;
    int r = check_async(c);
    if (r) return r;
    return read_flags(c);
}

// Layout of a checkpoint that names tile t: this context's own (P.plain), or one it accepts.
static CkptHeader ckpt_layout(const lb_ctx* c, const int (&t)[3])
{
    CkptHeader h;
    memset(&h, 0, sizeof(h));
    memcpy(h.magic, CKPT_MAGIC, 8);
    const Geom& G = c->P.G;
    h.nx = G.nx; h.ny = G.ny; h.nz = G.nz; h.nboxes = G.nboxes;
    h.storage = c->p.storage; h.collision = c->p.collision;
    h.tx = t[0]; h.ty = t[1]; h.tz = t[2];
    h.steps = c->steps;
    h.npoints = total_points(c);
    h.pop_bytes = (int64_t)G.sbox * G.nboxes * (int64_t)storage_bytes(c->p.storage);
    const int64_t tiles = h.tiles = tiles_of(G, t);
    size_t o = align_up(sizeof(CkptHeader));
    auto take = [&](size_t b) { const size_t at = o; o = align_up(o + std::max<size_t>(b, 1)); return (int64_t)at; };
    h.off_pop = take(h.pop_bytes);
    h.off_boxes = take(sizeof(BoxDev) * G.nboxes);
    h.off_tmax = take(sizeof(float) * tiles);
    h.off_smax = take(sizeof(unsigned) * SMAX_SLOTS * SMAX_STRIDE);
    h.off_tctr = take(sizeof(unsigned long long));
    h.off_nf = take(sizeof(int) * G.nboxes);
    h.off_win = take(sizeof(int4) * std::max<long long>(h.npoints, 1));
    h.total = (int64_t)o;
    return h;
}

int lb_checkpoint_bytes(const lb_ctx* c, size_t* bytes)
{
    if (!c || !bytes) return LB_ERR_ARG;
    *bytes = (size_t)ckpt_layout(c, c->P.plain).total;
    return LB_OK;
}

int lb_checkpoint_save(lb_ctx* c, void* dst)
{
    if (!c) return LB_ERR_ARG;
    clear_stale_error();
    if (!dst || ((uintptr_t)dst % ALIGN) != 0) return fail(c, LB_ERR_ARG, "checkpoint buffer NULL or not 256-byte aligned");
    // the binning windows are part of the state once the registered sets have been binned
    if (total_points(c) > 0 && c->binned_gen != c->gen)
        return fail(c, LB_ERR_STATE, "checkpoint: step once after changing the point sets");
    c->ckpt = ckpt_layout(c, c->P.plain);
    const CkptHeader& h = c->ckpt;
    char* d = (char*)dst;
    hipStream_t s = c->stream;
    int r = LB_OK;
    auto cp = [&](int64_t off, const void* src, size_t n) {
        if (!r) r = hip_check(c, hipMemcpyAsync(d + off, src, n, hipMemcpyDefault, s), "checkpoint copy");
    };
    cp(0, &c->ckpt, sizeof(CkptHeader));
    cp(h.off_pop, c->pop(c->cur), (size_t)h.pop_bytes);
    cp(h.off_boxes, c->boxes(), sizeof(BoxDev) * c->p.nboxes);
    cp(h.off_tmax, c->tmax(), sizeof(float) * h.tiles);
    cp(h.off_smax, c->smax(), sizeof(unsigned) * SMAX_SLOTS * SMAX_STRIDE);
    cp(h.off_tctr, c->tctr() + c->cur, sizeof(unsigned long long));
    cp(h.off_nf, c->nf(), sizeof(int) * c->p.nboxes);
    if (h.npoints > 0) cp(h.off_win, c->win(), sizeof(int4) * h.npoints);
    return r ? r : check_async(c);
}

int lb_checkpoint_load(lb_ctx* c, const void* src)
{
    if (!c) return LB_ERR_ARG;
    clear_stale_error();
    if (!src || ((uintptr_t)src % ALIGN) != 0) return fail(c, LB_ERR_ARG, "checkpoint buffer NULL or not 256-byte aligned");
    CkptHeader h;
    int r = hip_check(c, hipStreamSynchronize(c->stream), "hipStreamSynchronize");
    if (!r) r = hip_check(c, hipMemcpy(&h, src, sizeof(h), hipMemcpyDefault), "checkpoint header");
    if (r) return r;
    if (memcmp(h.magic, CKPT_MAGIC, 8) != 0) return fail(c, LB_ERR_ARG, "not a checkpoint");
    // The tile that checkpoints of this context name or, where the caller named neither tile nor variant, one that the
    // library has chosen for lattices of some size (such contexts have written their own tile, and the rules have changed).
    // Only the per-tile maxima depend on the tile, and those matter for batches of FP16 boxes alone, whose default is the
    // plain tile.
    const Plan& P = c->P;
    int mx, my;
    march_tile(c->p.nx, c->p.ny, mx, my);
    const int tiles[][3] = {{P.plain[0], P.plain[1], P.plain[2]}, {64, 2, 2}, {64, 4, 1}, {32, 4, 2}, {16, 4, 4}, {128, 2, 1},
                            {128, 1, 2}, {256, 1, 1}, {mx, my, 1}};
    const bool any = c->p.tile_x <= 0 && c->p.variant == 0 && !(c->p.storage == LB_STORAGE_FP16 && c->p.nboxes > 1);
    const int* known = nullptr;
    CkptHeader want{};
    for (auto& t : tiles)
        if (!known && (any || &t == &tiles[0]) && h.tx == t[0] && h.ty == t[1] && h.tz == t[2]) {
            known = t;
            want = ckpt_layout(c, t);
        }
    if (!known || h.nx != want.nx || h.ny != want.ny || h.nz != want.nz || h.nboxes != want.nboxes ||
        h.storage != want.storage || h.collision != want.collision || h.tiles != want.tiles ||
        h.npoints != want.npoints || h.total != want.total)
        return fail(c, LB_ERR_ARG, "checkpoint of another lattice, tiling or point count");
    const char* d = (const char*)src;
    hipStream_t s = c->stream;
    auto cp = [&](void* dst, int64_t off, size_t n) {
        if (!r) r = hip_check(c, hipMemcpyAsync(dst, d + off, n, hipMemcpyDefault, s), "checkpoint copy");
    };
    cp(c->pop(c->cur), want.off_pop, (size_t)want.pop_bytes);
    cp(c->boxes(), want.off_boxes, sizeof(BoxDev) * c->p.nboxes);
    if (known == tiles[0]) cp(c->tmax(), want.off_tmax, sizeof(float) * want.tiles);
    cp(c->smax(), want.off_smax, sizeof(unsigned) * SMAX_SLOTS * SMAX_STRIDE);
    cp(c->tctr() + c->cur, want.off_tctr, sizeof(unsigned long long));
    cp(c->nf(), want.off_nf, sizeof(int) * c->p.nboxes);
    if (want.npoints > 0) cp(c->win(), want.off_win, sizeof(int4) * want.npoints);
    if (r) return r;
    // rebuild the tile lists at the next step with the saved windows: the lists flag raised,
    // no box choosing new windows unless one of its points has left its window
    launch_fill_u32(c->rebin(), 1, 1u, s);
    launch_fill_u32(c->rebox(), c->p.nboxes, 0u, s);
    c->binned_gen = c->gen;
    c->bins_valid = false;
    c->gc_valid = false;
    c->field_valid = false;
    c->steps = h.steps;
    return check_async(c);
}

int lb_destroy(lb_ctx* c)
{
    if (!c) return LB_ERR_ARG;
    (void)hipStreamSynchronize(c->stream);
    drop_graphs(c);
    for (auto e : c->ev) (void)hipEventDestroy(e);
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    delete c;
    return LB_OK;
}

const char* lb_status_string(int status)
{
    switch (status) {
    case LB_OK: return "ok";
    case LB_ERR_ARG: return "invalid argument";
    case LB_ERR_SIZE: return "size limit or workspace too small";
    case LB_ERR_HIP: return "HIP runtime error";
    case LB_ERR_NONFINITE: return "non-finite value detected";
    case LB_ERR_CAPACITY: return "capacity exceeded";
    case LB_ERR_STATE: return "invalid state";
    case LB_ERR_NEGATIVE_DENSITY: return "non-positive density";
    }
    return "unknown status";
}

const char* lb_last_error(const lb_ctx* c) { return c ? c->err.c_str() : g_err.c_str(); }

int64_t lb_steps_taken(const lb_ctx* c) { return c ? c->steps : -1; }

int lb_kernel_timing(lb_ctx* c, int enable)
{
    if (!c) return LB_ERR_ARG;
    c->timing = enable != 0;
    c->ev_used = 0;
    c->timed_ms = 0.0;
    c->timed_launches = 0;
    return LB_OK;
}

int lb_kernel_time(lb_ctx* c, double* total_ms, int64_t* launches)
{
    if (!c || !total_ms || !launches) return LB_ERR_ARG;
    int r = hip_check(c, hipStreamSynchronize(c->stream), "hipStreamSynchronize");
    if (r) return r;
    double ms = 0.0;
    for (size_t k = 0; k + 1 < c->ev_used; k += 2) {
        float t = 0.0f;
        r = hip_check(c, hipEventElapsedTime(&t, c->ev[k], c->ev[k + 1]), "hipEventElapsedTime");
        if (r) return r;
        ms += t;
    }
    *total_ms = ms;
    *launches = c->timed_launches;
    return LB_OK;
}

int lb_expand_multipoles(int64_t n, const int32_t* type, const double* center, const double* axis, const double* e1,
                         const double* strength, double sep, int64_t* n_out, double* pos_out, double* force_out)
{
    if (n < 0 || !n_out) return LB_ERR_ARG;
    if (n > 0 && (!type || !center || !axis || !strength || !pos_out || !force_out)) return LB_ERR_ARG;
    int64_t m = 0;
    auto put = [&](const double* R, double dr0, double dr1, double dr2, double f0, double f1, double f2) {
        pos_out[3 * m] = R[0] + dr0;
        pos_out[3 * m + 1] = R[1] + dr1;
        pos_out[3 * m + 2] = R[2] + dr2;
        force_out[3 * m] = f0;
        force_out[3 * m + 1] = f1;
        force_out[3 * m + 2] = f2;
        ++m;
    };
    const double h = 0.5 * sep;
    for (int64_t i = 0; i < n; ++i) {
        const double* R = center + 3 * i;
        const double* a = axis + 3 * i;
        const double s = strength[i];
        if (type[i] == 0) {
            put(R, 0, 0, 0, s * a[0], s * a[1], s * a[2]);
        } else if (type[i] == 1) {
            put(R, h * a[0], h * a[1], h * a[2], s * a[0], s * a[1], s * a[2]);
            put(R, -h * a[0], -h * a[1], -h * a[2], -s * a[0], -s * a[1], -s * a[2]);
        } else if (type[i] == 2) {
            if (!e1) return LB_ERR_ARG;
            const double* u = e1 + 3 * i;
            const double v[3] = {a[1] * u[2] - a[2] * u[1], a[2] * u[0] - a[0] * u[2], a[0] * u[1] - a[1] * u[0]};
            put(R, h * u[0], h * u[1], h * u[2], s * v[0], s * v[1], s * v[2]);
            put(R, -h * u[0], -h * u[1], -h * u[2], -s * v[0], -s * v[1], -s * v[2]);
            put(R, h * v[0], h * v[1], h * v[2], -s * u[0], -s * u[1], -s * u[2]);
            put(R, -h * v[0], -h * v[1], -h * v[2], s * u[0], s * u[1], s * u[2]);
        } else {
            return LB_ERR_ARG;
        }
    }
    *n_out = m;
    return LB_OK;
}

}  // extern "C"
