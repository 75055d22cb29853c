// Shared machinery of the cell-pair kernels (forces, adjoint, virial
// gradient): the 27-cell neighbourhood table, LDS staging in the home cell's
// frame, the dot-product screen into accept words and the walk over the
// accepted bits. See forces.hip for the design.
#pragma once

#include <type_traits>

#include "md_device.h"

namespace mdlj {
namespace {


// The 27-cell neighbourhood of a home cell as runs of memory-contiguous cells
// that share one image shift ("segments"): the three cells of an x-row are
// consecutive in the sorted arrays unless the row wraps around the box in x,
// so an interior home cell has 9 segments and a cell on an x face 27 (one per
// cell). Segments list the cells in the order dx, dy, dz (dx fastest) and
// tile the neighbourhood index range [0, total) in that order.
struct Neighbourhood {
    int total;       // atoms in the 27 cells
    int home_pos;    // neighbourhood index of the home cell's first atom
    int home_first;  // its sorted slot
    int n_home;
    int nseg;
    float origin[3];    // home-cell origin
    int seg_pos[27];    // neighbourhood index of the segment's first atom
    int seg_first[27];  // its sorted slot
    int seg_len[27];
    float sx[27], sy[27], sz[27];  // frame offset o - sh of the segment's cells
};

// The same table while it is built, in registers: lane l < 27 first holds
// neighbour cell l (HoodLoads: its CSR range, still in flight), then segment l
// (HoodSegs). The uniform fields are the same in every lane.
struct HoodLoads {
    int first = 0, next = 0;  // start[cj], start[cj + 1]
    float bx = 0.f, by = 0.f, bz = 0.f;
    int cell = 0;  // the home cell
    bool rows = false;
};

// Origin of cell c (local index) in the box. The frame offsets o +- L are
// formed from this rounded product; contraction is off wherever they are
// computed, since fma(i, s, -L) is not the exact o - L the frame relies on.
__device__ __forceinline__ void cell_origin(const SimArgs& a, int c, float& ox, float& oy, float& oz) {
#pragma clang fp contract(off)
    const int nc = a.nc;
    ox = static_cast<float>(c % nc) * a.s;
    oy = static_cast<float>((c / nc) % nc) * a.s;
    oz = static_cast<float>(c / (nc * nc)) * a.s;
}

// Uniform facts are spread over lanes (meta: lane 0 total, 1 home_pos,
// 2 home_first, 3 n_home, 4 nseg; org: lanes 0..2 the home-cell origin) so
// that a table held across the pair loops costs vector registers, not scalar
// ones.
struct HoodSegs {
    int pos = 0, first = 0, len = 0;
    float x = 0.f, y = 0.f, z = 0.f;
    int meta = 0;
    float org = 0.f;
    __device__ __forceinline__ int total() const { return __builtin_amdgcn_readlane(meta, 0); }
    __device__ __forceinline__ int home_pos() const { return __builtin_amdgcn_readlane(meta, 1); }
    __device__ __forceinline__ int home_first() const { return __builtin_amdgcn_readlane(meta, 2); }
    __device__ __forceinline__ int n_home() const { return __builtin_amdgcn_readlane(meta, 3); }
    __device__ __forceinline__ int nseg() const { return __builtin_amdgcn_readlane(meta, 4); }
    __device__ __forceinline__ float origin(int d) const {
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(org), d));
    }
};

// Issue the CSR loads of home cell c's 27 neighbours (lanes 0..26); nothing
// waits for them here.
__device__ __forceinline__ void hood_issue(const SimArgs& a, int c, HoodLoads& h) {
#pragma clang fp contract(off)
    const int lane = __lane_id();
    const int nc = a.nc;
    const int ix = c % nc, iy = (c / nc) % nc, iz = c / (nc * nc);
    float ox, oy, oz;
    cell_origin(a, c, ox, oy, oz);
    h.cell = c;
    h.rows = ix >= 1 && ix <= nc - 2;  // x-rows are contiguous and unshifted in x
    h.bx = ox;
    h.by = oy;
    h.bz = oz;
    if (lane < 27) {
        int jx = ix + lane % 3 - 1, jy = iy + (lane / 3) % 3 - 1, jz = iz + lane / 9 - 1;
        if (jx < 0) { jx += nc; h.bx = ox + a.box; } else if (jx >= nc) { jx -= nc; h.bx = ox - a.box; }
        if (jy < 0) { jy += nc; h.by = oy + a.box; } else if (jy >= nc) { jy -= nc; h.by = oy - a.box; }
        if (jz < 0) { jz += nc; h.bz = oz + a.box; } else if (jz >= nc) { jz -= nc; h.bz = oz - a.box; }
        const int cj = a.cbase + jx + nc * (jy + nc * jz);
        h.first = a.start[cj];
        h.next = a.start[cj + 1];
    }
}

__device__ __forceinline__ int lane_value(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float lane_value(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Segments of a neighbourhood from its CSR ranges (waits for hood_issue's loads).
__device__ __forceinline__ void hood_segments(const SimArgs& a, const HoodLoads& h, HoodSegs& g) {
    const int lane = __lane_id();
    const int cnt = lane < 27 ? h.next - h.first : 0;
    const int incl = wave_incl_scan(cnt);
    const int pos = incl - cnt;
    int nseg;
    if (h.rows) {
        // segment r = cells 3r .. 3r + 2, gathered from lanes 3r and 3r + 2
        const int src = lane < 9 ? 3 * lane : 0;
        const int end = __shfl(incl, lane < 9 ? 3 * lane + 2 : 0);
        g.pos = __shfl(pos, src);
        g.first = __shfl(h.first, src);
        g.len = end - g.pos;
        g.x = __shfl(h.bx, src);
        g.y = __shfl(h.by, src);
        g.z = __shfl(h.bz, src);
        nseg = 9;
    } else {
        g.pos = pos;
        g.first = h.first;
        g.len = cnt;
        g.x = h.bx;
        g.y = h.by;
        g.z = h.bz;
        nseg = 27;
    }
    const int total = __shfl(incl, 26), home_pos = __shfl(pos, 13), home_first = __shfl(h.first, 13),
              n_home = __shfl(cnt, 13);
    g.meta = lane == 0 ? total : lane == 1 ? home_pos : lane == 2 ? home_first : lane == 3 ? n_home : nseg;
    float ox, oy, oz;
    cell_origin(a, h.cell, ox, oy, oz);
    g.org = lane == 0 ? ox : lane == 1 ? oy : oz;
}

// Write the table to LDS (the caller synchronises before it is read).
__device__ __forceinline__ void hood_store(const HoodSegs& g, Neighbourhood& nb) {
    const int lane = __lane_id();
    if (lane < g.nseg()) {
        nb.seg_pos[lane] = g.pos;
        nb.seg_first[lane] = g.first;
        nb.seg_len[lane] = g.len;
        nb.sx[lane] = g.x;
        nb.sy[lane] = g.y;
        nb.sz[lane] = g.z;
    }
    if (lane == 0) nb.total = g.meta;
    if (lane == 1) nb.home_pos = g.meta;
    if (lane == 2) nb.home_first = g.meta;
    if (lane == 3) nb.n_home = g.meta;
    if (lane == 4) nb.nseg = g.meta;
    if (lane < 3) nb.origin[lane] = g.org;
}

// The segment table of nb back in registers (lane l holds segment l).
__device__ __forceinline__ HoodSegs hood_from_lds(const Neighbourhood& nb) {
    const int lane = __lane_id();
    HoodSegs g;
    const int nseg = nb.nseg;
    g.meta = lane == 0 ? nb.total : lane == 1 ? nb.home_pos : lane == 2 ? nb.home_first : lane == 3 ? nb.n_home : nseg;
    g.org = nb.origin[lane < 3 ? lane : 0];
    if (lane < nseg) {
        g.pos = nb.seg_pos[lane];
        g.first = nb.seg_first[lane];
        g.len = nb.seg_len[lane];
        g.x = nb.sx[lane];
        g.y = nb.sy[lane];
        g.z = nb.sz[lane];
    }
    return g;
}

// Fill the neighbourhood table of home cell c and synchronise.
__device__ __forceinline__ void load_neighbourhood(const SimArgs& a, int c, Neighbourhood& nb,
                                                   float& ox, float& oy, float& oz) {
    HoodLoads h;
    hood_issue(a, c, h);
    HoodSegs g;
    hood_segments(a, h, g);
    if (threadIdx.x < kWave) hood_store(g, nb);  // every wavefront holds the same table
    cell_origin(a, c, ox, oy, oz);
    __syncthreads();
}

// Staging of neighbourhood atoms [t0, t1) into the tile, frame-translated: a
// uniform cursor (segment sg, neighbourhood index g) walks the segments in
// chunks of at most one wavefront; a batch of B chunks has its loads in flight
// before its LDS stores. w carries |x|^2 in the frame (for the screen); with
// WITH_VEC the matching entries of a per-atom vector (sorted order) go to vtile
// as well.
struct StageCursor {
    int sg, g;
};

// An entry of the vector tile: all of a float4, or its first three components
// in 12 bytes.
struct Float3 {
    float x, y, z;
};
__device__ __forceinline__ void put(float4& d, const float4& v) { d = v; }
__device__ __forceinline__ void put(Float3& d, const float4& v) { d = Float3{v.x, v.y, v.z}; }

__device__ __forceinline__ StageCursor stage_begin(const HoodSegs& h, int t0) {
    StageCursor cur{0, t0};
    const int nseg = h.nseg();
    while (cur.sg < nseg && lane_value(h.pos, cur.sg) + lane_value(h.len, cur.sg) <= t0) ++cur.sg;
    return cur;
}

__device__ __forceinline__ bool stage_more(const HoodSegs& h, const StageCursor& cur, int t1) {
    return cur.g < t1 && cur.sg < h.nseg();
}

// One batch of chunks: per chunk the loaded atoms (one per lane). The chunk
// boundaries are not stored: the commit replays the cursor from the position
// the issue started at (a few scalar operations per chunk, and no scalar
// registers held between issue and commit).
template <int B, bool WITH_VEC>
struct StageBatch {
    float4 q[B], vq[B];
};

// Bounds of the chunk at the cursor: atoms [cur.g, ce) of segment cur.sg,
// whose first atom has neighbourhood index p and sorted slot first; advances
// the cursor past it.
__device__ __forceinline__ void stage_chunk(const HoodSegs& h, StageCursor& cur, int t1, int& p, int& first,
                                            int& base, int& cnt, int& seg) {
    p = lane_value(h.pos, cur.sg);
    const int end = p + lane_value(h.len, cur.sg);
    const int ce = min(min(cur.g + kWave, end), t1);
    first = lane_value(h.first, cur.sg);
    base = cur.g;
    cnt = ce - cur.g;
    seg = cur.sg;
    cur.g = ce;
    if (cur.g >= end) ++cur.sg;
}

template <int B, bool WITH_VEC>
__device__ __forceinline__ void stage_issue(const SimArgs& a, const HoodSegs& h, StageCursor& cur, int t1,
                                            StageBatch<B, WITH_VEC>& b, const float4* vec) {
    const int lane = __lane_id();
#pragma unroll
    for (int u = 0; u < B; ++u) {
        int slot = 0;  // lanes without an atom load slot 0 (always valid) and store nothing
        if (stage_more(h, cur, t1)) {
            int p, first, base, cnt, seg;
            stage_chunk(h, cur, t1, p, first, base, cnt, seg);
            if (lane < cnt) slot = first + (base - p) + lane;
        }
        b.q[u] = a.pos0[slot];
        if (WITH_VEC) b.vq[u] = vec[slot];
    }
}

// cur: the cursor stage_issue started from; on return, past the batch.
template <int B, bool WITH_VEC, class VT>
__device__ __forceinline__ void stage_commit(const HoodSegs& h, const StageBatch<B, WITH_VEC>& b, StageCursor& cur,
                                             int t0, int t1, float4* tile, VT* vtile) {
    const int lane = __lane_id();
#pragma unroll
    for (int u = 0; u < B; ++u) {
        if (stage_more(h, cur, t1)) {
            int p, first, base, cnt, seg;
            stage_chunk(h, cur, t1, p, first, base, cnt, seg);
            if (lane < cnt) {
                const int dst = base - t0 + lane;
                const float x = b.q[u].x - lane_value(h.x, seg);
                const float y = b.q[u].y - lane_value(h.y, seg);
                const float z = b.q[u].z - lane_value(h.z, seg);
                tile[dst] = make_float4(x, y, z, x * x + y * y + z * z);
                if (WITH_VEC) put(vtile[dst], b.vq[u]);
            }
        }
    }
}

// Staging of a whole neighbourhood in one pass (total <= tile capacity), with
// few instructions per segment: every lane of a wavefront loads and stores
// entry pos + lane of each segment whether or not the segment has that many
// atoms. Segments are written in order and tile [0, total) without gaps, so
// the surplus entries of segment k (indices pos_k + len_k .. pos_k + 63) are
// overwritten by a later segment, or fall into the padding after total,
// which the caller fills afterwards; loads past the arrays' end are clamped.
// Atoms 64 and up of a longer segment follow, masked, after every segment's
// first 64: no surplus store reaches that far (pos_j + 63 < pos_k + 64 for
// j < k). The tile needs room for total + 63 entries.
__device__ __forceinline__ void stage_whole(const SimArgs& a, const HoodSegs& h, float4* tile) {
    const int lane = __lane_id();
    const int nseg = h.nseg();  // 9 or 27
    const int last = a.natoms - 1;
    // 32-bit byte offsets from the array base (scalar base + vector offset loads)
    const char* pbase = reinterpret_cast<const char*>(a.pos0);
    for (int k0 = 0; k0 < nseg; k0 += 9) {
        float4 q[9];
#pragma unroll
        for (int u = 0; u < 9; ++u) {
            const uint32_t off = static_cast<uint32_t>(min(lane_value(h.first, k0 + u) + lane, last)) << 4;
            q[u] = *reinterpret_cast<const float4*>(pbase + off);
        }
#pragma unroll
        for (int u = 0; u < 9; ++u) {
            const int k = k0 + u;
            const float x = q[u].x - lane_value(h.x, k);
            const float y = q[u].y - lane_value(h.y, k);
            const float z = q[u].z - lane_value(h.z, k);
            tile[lane_value(h.pos, k) + lane] = make_float4(x, y, z, x * x + y * y + z * z);
            // store as each load arrives: nine results held for one burst of
            // stores would cost 36 more registers
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    uint64_t longs = __ballot(lane < nseg && h.len > kWave);
    while (longs) {
        const int k = __ffsll(static_cast<unsigned long long>(longs)) - 1;
        longs &= longs - 1;
        const int len = lane_value(h.len, k), first = lane_value(h.first, k), pos = lane_value(h.pos, k);
        const float sx = lane_value(h.x, k), sy = lane_value(h.y, k), sz = lane_value(h.z, k);
        for (int off = kWave + lane; off - lane < len; off += kWave) {
            if (off < len) {
                const float4 q = a.pos0[first + off];
                const float x = q.x - sx, y = q.y - sy, z = q.z - sz;
                tile[pos + off] = make_float4(x, y, z, x * x + y * y + z * z);
            }
        }
    }
}

// Neighbourhood of a home cell for the one-pass staging, in scalar registers:
// nine x-rows (dy, dz). In each row the cells that need no image shift in x are
// consecutive in the sorted arrays (piece A: three cells, or two for a home
// cell on an x face); on an x face the row's third cell wraps around the box
// (piece B, one cell, shifted by -+L in x). Pieces are staged in the order
// A0..A8, B0..B8, so the tile holds the neighbourhood without gaps. The CSR
// offsets come from scalar loads (the table is uniform, and the vector units
// are what bounds the cell passes: one vector load with its offsets moved to
// scalar registers lane by lane took about 60 vector instructions more per
// cell).
struct Pieces {
    int first[9];  // sorted slot of each piece's first atom
    int pos[10];   // tile index of each piece's first atom; pos[9]: of the one after the last
};

struct RowHood {
    Pieces a;
    int total, home_first, n_home, home_pos;
    int ix, iy, iz;
    float ox, oy, oz;    // home-cell origin
    float fxb;           // frame offset in x of the B pieces
    float fy[3], fz[3];  // frame offsets o - sh of the rows with dy, dz = -1, 0, 1
    bool face;
};

__device__ __forceinline__ int scalar_load(const int* p) {
    return *(const __attribute__((address_space(4))) int*)(reinterpret_cast<uintptr_t>(p));
}

// c / nc and c % nc for a cell or row index 0 <= c < nc^3 (uniform): the
// quotient from nc_magic = ceil(2^32 / nc) is at most one too large.
__device__ __forceinline__ int div_nc(const SimArgs& a, int c, int& rem) {
    int q = static_cast<int>(__umulhi(static_cast<uint32_t>(c), a.nc_magic));
    rem = c - q * a.nc;
    if (rem < 0) {
        --q;
        rem += a.nc;
    }
    return q;
}

// CSR offsets of cells [c0, c0 + n) of the nine x-rows around (iy, iz): the
// first atom of each row's piece and the one past its last.
__device__ __forceinline__ void piece_bounds(const SimArgs& a, const RowHood& r, int c0, int n, int (&first)[9],
                                             int (&end)[9]) {
    const int nc = a.nc;
    const int* base = a.start + a.cbase + c0;
    // (negative below the edge: the sign bit selects, in scalar instructions)
    const int by = r.iy - 1, bz = r.iz - 1, ey = r.iy + 1 - nc, ez = r.iz + 1 - nc;
    const int jy[3] = {by + (by >> 31 & nc), r.iy, ey + (ey >> 31 & nc)};
    const int jz[3] = {bz + (bz >> 31 & nc), r.iz, ez + (ez >> 31 & nc)};
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int* p = base + nc * (jy[k % 3] + nc * jz[k / 3]);
        first[k] = scalar_load(p);
        end[k] = scalar_load(p + n);
    }
}

// Tile indices of nine pieces from p on; returns the one after the last.
__device__ __forceinline__ int place_pieces(Pieces& t, const int (&end)[9], int p) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        t.pos[k] = p;
        p += end[k] - t.first[k];
    }
    t.pos[9] = p;
    return p;
}

__device__ __forceinline__ void row_hood(const SimArgs& a, int c_in, RowHood& r) {
#pragma clang fp contract(off)
    const int c = __builtin_amdgcn_readfirstlane(c_in);
    const int nc = a.nc;
    const int row = div_nc(a, c, r.ix);
    r.iz = div_nc(a, row, r.iy);
    r.face = r.ix == 0 || r.ix == nc - 1;
    // piece A: three cells, or two on a face
    const int a0 = r.ix == 0 ? 0 : r.ix - 1, n = r.face ? 2 : 3;
    int end[9];
    piece_bounds(a, r, a0, n, r.a.first, end);
    const int* home = a.start + a.cbase + c;
    r.home_first = scalar_load(home);
    r.n_home = scalar_load(home + 1) - r.home_first;
    const int by = r.iy - 1, bz = r.iz - 1, ey = r.iy + 1 - nc, ez = r.iz + 1 - nc;
    r.ox = static_cast<float>(r.ix) * a.s;
    r.oy = static_cast<float>(r.iy) * a.s;
    r.oz = static_cast<float>(r.iz) * a.s;
    // (the shifts are selected as scalars; adding zero is exact)
    const int L = __float_as_int(a.box);
    r.fxb = r.ox + __int_as_float(r.ix == 0 ? L : L ^ static_cast<int>(0x80000000u));
    r.fy[0] = r.oy + __int_as_float(by >> 31 & L);
    r.fy[1] = r.oy;
    r.fy[2] = r.oy - __int_as_float(~(ey >> 31) & L);
    r.fz[0] = r.oz + __int_as_float(bz >> 31 & L);
    r.fz[1] = r.oz;
    r.fz[2] = r.oz - __int_as_float(~(ez >> 31) & L);
    r.total = place_pieces(r.a, end, 0);
    r.home_pos = r.a.pos[4] + (r.home_first - r.a.first[4]);
    if (r.face) {
        int f[9], e[9];
        piece_bounds(a, r, r.ix == 0 ? nc - 1 : 0, 1, f, e);
#pragma unroll
        for (int k = 0; k < 9; ++k) r.total += e[k] - f[k];
    }
}

// Second tile of the staging functions below (SECOND): none; the untranslated
// positions (w = user index); the entries of vsrc, a per-atom vector in
// sorted order; or (SECOND_CODE, 32-bit entries) each atom's neighbour-list
// entry: its sorted slot with the code of the periodic image the frame
// translation applied. Any of them goes to raw at the same indices as the
// positions.
enum { SECOND_NONE = 0, SECOND_RAW = 1, SECOND_VEC = 2, SECOND_CODE = 3 };

// Image shift along one axis of a neighbour whose atoms are staged at
// x - f in the frame of origin o: the partner of the home atom is x + s L
// with s L = o - f, i.e. s = -1, 0 or +1.
__device__ __forceinline__ int image_shift(float o, float f, float box) {
    const float d = o - f;
    return d > 0.5f * box ? 1 : (d < -0.5f * box ? -1 : 0);
}

__device__ __forceinline__ uint32_t list_entry(int slot, int sx, int sy, int sz) {
    return static_cast<uint32_t>(slot) | (static_cast<uint32_t>((sx + 1) + 3 * (sy + 1) + 9 * (sz + 1)) << kSlotBits);
}

// The float4 at byte offset off of an array, by a bounds-checked buffer load
// (offsets past the end give zeros): no 64-bit address arithmetic, and no
// clamps. W: with the fourth component.
template <bool W>
__device__ __forceinline__ float4 load_slot(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    if (W) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(off), 0, 0);
        return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
    }
    const auto v = __builtin_amdgcn_raw_buffer_load_b96(r, static_cast<int>(off), 0, 0);
    return make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), 0.f);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t slot_buffer(const float4* p, int n) {
    // stride 0, n <= 2^27 16-byte slots, 32-bit data format
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float4*>(p), 0, static_cast<int>(static_cast<uint32_t>(n) << 4),
                                             0x00020000);
}

// Staging of nine pieces in one pass, with few instructions per piece: every
// lane loads and stores entry pos + lane of each piece whether or not it has
// that many atoms. Pieces are written in order and without gaps, so the
// surplus entries of a piece (up to pos + 63) are overwritten by a later one,
// or fall into the padding after the total, which the caller fills
// afterwards. Atoms 64 and up of a longer piece follow, masked, after every
// piece's first 64: no surplus store reaches that far. The tile needs room for
// total + 63 entries.
template <int SECOND, class VT>
__device__ __forceinline__ void stage_nine(const SimArgs& a, const RowHood& r, const Pieces& t, float fx, float4* tile,
                                           VT* raw, const float4* vsrc) {
    const int lane = lane_here();
    const uint32_t lane16 = 16u * static_cast<uint32_t>(lane);
    const __amdgpu_buffer_rsrc_t pos = slot_buffer(a.pos0, a.natoms);
    float4 q[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) q[k] = load_slot<SECOND == SECOND_RAW>(pos, lane16 + 16u * t.first[k]);
    uint32_t* codes = reinterpret_cast<uint32_t*>(raw);
    const int sx = SECOND == SECOND_CODE ? image_shift(r.ox, fx, a.box) : 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const float x = q[k].x - fx;
        const float y = q[k].y - r.fy[k % 3];
        const float z = q[k].z - r.fz[k / 3];
        tile[t.pos[k] + lane] = make_float4(x, y, z, x * x + y * y + z * z);
        if (SECOND == SECOND_RAW) put(raw[t.pos[k] + lane], q[k]);
        if (SECOND == SECOND_CODE)
            codes[t.pos[k] + lane] = list_entry(t.first[k] + lane, sx, image_shift(r.oy, r.fy[k % 3], a.box),
                                                image_shift(r.oz, r.fz[k / 3], a.box));
        // store as each load arrives: nine results held for one burst of
        // stores would cost 36 more registers
        __builtin_amdgcn_sched_barrier(0);
    }
    if (SECOND == SECOND_VEC) {  // a second round (the positions' registers are free again)
        const __amdgpu_buffer_rsrc_t vec = slot_buffer(vsrc, a.natoms);
#pragma unroll
        for (int k = 0; k < 9; ++k) q[k] = load_slot<std::is_same_v<VT, float4>>(vec, lane16 + 16u * t.first[k]);
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            put(raw[t.pos[k] + lane], q[k]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int len = t.pos[k + 1] - t.pos[k];
        if (len > kWave) {  // uniform; rare
            for (int off = kWave + lane; off - lane < len; off += kWave) {
                if (off < len) {
                    const float4 u = a.pos0[t.first[k] + off];
                    const float x = u.x - fx, y = u.y - r.fy[k % 3], z = u.z - r.fz[k / 3];
                    tile[t.pos[k] + off] = make_float4(x, y, z, x * x + y * y + z * z);
                    if (SECOND == SECOND_RAW) put(raw[t.pos[k] + off], u);
                    if (SECOND == SECOND_VEC) put(raw[t.pos[k] + off], vsrc[t.first[k] + off]);
                    if (SECOND == SECOND_CODE)
                        codes[t.pos[k] + off] = list_entry(t.first[k] + off, sx, image_shift(r.oy, r.fy[k % 3], a.box),
                                                           image_shift(r.oz, r.fz[k / 3], a.box));
                }
            }
        }
    }
}

// The whole neighbourhood of r in one pass (total <= tile capacity).
template <int SECOND = SECOND_NONE, class VT = float4>
__device__ __forceinline__ void stage_hood(const SimArgs& a, const RowHood& r, float4* tile, VT* raw = nullptr,
                                           const float4* vsrc = nullptr) {
    stage_nine<SECOND>(a, r, r.a, r.ox, tile, raw, vsrc);
    if (r.face) {  // the table of the B pieces is read again (two tables do not fit the scalar registers)
        Pieces b;
        int end[9];
        piece_bounds(a, r, r.ix == 0 ? a.nc - 1 : 0, 1, b.first, end);
        place_pieces(b, end, r.a.pos[9]);
        stage_nine<SECOND>(a, r, b, r.fxb, tile, raw, vsrc);
    }
}

// Stage neighbourhood atoms [t0, t0 + tn) of the table in nb (an interior
// cell's neighbourhood costs one global round trip).
// B chunks in flight per batch: 9, or with a vector 5 (the neighbour export:
// 70.4 us with three, 69.1 with five, N = 32,000 and tiles of 192 atoms) and 3
// for one of 12 bytes (the adjoint pass, whose registers are short: a seed at N =
// 100,003 and tiles of 192 atoms 224 us with three, 229 with five).
template <bool WITH_VEC = false, class VT = float4,
          int B = (!WITH_VEC ? 9 : std::is_same_v<VT, float4> ? 5 : 3)>
__device__ __forceinline__ void stage_tile(const SimArgs& a, const Neighbourhood& nb, float4* tile,
                                           int t0, int tn, const float4* vec = nullptr,
                                           VT* vtile = nullptr) {
    const HoodSegs h = hood_from_lds(nb);
    if (!WITH_VEC && t0 == 0 && tn == h.total()) {
        stage_whole(a, h, tile);
        return;
    }
    const int t1 = t0 + tn;
    StageCursor cur = stage_begin(h, t0);
    while (stage_more(h, cur, t1)) {
        StageBatch<B, WITH_VEC> b;
        StageCursor issue = cur;
        stage_issue(a, h, issue, t1, b, vec);
        stage_commit<B>(h, b, cur, t0, t1, tile, vtile);
    }
}

// Neighbour-list entries (list_entry) of neighbourhood atoms [t0, t0 + tn) of
// the table in nb, into codes[0, tn): the companion of stage_tile for the
// pass that writes the neighbour lists.
__device__ __forceinline__ void stage_codes(const SimArgs& a, const Neighbourhood& nb, uint32_t* codes, int t0,
                                            int tn) {
    const int lane = __lane_id();
    const int t1 = t0 + tn;
    const int nseg = nb.nseg;
    for (int k = 0; k < nseg; ++k) {  // uniform
        const int p = nb.seg_pos[k], len = nb.seg_len[k], first = nb.seg_first[k];
        const int lo = max(p, t0), hi = min(p + len, t1);
        const int sx = image_shift(nb.origin[0], nb.sx[k], a.box);
        const int sy = image_shift(nb.origin[1], nb.sy[k], a.box);
        const int sz = image_shift(nb.origin[2], nb.sz[k], a.box);
        for (int t = lo + lane; t < hi; t += kWave) codes[t - t0] = list_entry(first + (t - p), sx, sy, sz);
    }
}

// Cell-pair kernels. One wavefront per home cell; lane = (home atom h, slice s)
// with ns slices per atom: four for 11..16 atoms, else floor(64 / atoms) (at
// most 16), so that a cell of 15 atoms keeps 60 lanes busy and one of 20 atoms
// too. The staged candidates are screened in spans of up to 128 per lane (160
// or 192 with three slices, 256 with two):
//  screen : lane (h, s) gets the verdicts on candidates s, s + ns, s + 2 ns, ...
//           (slices interleave, so every slice samples the whole neighbourhood
//           and the slices of one atom find similar numbers of partners): the
//           sign of r^2 - bound = |x_j|^2 - 2 x_i.x_j - (bound - |x_i|^2)
//           against a bound a little above r_c^2, shifted into 32-bit accept
//           words. Cells of 11..32 atoms screen on the matrix cores, others on
//           the VALU.
//  pairs  : the home atom's own bit is cleared; every lane walks the set bits
//           of its words, recomputes the exact displacement, keeps
//           r^2 < r_c^2 and applies the kernel's pair operation (for the force
//           kernel: the truncated, shifted LJ force of section 2).
// Slice partials are summed in slice order, so the result does not depend on
// timing.
constexpr int kWords = 4;              // accept words per lane per span
constexpr int kGroups = 32 * kWords;   // candidates per lane of one walk
// Words of a walk of three slices (17..21 atoms a cell), where the words are not
// kept: four, 128 candidates a slice, leave a second walk of a few candidates to
// neighbourhoods of 27 x 15 atoms and more; five reach 27 x 17.7. Measured with
// four, five and six (one more select per candidate each): N = 4,000 838, 825 and
// 816 us for 50 steps, N = 108,000 (rho 1.0) 616, 586 and 593 for 20, N = 256,000
// 1042, 1027 and 1035 for 20.
constexpr int kLongWords = 5;
// The same where the words are kept, in records of four: six words (27 x 21
// atoms), as two records, where they hold all candidates of a cell, so that the
// records are those of spans of four words. With the records of a cell's lanes
// side by side, a step of pair lists (N = 131,072, 18.5 atoms a cell) 32.2 -> 28.1
// us, the recording one 43.6 -> 40.0.
constexpr int kKeptWords = 6;
constexpr int kMaxSlices = 16;
constexpr int kScreenUnroll = 4;
constexpr int kTilePad = kMaxSlices * (kScreenUnroll + 1);  // far-away entries after the staged atoms
constexpr int kMaxCellWaves = 4;                            // wavefronts per force workgroup
constexpr int kMfmaMinHome = 11, kMfmaMaxHome = 32;  // home atoms screened on the matrix cores

// LDS entries (float4) of a force workgroup: the tile and its padding, which
// the reduction reuses (five floats per lane and wavefront)
__host__ __device__ constexpr size_t cell_lds_entries(int tile_cap, int waves) {
    return static_cast<size_t>(tile_cap + kTilePad > 80 * waves ? tile_cap + kTilePad : 80 * waves);
}

// The lanes of a chunk of nh <= 64 home atoms: lane l holds atom h = l % hs and
// slice s = l / hs if act.
struct HomeLanes {
    int ns, hs;  // uniform
    int h, s;
    bool act;
};

__device__ __forceinline__ HomeLanes home_lanes(int nh) {
    const int lane = lane_here();
    HomeLanes v;
    if (nh >= kMfmaMinHome && nh <= 16) {  // uniform
        v.ns = 4;
        v.hs = 16;
        v.h = lane & 15;
        v.s = lane >> 4;
        v.act = v.h < nh;
    } else {
        // x / nh for x <= 64, nh <= 64: x ceil(2^16 / nh) / 2^16
        const uint32_t m = (65535u + nh) / static_cast<uint32_t>(nh);
        v.ns = min(kMaxSlices, static_cast<int>((64u * m) >> 16));
        v.hs = nh;
        v.s = static_cast<int>((static_cast<uint32_t>(lane) * m) >> 16);
        v.h = lane - v.s * nh;
        v.act = v.s < v.ns;
    }
    return v;
}

// The padding entries after the staged atoms: 100 cell sides away on every
// axis, so that no screen and no cutoff test accepts them (r_c is at most a
// cell side; the scaled values stay finite in 16 bits).
__device__ __forceinline__ float4 pad_entry(const SimArgs& a) {
    const float far = 100.0f * a.s;
    return make_float4(far, far, far, 3.0f * far * far);
}

// VALU screen of one span: word w, bit 31 - k holds the verdict on the lane's
// candidate 32 w + k, i.e. tile entry first + (32 w + k) * ns. groups is the
// largest candidate count of any slice (uniform); entries past the staged
// atoms are padding that never passes. NS > 0 fixes the stride at compile
// time (immediate LDS offsets); NS = 0 takes it from ns.
template <int NS>
__device__ __forceinline__ void screen_span(const float4* tile, int first, int ns_rt, int groups, float mx,
                                            float my, float mz, float thr_i, uint32_t (&wd)[kWords]) {
    const int ns = NS > 0 ? NS : ns_rt;
    const float4* cand = tile + first;
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
        uint32_t bits = 0;
        const int n = min(32, groups - 32 * w);  // uniform
        if (n > 0) {
            for (int k0 = 0; k0 < n; k0 += kScreenUnroll) {
#pragma unroll
                for (int u = 0; u < kScreenUnroll; ++u) {
                    const float4 q = cand[(32 * w + k0 + u) * ns];
                    // negative iff accepted; its sign bit is shifted into the word
                    const float d = fmaf(mx, q.x, fmaf(my, q.y, fmaf(mz, q.z, q.w - thr_i)));
                    bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(d), 31);
                }
            }
            const int done = (n + kScreenUnroll - 1) / kScreenUnroll * kScreenUnroll;
            if (done < 32) bits <<= (32 - done);
        }
        wd[w] = bits;
    }
}

// v of lane src (0 .. 63).
__device__ __forceinline__ int from_lane(int v, int src) { return __builtin_amdgcn_ds_bpermute(4 * src, v); }
__device__ __forceinline__ uint32_t from_lane(uint32_t v, int src) {
    return static_cast<uint32_t>(from_lane(static_cast<int>(v), src));
}
__device__ __forceinline__ float from_lane(float v, int src) { return __int_as_float(from_lane(__float_as_int(v), src)); }

// ---- screen on the matrix cores ------------------------------------------
// The screen runs as matrix products D = A B + C with A 16 candidates (rows),
// B 16 home atoms (columns) and D[j][i] = r^2 - bound, negative iff accepted.
// Lane l receives D[4 (l / 16) + q][l % 16], q = 0..3. Row 4 r + q is
// candidate 4 b + q of slice r for block b, so that lane (atom l % 16, r = l /
// 16) gets the verdicts on its slice's candidates in order: four sign bits per
// block, one v_alignbit each. The words are those of the VALU screen, and the
// same walk takes them.
//  * Four slices (11..16 atoms): r = 0..3 are the slices.
//  * Three slices (17..21 atoms): r = 0..2; r = 3 goes unused. The atoms past
//    16 take a second product, and the words move to the walk's lanes.
//  * Two slices (22..32 atoms): r % 2 is the slice, r / 2 the half of its
//    candidates, so that a lane walks two sets of words in turn.
// The products are 16-bit (16 x 16 x 16): a 32-bit 16 x 16 x 4 product takes
// 32 cycles in which the SIMD issues no vector instruction (time per wavefront
// = 4 x vector instructions + product cycles, measured), the 16-bit one runs
// beside them. In units of the cell side, with v = x_i and u = x_j - 1/2:
//   r^2 = |x_j|^2 - 2 v.u + (|v|^2 - v.1),
// so one K quarter (four values) holds (u, |x_j|^2) against (-2 v, 1) and the
// rest goes to C in 32 bits. Each of A's four lane groups holds the candidates
// of one of four blocks; a block's product takes them against a B that is zero
// in the other groups, so a candidate is read from LDS and rounded once. The
// bound is raised by more than the rounding can take off (screen16_bound on the
// host), so no pair that the exact test accepts is dropped; the few candidates
// accepted beyond r_c add exact zeros. A candidate that overflows 16 bits (256
// sides and more away: an atom that list or skin steps go on with after
// MD_DEV_SKIN; staged positions are always finite) makes 0 x inf in the other
// groups' products. This chip gives that NaN with its sign bit set, whatever the
// operands: the three verdicts beside it are accepts, which the exact test settles,
// and no pair is lost.
// Measured against the 32-bit product (11..16 atoms) and the VALU (17..32), with
// the walk's loads ahead of its arithmetic and the neighbourhood table in scalar
// registers; same results bit for bit, time of one step's force kernel:
// N = 2,048,000 (15 atoms a cell) 324 -> 292 us, N = 256,000 53.5 -> 49.9 us (per
// wavefront 504 matrix cycles for 804, waiting 1,270 cycles for 1,840),
// N = 4,000 16.1 -> 14.2 us, a gas of 14 a cell 44.0 -> 42.0 us (N = 256,000),
// 16 a cell and more (VALU before) 32.2 -> 30.1 us (N = 108,000). Both column
// groups of 17..32 atoms then in one pass over the candidates, each read and
// rounded once: whole runs another 3 to 5% (N = 4,000, 32,000 and 108,000, the
// gas), 3% at N = 256,000, whose cells hold 14.6 +- 2. Up to ten atoms
// keep six or more slices, whose candidates a product of sixteen columns would
// serve less than two thirds full: the VALU screen stays there by that reasoning
// (products for every cell size were timed only together with another order of
// the sums: N = 4,000 1.20x, a gas and dense states 0.95x).
typedef float mfma_f4 __attribute__((ext_vector_type(4)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ half4 as_half4(uint32_t lo, uint32_t hi) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(half4, (u2{lo, hi}));
}

// A group's operands in this lane: B of each block of four (zero outside the
// block's lane group) and C.
struct HomeOps {
    half4 b[4];
    float c;
};

// vx, vy, vz: position of the lane's column's home atom in units of the cell
// side (on: it has one).
__device__ __forceinline__ HomeOps home_ops(float vx, float vy, float vz, bool on, float bound16) {
    const int group = lane_here() >> 4;
    half4 p = {static_cast<_Float16>(-2.0f * vx), static_cast<_Float16>(-2.0f * vy), static_cast<_Float16>(-2.0f * vz),
               static_cast<_Float16>(1.0f)};
    if (!on) p = half4{0, 0, 0, static_cast<_Float16>(1.0f)};
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    const u2 w = __builtin_bit_cast(u2, p);
    HomeOps h;
#pragma unroll
    for (int k = 0; k < 4; ++k) h.b[k] = as_half4(group == k ? w[0] : 0u, group == k ? w[1] : 0u);
    h.c = on ? fmaf(vz, vz, fmaf(vy, vy, vx * vx)) - (vx + vy + vz) - bound16 : __builtin_huge_valf();
    return h;
}

// Screen nblk <= 8 WORDS blocks of four candidates per row group against GROUPS
// groups of columns: word w, bit 31 - k holds the verdict on the row group's
// candidate 32 w + k. base: this lane's candidate of the first four blocks; four
// blocks on, it lies 16 NS entries further (NS: slices).
template <int NS, int GROUPS, int WORDS>
__device__ __forceinline__ void screen_mfma(const float4* base, int nblk, float inv_s, const HomeOps (&h)[GROUPS],
                                            uint32_t (&wd)[GROUPS][WORDS]) {
    const float inv_s2 = inv_s * inv_s;
    auto four = [&](int g, uint32_t (&bits)[GROUPS]) {
        const float4 x = base[g * 16 * NS];
        // scaled and rounded, two values per register (in one block, with the
        // two wait states that a product needs after its operands' writes)
        uint32_t lo, hi;
        asm("v_fma_mixlo_f16 %0, %2, %6, -0.5 op_sel_hi:[0,0,0]\n\t"
            "v_fma_mixlo_f16 %1, %4, %6, -0.5 op_sel_hi:[0,0,0]\n\t"
            "v_fma_mixhi_f16 %0, %3, %6, -0.5 op_sel_hi:[0,0,0]\n\t"
            "v_fma_mixhi_f16 %1, %5, %7, 0 op_sel_hi:[0,0,0]\n\t"
            "s_nop 1"
            : "=&v"(lo), "=&v"(hi)
            : "v"(x.x), "v"(x.y), "v"(x.z), "v"(x.w), "s"(inv_s), "s"(inv_s2));
        const half4 a = as_half4(lo, hi);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int e = 0; e < GROUPS; ++e) {
                const mfma_f4 c = {h[e].c, h[e].c, h[e].c, h[e].c};
                const mfma_f4 d = __builtin_amdgcn_mfma_f32_16x16x16f16(a, h[e].b[u], c, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q) bits[e] = __builtin_amdgcn_alignbit(bits[e], __float_as_uint(d[q]), 31);
            }
        }
    };
    // straight-line code per word: all LDS offsets are immediates
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
        uint32_t bits[GROUPS] = {};
        if (nblk > 8 * w) {  // uniform
            four(2 * w, bits);
            if (nblk > 8 * w + 4) {  // may run past nblk: padding
                four(2 * w + 1, bits);
            } else {
#pragma unroll
                for (int e = 0; e < GROUPS; ++e) bits[e] <<= 16;
            }
        }
#pragma unroll
        for (int e = 0; e < GROUPS; ++e) wd[e][w] = bits[e];
    }
}

// Accept words of one span of a chunk of 11..16 (NS = 4), 17..21 (3) or 22..32 (2)
// home atoms, in the walk's layout. x, y, z: this lane's home atom (frame); g0:
// the span's first candidate of each slice, nblk: its blocks (per half with two
// slices). wd2: the words of the second half (two slices).
template <int NS, int WORDS>
__device__ __forceinline__ void screen_home(const SimArgs& a, const float4* tile, const HomeLanes& hl, int nh, int g0,
                                            int nblk, float x, float y, float z, float bound16,
                                            uint32_t (&wd)[WORDS], uint32_t (&wd2)[WORDS]) {
    const int lane = lane_here();
    const int q = lane & 3, r = (lane >> 2) & 3;  // this lane's row of A: candidate q of row group r
    const int gq = g0 + 4 * (lane >> 4) + q;      // ... of the block of its lane group
    const float vx = x * a.inv_s, vy = y * a.inv_s, vz = z * a.inv_s;
    if constexpr (NS == 4) {
        const HomeOps ops[1] = {home_ops(vx, vy, vz, hl.act, bound16)};
        uint32_t v[1][WORDS];
        screen_mfma<4>(tile + 4 * gq + r, nblk, a.inv_s, ops, v);
#pragma unroll
        for (int w = 0; w < WORDS; ++w) wd[w] = v[0][w];
    } else {
        const int part = NS == 2 ? r >> 1 : 0, slice = NS == 2 ? r & 1 : r;
        const float4* base = tile + NS * (gq + 4 * nblk * part) + slice;
        // atom h's words lie in lane h % 16 + 16 (row group of its slice and half)
        const int src = (hl.h & 15) + 16 * (hl.act ? hl.s : 0);
        const int e = lane & 15;  // lane e of the chunk holds atom e (slice 0)
        const HomeOps ops[2] = {home_ops(from_lane(vx, e), from_lane(vy, e), from_lane(vz, e), true, bound16),
                                home_ops(from_lane(vx, e + 16), from_lane(vy, e + 16), from_lane(vz, e + 16),
                                         e + 16 < nh, bound16)};
        uint32_t v[2][WORDS];
        screen_mfma<NS>(base, nblk, a.inv_s, ops, v);
        const bool second = hl.h >= 16;
#pragma unroll
        for (int w = 0; w < WORDS; ++w) {
            const uint32_t lo = from_lane(v[0][w], src), hi = from_lane(v[1][w], src);
            wd[w] = hl.act ? (second ? hi : lo) : 0;
            if (NS == 2) {
                const uint32_t lo2 = from_lane(v[0][w], src + 32), hi2 = from_lane(v[1][w], src + 32);
                wd2[w] = hl.act ? (second ? hi2 : lo2) : 0;
            }
        }
    }
}

// The 32-bit form for 11..16 atoms, for the pass that writes neighbour lists:
// what it accepts is what the lists hold, in their order, so its bound is the
// list radius without the 16-bit margin. A's rows are the candidates' (x, y, z,
// |x|^2), B's columns (-2 x_i, -2 y_i, -2 z_i, 1) and C = -(bound - |x_i|^2):
// lane l supplies B[l / 16][l % 16] and A[l % 16][l / 16].
__device__ __forceinline__ void screen_home32(const float4* tile, const HomeLanes& hl, int g0, int nblk, float x,
                                              float y, float z, float bound, uint32_t (&wd)[kWords]) {
    const int lane = lane_here();
    const int comp = lane >> 4;
    const int q = lane & 3, r = (lane >> 2) & 3;
    const float* base = reinterpret_cast<const float*>(tile + 4 * (g0 + q) + r) + comp;
    const float ai = fmaf(z, z, fmaf(y, y, x * x));
    const float bval = comp == 3 ? 1.0f : (hl.act ? -2.0f * (comp == 0 ? x : (comp == 1 ? y : z)) : 0.0f);
    const float cneg = hl.act ? -(bound - ai) : __builtin_huge_valf();
    const mfma_f4 c = {cneg, cneg, cneg, cneg};
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
        uint32_t bits = 0;
        const int nb = min(8, nblk - 8 * w);  // uniform
        if (nb > 0) {
            for (int b0 = 0; b0 < nb; b0 += 4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const mfma_f4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(base[(8 * w + b0 + u) * 64], bval, c, 0, 0, 0);
#pragma unroll
                    for (int k = 0; k < 4; ++k) bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(d[k]), 31);
                }
            }
            const int done = (nb + 3) / 4 * 4;  // blocks shifted in (the last four may run past nb)
            if (done < 8) bits <<= (32 - 4 * done);
        }
        wd[w] = bits;
    }
}

// Drop the verdicts past the first n candidates (uniform) of a lane's words.
template <int WORDS>
__device__ __forceinline__ void keep_first(int n, uint32_t (&wd)[WORDS]) {
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
        const int valid = n - 32 * w;
        wd[w] &= valid >= 32 ? ~0u : (valid <= 0 ? 0u : ~0u << (32 - valid));
    }
}

// The LDS byte address of a pointer into shared memory (the low half of its
// generic address), and a 16-byte load from such an address: walks that
// carry absolute LDS addresses read their candidates with no add.
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p));
}
typedef float lds_float4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 lds_load(uint32_t addr) {
    const lds_float4 v = *(const __attribute__((address_space(3))) lds_float4*)(static_cast<uintptr_t>(addr));
    return make_float4(v.x, v.y, v.z, v.w);
}
// Marks a loaded value as used here: its register then stays its own until
// this point. (A candidate's w is read by nobody; reused while the load is in
// flight, its register would make the wavefront wait for that load first.)
__device__ __forceinline__ void keep(float v) { asm volatile("" ::"v"(v)); }

// Largest value of any lane, uniform.
__device__ __forceinline__ int wave_max(int v) {
    auto ror = [](int x, auto ctrl) {
        return max(x, __builtin_amdgcn_update_dpp(x, x, decltype(ctrl)::value, 0xf, 0xf, false));
    };
    v = ror(v, std::integral_constant<int, 0x128>{});  // row_ror: 8, 4, 2, 1
    v = ror(v, std::integral_constant<int, 0x124>{});
    v = ror(v, std::integral_constant<int, 0x122>{});
    v = ror(v, std::integral_constant<int, 0x121>{});
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// The accepted candidates of one set of words in order, as LDS byte addresses:
// the word's candidate 0 lies at wb, candidates cstep bytes apart. A lane that
// has spent its bits gets pad, the address of the padding entry past every
// staged atom. The words rotate through registers (never indexed, which
// would put them in scratch memory); an exhausted word is replaced by the next
// one without a branch.
template <int WORDS>
struct BitWalk {
    uint32_t wb, wstep, cstep, pad, m, more[WORDS - 1];
    __device__ __forceinline__ uint32_t next() {
        const bool turn = (m == 0u);
        m = turn ? more[0] : m;
#pragma unroll
        for (int w = 0; w < WORDS - 2; ++w) more[w] = turn ? more[w + 1] : more[w];
        more[WORDS - 2] = turn ? 0u : more[WORDS - 2];
        wb += turn ? wstep : 0u;
        // all ones for a spent lane (m = 0): its shift clears no bit of m, and
        // its address (16 bits of ones times 16 to 256 bytes, which cannot
        // wrap) lies past the padding entry
        const uint32_t k = __builtin_clzg(m, -1);
        m &= ~(0x80000000u >> (k & 31u));
        uint32_t at;
        if (__builtin_constant_p(cstep) && cstep == 64) asm("v_mad_u32_u16 %0, %1, 64, %2" : "=v"(at) : "v"(k), "v"(wb));
        else asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(at) : "v"(k), "s"(cstep), "v"(wb));
        return min(at, pad);
    }
};

// Walk a lane's accept words, op(op.load(address)) for each candidate in
// order, two per step: the next two candidates' loads are issued before this
// step's arithmetic, so their latency is covered (two register sets take
// turns, which saves copying them). The trip count is the busiest lane's,
// reduced once, so the loop needs no test on the lanes.
template <int WORDS, class Op>
__device__ __forceinline__ void walk_bits(int ns, uint32_t wb0, uint32_t pad, const uint32_t (&wd)[WORDS], Op& op) {
    const uint32_t cstep = static_cast<uint32_t>(ns) * sizeof(float4);
    // a lane's steps: its bits, and one for each empty word before its last bit
    int steps = __builtin_popcount(wd[WORDS - 1]);
#pragma unroll
    for (int w = WORDS - 2; w >= 0; --w) steps += max(__builtin_popcount(wd[w]), min(steps, 1));
    const int trips = wave_max(steps);
    if (trips == 0) return;
    BitWalk<WORDS> b{wb0, 32u * cstep, cstep, pad, wd[0], {}};
#pragma unroll
    for (int w = 1; w < WORDS; ++w) b.more[w - 1] = wd[w];
    auto load = [&](typename Op::Entry (&q)[2]) {
        const uint32_t a0 = b.next(), a1 = b.next();
        q[0] = op.load(a0);
        q[1] = op.load(a1);
    };
    typename Op::Entry p[2], q[2];
    load(p);
    int sets = (trips + 1) >> 1;  // pairs of candidates still to take, p's among them
    for (; sets > 2; sets -= 2) {
        load(q);
        op(p[0]);
        op(p[1]);
        load(p);
        op(q[0]);
        op(q[1]);
    }
    if (sets == 2) load(q);
    op(p[0]);
    op(p[1]);
    if (sets == 2) {
        op(q[0]);
        op(q[1]);
    }
}

// Clear the screen bit of the home atom itself: g is its number among the
// words' candidates, if it lies in this lane's slice (own). The atoms of a cell
// are neighbours in the tile, so one or two words are touched: each is skipped
// unless some lane's bit lies in it.
template <int WORDS>
__device__ __forceinline__ void clear_self(int g, bool own, uint32_t (&wd)[WORDS]) {
    const uint32_t bit = 0x80000000u >> (g & 31);
    const int w = own ? g >> 5 : -1;
#pragma unroll
    for (int i = 0; i < WORDS; ++i)
        if (__any(w == i)) wd[i] &= w == i ? ~bit : ~0u;
}

// One pass over the tn staged candidates for a chunk of nh home atoms: fn(wd,
// first, n) for every set of accept words (this lane's n-th candidate is tile
// entry first + n ns; n: candidates of the largest slice in the set), with the
// home atom's own bit cleared. x, y, z: this lane's home atom in the frame;
// bound, bound16: the screens' bounds (EXACT: only the first is used);
// self_t: its tile index (may be outside); wv, nw: this wavefront takes the
// wv-th of nw contiguous ranges of the candidates. kept(wd, n): true if it
// supplied the words itself. LONG: the words of a walk with three slices (WHOLE:
// only where one walk takes all candidates, else kWords).
template <bool EXACT, int LONG, bool WHOLE, class Kept, class Fn>
__device__ __forceinline__ void for_each_words(const SimArgs& a, const float4* tile, int tn, const HomeLanes& hl,
                                               int nh, float x, float y, float z, float bound, float bound16,
                                               int self_t, int wv, int nw, Kept kept, Fn fn) {
    const int ns = hl.ns;
    const bool four = nh >= kMfmaMinHome && nh <= 16;
    const bool mat = nh >= kMfmaMinHome && nh <= (EXACT ? 16 : kMfmaMaxHome);  // uniform
    // this wavefront's candidates [g_lo, g_hi) of every slice, split at
    // multiples of the screen's step (so no verdict is taken twice): 16 with
    // four slices, else four
    int g_lo = 0, g_hi;
    if (four) {
        const int nblk = (tn + 15) / 16;
        g_hi = 4 * nblk;
        if (nw > 1) {
            const int q4 = (nblk + 3) >> 2;
            g_lo = 16 * ((q4 * wv) / nw);
            g_hi = min(g_hi, 16 * ((q4 * (wv + 1)) / nw));
        }
    } else {
        g_hi = (tn + ns - 1) / ns;
        if (nw > 1) {
            const int q4 = (g_hi + kScreenUnroll - 1) / kScreenUnroll;
            g_lo = kScreenUnroll * ((q4 * wv) / nw);
            g_hi = min(g_hi, kScreenUnroll * ((q4 * (wv + 1)) / nw));
        }
    }
    if (mat) {
        // spans of W words (a half of the span each with two slices)
        auto spans = [&](auto slices, auto words) {
            constexpr int NS = decltype(slices)::value, W = decltype(words)::value;
            constexpr int span = (NS == 2 ? 2 : 1) * 32 * W;
            for (int g0 = g_lo; g0 < g_hi; g0 += span) {
                const int groups = min(span, g_hi - g0);
                const int blocks = (groups + 3) >> 2;
                // per half: whole steps of the screen (four blocks), so the first
                // half does not run into the second
                const int nblk = NS == 2 ? ((blocks + 7) >> 3) << 2 : blocks;
                uint32_t wd[W], wd2[W];
                const int n1 = min(groups, 4 * nblk);
                const bool had = kept(wd, n1);
                if (!had) {
                    if constexpr (EXACT) screen_home32(tile, hl, g0, nblk, x, y, z, bound, wd);
                    else screen_home<NS>(a, tile, hl, nh, g0, nblk, x, y, z, bound16, wd, wd2);
                    if (nw > 1 && NS != 4) keep_first(n1, wd);  // the screen's last step may be the next range's
                    // the home atom's own slice and number, from its tile index
                    const int c = self_t - g0 * NS;
                    if (NS == 4) {
                        clear_self(c >> 2, (c & 3) == hl.s, wd);
                    } else if (c >= 0) {
                        const int g = c / NS;
                        const bool own = hl.act && c - g * NS == hl.s;
                        clear_self(g < 4 * nblk ? g : -1, own, wd);
                        if (NS == 2) clear_self(g - 4 * nblk, own, wd2);
                    }
                }
                const int first = g0 * NS + (hl.act ? hl.s : 0);
                fn(wd, first, n1);
                if (NS == 2 && groups > n1) {
                    if (!had) keep_first(groups - n1, wd2);  // likewise
                    kept(wd2, groups - n1);
                    fn(wd2, first + 4 * nblk * NS, groups - n1);
                }
            }
        };
        using std::integral_constant;
        constexpr integral_constant<int, kWords> words{};
        if constexpr (EXACT) {
            spans(integral_constant<int, 4>{}, words);
        } else {
            constexpr integral_constant<int, LONG> longer{};
            if (ns == 4) spans(integral_constant<int, 4>{}, words);
            else if (ns == 2) spans(integral_constant<int, 2>{}, words);
            else if (!WHOLE || g_hi - g_lo <= 32 * LONG) spans(integral_constant<int, 3>{}, longer);
            else spans(integral_constant<int, 3>{}, words);
        }
        return;
    }
    const float ai = fmaf(z, z, fmaf(y, y, x * x));
    // idle lanes get a bound no candidate can meet (q.w - thr_i = +inf)
    const float thr_i = hl.act ? bound - ai : -__builtin_huge_valf();
    const float mx = -2.0f * x, my = -2.0f * y, mz = -2.0f * z;
    for (int g0 = g_lo; g0 < g_hi; g0 += kGroups) {
        const int groups = min(kGroups, g_hi - g0);
        const int first = g0 * ns + (hl.act ? hl.s : 0);
        uint32_t wd[kWords];
        const bool had = kept(wd, groups);
        if (!had) {
            // (EXACT only: the others' cells of two and three slices took the matrix
            // screen. Strides fixed at compile time, the recording pass takes
            // 134.6 us for 135.8 at 21 atoms a cell, N = 256,000)
            if (EXACT && ns == 3) screen_span<3>(tile, first, ns, groups, mx, my, mz, thr_i, wd);
            else if (EXACT && ns == 2) screen_span<2>(tile, first, ns, groups, mx, my, mz, thr_i, wd);
            else if (ns == 6) screen_span<6>(tile, first, ns, groups, mx, my, mz, thr_i, wd);
            else screen_span<0>(tile, first, ns, groups, mx, my, mz, thr_i, wd);
            const int c = self_t - first;
            if (hl.act && c >= 0) {
                int d = ns;
                asm("" : "+s"(d));  // the reciprocal is made here, not ahead of every path
                const int g = c / d;
                clear_self(g, g * ns == c, wd);
            }
        }
        fn(wd, first, groups);
    }
}

}  // namespace
}  // namespace mdlj
