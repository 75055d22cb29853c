// Truncated, force-shifted Lennard-Jones forces over the cell list
// (section 2: force sum, f_LJ and the shifted f(r); section 3: partners in
// the home cell and its 26 neighbours).
//
// One wavefront per home cell. The wavefront stages the 27-cell neighbourhood
// into LDS once, translated into the home cell's frame so that the periodic
// image shift costs nothing per pair, and every lane then runs its home atom
// against the staged atoms. This replaces the paper's fixed array of 32
// placeholders per cell (section 3.1) by exact CSR ranges: no capacity limit
// and no virtual particles.
//
// Frame arithmetic: with home-cell origin o and image shift sh of a
// neighbour cell, the displacement is d = (x_i - o) - (x_j - (o - sh)).
// o - sh is exact in FP32 (o = 0 with sh = -L gives L; o >= L/2 with sh = +L
// is a Sterbenz subtraction), and both differences are of numbers within a
// few cells of each other, so d carries only the rounding of small numbers
// instead of ulp(L).
#include "cell_pairs.h"

namespace mdlj {

namespace {

template <bool ENERGY>
__device__ __forceinline__ float pair_force(const SimArgs& a, const float4 q, float xi, float yi, float zi,
                                            bool in, float& fx, float& fy, float& fz, float& u_loc, float& w_loc) {
    const float dx = xi - q.x, dy = yi - q.y, dz = zi - q.z;
    const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
    // the atom itself never reaches this point (its screen bit is cleared)
    const bool ok = in && (r2 < a.rc2);
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float ir2 = rinv * rinv;
    const float ir6 = ir2 * ir2 * ir2;
    // f(r) / r = 24 eps (2 sigma^12 r^-14 - sigma^6 r^-8) - f_LJ(r_c) / r
    float fr = fmaf(ir2 * ir6, fmaf(a.c12, ir6, -a.c6), -a.fc * rinv);
    fr = ok ? fr : 0.0f;
    fx = fmaf(fr, dx, fx);
    fy = fmaf(fr, dy, fy);
    fz = fmaf(fr, dz, fz);
    if (ENERGY) {
        const float r = r2 * rinv;
        const float u = ir6 * fmaf(a.e12, ir6, -a.e6) - a.uc + (r - a.rc) * a.fc;
        u_loc += ok ? u : 0.0f;
        w_loc += fr * r2;
    }
    return r2;
}

// Pair operation of the force walk (the padding entry fails the cutoff test).
template <bool ENERGY>
struct ForceOp {
    const SimArgs& a;
    float xi, yi, zi;
    float fx = 0.f, fy = 0.f, fz = 0.f, u_loc = 0.f, w_loc = 0.f;
    using Entry = float4;
    __device__ __forceinline__ Entry load(uint32_t addr) const { return lds_load(addr); }
    __device__ __forceinline__ void operator()(const Entry& q) {
        keep(q.w);
        pair_force<ENERGY>(a, q, xi, yi, zi, true, fx, fy, fz, u_loc, w_loc);
    }
};

// Pair operation of the pass that writes the neighbour lists: the force as
// ForceOp, and every candidate the walk visits (all within the list radius)
// appended to the home atom's list at this lane's next free entry.
template <bool ENERGY>
struct RecordOp {
    const SimArgs& a;
    uint32_t tile0;     // LDS address of the tile
    uint32_t pad;       // and of the padding entry after the staged atoms
    const char* cbase;  // list entries of the staged atoms (4 bytes each, at a quarter of the tile's offsets)
    float xi, yi, zi;
    uint32_t* row;      // the home atom's list: entry k at row[4 n (k / 4) + k % 4]
    int next;
    float fx = 0.f, fy = 0.f, fz = 0.f, u_loc = 0.f, w_loc = 0.f;
    struct Entry {
        float4 q;
        uint32_t code;
        bool live;  // not a spent lane
    };
    __device__ __forceinline__ Entry load(uint32_t addr) const {
        return Entry{lds_load(addr), *reinterpret_cast<const uint32_t*>(cbase + ((addr - tile0) >> 2)), addr < pad};
    }
    __device__ __forceinline__ void operator()(const Entry& e) {
        keep(e.q.w);
        pair_force<ENERGY>(a, e.q, xi, yi, zi, true, fx, fy, fz, u_loc, w_loc);
        if (e.live) {
            if (next < a.nlist_cap) row[4 * static_cast<size_t>(a.n) * (next >> 2) + (next & 3)] = e.code;
            ++next;
        }
    }
};

// Neighbour export from the force kernel's own staging, screen and walk: every
// pair the walk visits and the exact FP32 cutoff test of pair_force accepts
// appends the partner's user index to the home atom's row (row order follows
// the atomics, so it is unspecified).
struct ExportArgs {
    int* counts;
    int* idx;
    int max_nb;
};

struct ExportOp {
    const SimArgs& a;
    uint32_t tile0;     // LDS address of the tile
    const char* rbase;  // untranslated positions (user index in w) at the same offsets
    float xi, yi, zi;
    int idi;
    const ExportArgs& ex;
    bool over = false;
    struct Entry {
        float4 q;
        uint32_t off;  // from the tile
    };
    __device__ __forceinline__ Entry load(uint32_t addr) const { return Entry{lds_load(addr), addr - tile0}; }
    __device__ __forceinline__ void operator()(const Entry& e) {
        const float4 q = e.q;
        const float dx = xi - q.x, dy = yi - q.y, dz = zi - q.z;
        const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        if (r2 < a.rc2) {
            const int idj = __float_as_int(reinterpret_cast<const float4*>(rbase + e.off)->w);
            const int slot = atomicAdd(&ex.counts[idi], 1);
            if (slot < ex.max_nb) ex.idx[static_cast<size_t>(idi) * ex.max_nb + slot] = idj;
            else over = true;
        }
    }
};

// Kept accept words (pair lists as bitmasks): each four of a lane's words are one
// 16-byte record, and record j of a cell's 64 lanes is one run of 1 KB (a lane
// reads the records that its cell has, not the room for all); records past
// kListSpans are only counted (the cell then screens).
template <int WORDS>
__device__ __forceinline__ void keep_words(uint4* rows, int& n, int groups, const uint32_t (&wd)[WORDS]) {
    if (n < kListSpans) rows[n * kWave] = make_uint4(wd[0], wd[1], wd[2], wd[3]);
    ++n;
    if constexpr (WORDS > kWords) {
        static_assert(WORDS == kWords + 2, "two records");
        if (groups > kGroups) {  // uniform
            if (n < kListSpans) rows[n * kWave] = make_uint4(wd[4], wd[5], 0u, 0u);
            ++n;
        }
    }
}

// The kept words from record j on; record 0 and the two words of record 1 that
// a walk of six takes were requested before the staging (w0, w1). Bits past the
// set's groups candidates per lane are dropped, so a walk never leaves the staged
// span, whatever the words hold.
template <int WORDS>
__device__ __forceinline__ void kept_words(const uint4* rows, const uint4& w0, const uint2& w1, int& j, int groups,
                                           uint32_t (&wd)[WORDS]) {
    uint4 v = w0;
    if (j > 0) v = j < kListSpans ? rows[j * kWave] : make_uint4(0u, 0u, 0u, 0u);
    ++j;
    wd[0] = v.x;
    wd[1] = v.y;
    wd[2] = v.z;
    wd[3] = v.w;
    if constexpr (WORDS > kWords) {  // one walk takes all candidates: the records are 0 and 1
        const bool two = groups > kGroups;
        wd[4] = two ? w1.x : 0u;
        wd[5] = two ? w1.y : 0u;
        j += two ? 1 : 0;
    }
    keep_first(groups, wd);
}

// Forces on the atoms of home cell c (local index of the system described by
// a); one wavefront. Energy partials go to a.epart[3 (a.cbase + c) + 0..2].
// KICK completes the step's velocity (v += dt/(2m) F). DRIFT (with KICK) goes
// on into the next step's first half with the same force, as the drift kernel
// would (half kick, drift, wrap, cell, binning into the next rebuild's
// buckets) instead of writing vel0; force and vel0 are then left stale, since
// the rebuild replaces the sorted state.
// SKIN (with DRIFT): a step between rebuilds. The drift writes the unwrapped
// next position and velocity to pos2/vel2 (same sorted slot) instead of
// binning, and raises DEV_SKIN if the atom has left its cell's box by more
// than skin_half (cells of side r_c + skin then still hold every partner
// within r_c in the 27-cell neighbourhood, section 3.1) or, with pair lists,
// has moved more than disp_half since they were recorded (section 3).
// LIST 1: the screen takes the list radius (the cell side) as its bound and
// each lane's accept words are kept (one 16-byte record per four), and the
// home positions go to posref. LIST 2: a lane walks its kept words instead of
// screening: the same candidates in the same order plus some beyond r_c,
// which add exact zeros, so the sums are bitwise those of the screen. A cell
// with more than kListSpans records per lane, or more than one pass, screens as
// usual (and with the plain bound).
// LIST 3: the screen takes the list radius and every candidate it accepts
// goes to the home atom's neighbour list (raw: the staged atoms' list
// entries, 4 bytes each); the slices of an atom append in slice order per
// span, so an atom's list is written without atomics.
// EXPORT: no forces; the pairs the walk accepts go to the neighbour rows of
// ex (raw: a second tile of untranslated positions).
template <bool KICK, bool ENERGY, bool WRITE, bool DRIFT, bool SKIN = false, int LIST = 0, bool EXPORT = false,
          int MW = 1>
__device__ __forceinline__ void force_cell(const SimArgs& a, int c, float4* tile, Neighbourhood& nb, float* red,
                                           float4* raw = nullptr, const ExportArgs& ex = ExportArgs{}) {
    // The workgroup holds nw <= MW wavefronts (1, 2 or 4). All of them compute
    // the neighbourhood table; wavefront 0 stages the tile they share, each
    // screens and walks its own contiguous range of every pass's candidates,
    // and wavefront 0 adds their partials (waves in order, then slices) and
    // runs the epilogue. MW = 1 compiles the one-wavefront kernel.
    const int lane = __lane_id();
    const int wv = MW == 1 ? 0 : static_cast<int>(threadIdx.x) >> 6;  // uniform per wavefront
    const int nw = MW == 1 ? 1 : static_cast<int>(blockDim.x) >> 6;
    float ox, oy, oz;
    // a neighbourhood and home atoms that fit one pass are staged here, from a
    // table in scalar registers; others take the LDS table and stage in the
    // pass loop below
    RowHood rh;
    row_hood(a, c, rh);
    const bool rows = rh.total <= a.tile_cap && rh.n_home <= kWave;  // uniform
    int total = rh.total, home_first = rh.home_first, n_home = rh.n_home, home_pos = rh.home_pos;
    ox = rh.ox;
    oy = rh.oy;
    oz = rh.oz;
    if (rows) {
        if (wv == 0) stage_hood<EXPORT ? SECOND_RAW : (LIST == 3 ? SECOND_CODE : SECOND_NONE)>(a, rh, tile, raw);
    } else {
        load_neighbourhood(a, c, nb, ox, oy, oz);
        total = nb.total;
        home_first = nb.home_first;
        n_home = nb.n_home;
        home_pos = nb.home_pos;
    }

    double u_acc = 0.0, w_acc = 0.0, k_acc = 0.0;
    bool bad = false, skin_out = false, over = false;
    const size_t lrow = (static_cast<size_t>(a.cbase + c) * kWave + lane);  // this lane's kept words
    uint4* lwords = reinterpret_cast<uint4*>(a.plist) + static_cast<size_t>(a.cbase + c) * kListSpans * kWave + lane;
    const bool list_fits = total <= a.tile_cap && n_home <= kWave;          // uniform
    int n_rec = 0;  // LIST 1, 2: sets of words kept, taken
    int list_n = 0;
    uint4 lw0 = make_uint4(0u, 0u, 0u, 0u);  // LIST 2: the first records' words, requested before staging
    uint2 lw1 = make_uint2(0u, 0u);
    if (LIST == 2) {
        list_n = a.plist_n[lrow];
        lw0 = lwords[0];
        lw1 = *reinterpret_cast<const uint2*>(lwords + kWave);
    }
    const bool use_list = LIST == 2 && list_fits && __all(list_n <= kListSpans);
    for (int h0 = 0; h0 < n_home; h0 += kWave) {
        const int nh = min(kWave, n_home - h0);
        const HomeLanes hl = home_lanes(nh);
        const int ns = hl.ns, hstride = hl.hs, h = hl.h, s = hl.s;
        const bool act = hl.act;
        // the lane that finishes home atom h (in wavefront 0); in the
        // four-slice layout lanes nh..15 have s == 0 but no atom
        const bool lead = act && s == 0 && wv == 0;
        // (lanes without an atom read past the arrays' end: zeros)
        const uint32_t at = 16u * static_cast<uint32_t>(home_first + h0 + h), past = ~15u;
        const float4 pi = load_slot<true>(slot_buffer(a.pos0, a.natoms), act ? at : past);
        float4 vel = make_float4(0.f, 0.f, 0.f, 0.f);  // fetched now, used by the epilogue
        if (KICK || ENERGY) vel = load_slot<true>(slot_buffer(late_args().vel0, a.natoms), lead ? at : past);
        float4 pref = pi;  // LIST: position when the lists were recorded
        if (LIST == 2 && SKIN && lead) pref = a.posref[home_first + h0 + h];
        if ((LIST == 1 || LIST == 3) && lead) a.posref[home_first + h0 + h] = pi;
        const float xi = pi.x - ox, yi = pi.y - oy, zi = pi.z - oz;
        // the list radius only where the words are kept: other cells sum as the plain screen does
        const bool wide = (LIST == 1 && list_fits) || LIST == 3;
        const float bound = wide ? a.list_screen2 : a.screen2, bound16 = wide ? a.list_screen16 : a.screen16;
        float fx = 0.f, fy = 0.f, fz = 0.f, u_loc = 0.f, w_loc = 0.f;
        int lcount = 0;  // LIST 3: the atom's entries so far
        uint32_t* lrow_list = LIST == 3 ? a.nlist + 4 * static_cast<size_t>(home_first + h0 + h) : nullptr;
        for (int t0 = 0; t0 < total; t0 += a.tile_cap) {
            const int tn = min(a.tile_cap, total - t0);
            if (!rows) {
                __syncthreads();
                if (wv == 0) {
                    if (EXPORT) stage_tile<true>(a, nb, tile, t0, tn, a.pos0, raw);
                    else stage_tile(a, nb, tile, t0, tn);
                    if (LIST == 3) stage_codes(a, nb, reinterpret_cast<uint32_t*>(raw), t0, tn);
                }
            }
            if (wv == 0)
                for (int t = lane; t < kTilePad; t += kWave) tile[tn + t] = pad_entry(a);
            __syncthreads();
            const int self_t = home_pos + h0 + h - t0;  // the home atom's own tile index (may be outside)
            const uint32_t tile0 = lds_address(tile);
            const uint32_t pad = tile0 + static_cast<uint32_t>(tn) * sizeof(float4);
            auto kept = [&](auto& wd, int groups) {
                if constexpr (LIST == 2) {
                    if (use_list) kept_words(lwords, lw0, lw1, n_rec, groups, wd);
                    return use_list;
                }
                return false;
            };
            constexpr bool kKept = LIST == 1 || LIST == 2;
            constexpr int kLong = kKept ? kKeptWords : kLongWords;
            for_each_words<LIST == 3, kLong, kKept>(a, tile, tn, hl, nh, xi, yi, zi, bound, bound16, self_t, wv, nw,
                                                    kept, [&](auto& wd, int first, int groups) {
                if constexpr (LIST == 1) {
                    if (list_fits) keep_words(lwords, n_rec, groups, wd);
                }
                const uint32_t wb0 = tile0 + static_cast<uint32_t>(first) * sizeof(float4);
                if constexpr (LIST == 3) {
                    // this lane's first entry for the accepted candidates
                    // (after those of the atom's lower slices)
                    const int cnt = __popc(wd[0]) + __popc(wd[1]) + __popc(wd[2]) + __popc(wd[3]);
                    int pre = 0, tot = 0;
                    for (int q = 0; q < ns; ++q) {
                        const int v = __shfl(cnt, h + q * hstride);
                        pre += q < s ? v : 0;
                        tot += v;
                    }
                    RecordOp<ENERGY> op{a,  tile0, pad, reinterpret_cast<const char*>(raw), xi, yi, zi, lrow_list,
                                        lcount + pre, fx, fy, fz, u_loc, w_loc};
                    lcount += tot;
                    walk_bits(ns, wb0, pad, wd, op);
                    fx = op.fx;
                    fy = op.fy;
                    fz = op.fz;
                    u_loc = op.u_loc;
                    w_loc = op.w_loc;
                } else if constexpr (EXPORT) {
                    ExportOp op{a, tile0, reinterpret_cast<const char*>(raw), xi, yi, zi, __float_as_int(pi.w), ex};
                    walk_bits(ns, wb0, pad, wd, op);
                    over = over || op.over;
                } else {
                    ForceOp<ENERGY> op{a, xi, yi, zi, fx, fy, fz, u_loc, w_loc};
                    if (ns == 4) walk_bits(4, wb0, pad, wd, op);
                    else walk_bits(ns, wb0, pad, wd, op);
                    fx = op.fx;
                    fy = op.fy;
                    fz = op.fz;
                    u_loc = op.u_loc;
                    w_loc = op.w_loc;
                }
            });
        }
        if (EXPORT) continue;
        // sum the slice partials of each home atom in slice order (red aliases the
        // tile: every lane has finished its walk at this barrier)
        __syncthreads();
        float* mine = red + 5 * kWave * wv;  // this wavefront's partials
        mine[0 * kWave + lane] = fx;
        mine[1 * kWave + lane] = fy;
        mine[2 * kWave + lane] = fz;
        if (ENERGY) {
            mine[3 * kWave + lane] = u_loc;
            mine[4 * kWave + lane] = w_loc;
        }
        __syncthreads();
        const int k = home_first + h0 + h;
        // the arguments of the epilogue, with this system's geometry
        SimArgs l = late_args();
        l.nc = a.nc;
        l.cbase = a.cbase;
        l.box = a.box;
        l.inv_box = a.inv_box;
        l.s = a.s;
        l.inv_s = a.inv_s;
        int c_next = -1;  // DRIFT: the home atom's next cell, -1 on lanes without one
        float4 p_next = pi, v_next = make_float4(0.f, 0.f, 0.f, 0.f);
        if (lead) {
            if (LIST == 3) {  // the atom's list length (the entries past the capacity were not kept)
                l.ncount[k] = min(lcount, l.nlist_cap);
                if (lcount > l.nlist_cap) over = true;
            }
            float gx = 0.f, gy = 0.f, gz = 0.f, gu = 0.f, gw = 0.f;
            for (int w = 0; w < nw; ++w) {
                const float* part = red + 5 * kWave * w + h;
                auto add = [&](const float* p) {
                    gx += p[0 * kWave];
                    gy += p[1 * kWave];
                    gz += p[2 * kWave];
                    if (ENERGY) {
                        gu += p[3 * kWave];
                        gw += p[4 * kWave];
                    }
                };
                if (ns == 4) {  // uniform: offsets are immediates, all reads in flight
#pragma unroll
                    for (int q = 0; q < 4; ++q) add(part + q * 16);
                } else {
                    for (int q = 0; q < ns; ++q) add(part + q * hstride);
                }
            }
            if (!finite3(gx, gy, gz)) bad = true;
            if (WRITE) l.force[k] = make_float4(gx, gy, gz, 0.f);
            if (KICK || ENERGY) {
                float4 v = vel;
                if (KICK) {
                    v.x += l.hdt_m * gx;
                    v.y += l.hdt_m * gy;
                    v.z += l.hdt_m * gz;
                    if (!DRIFT) l.vel0[k] = v;
                }
                if (ENERGY) {
                    u_acc += static_cast<double>(gu);
                    w_acc += static_cast<double>(gw);
                    k_acc += static_cast<double>(l.half_m) * (static_cast<double>(v.x) * v.x +
                                                              static_cast<double>(v.y) * v.y +
                                                              static_cast<double>(v.z) * v.z);
                }
                if (DRIFT) {
                    v_next = v;
                    if (SKIN) {
                        half_kick_drift_unwrapped(l, p_next, v_next, gx, gy, gz);
                        l.pos2[k] = p_next;
                        l.vel2[k] = v_next;
                        if (LIST != 0) {
                            const float ex = p_next.x - pref.x, ey = p_next.y - pref.y, ez = p_next.z - pref.z;
                            if (ex * ex + ey * ey + ez * ez > l.disp_half * l.disp_half) skin_out = true;
                        } else {
                            const float ex = fmaxf(fmaxf(ox - p_next.x, p_next.x - (ox + l.s)), 0.f);
                            const float ey = fmaxf(fmaxf(oy - p_next.y, p_next.y - (oy + l.s)), 0.f);
                            const float ez = fmaxf(fmaxf(oz - p_next.z, p_next.z - (oz + l.s)), 0.f);
                            if (ex * ex + ey * ey + ez * ez > l.skin_half * l.skin_half) skin_out = true;
                        }
                    } else {
                        c_next = half_kick_drift(l, p_next, v_next, gx, gy, gz);
                    }
                }
            }
        }
        if (DRIFT && !SKIN && wv == 0) bin_atom(l, p_next, v_next, c_next);  // all lanes of wavefront 0
    }
    const SimArgs l = late_args();
    if (LIST == 1) l.plist_n[lrow] = list_fits ? n_rec : kListSpans + 1;  // kept words of several passes are not used
    if ((EXPORT || LIST == 3) && over) atomicOr(&l.hdr[HDR_ERROR], DEV_NB_OVERFLOW);
    if (bad) atomicOr(&l.hdr[HDR_ERROR], DEV_NONFINITE);
    if (SKIN && skin_out) atomicOr(&l.hdr[HDR_ERROR], DEV_SKIN);
    if (ENERGY) {
        u_acc = wave_sum(u_acc);
        w_acc = wave_sum(w_acc);
        k_acc = wave_sum(k_acc);
        if (threadIdx.x == 0) {
            double* e = l.epart + 3 * static_cast<size_t>(a.cbase + c);
            e[0] = u_acc;
            e[1] = w_acc;
            e[2] = k_acc;
        }
    }
}

template <bool KICK, bool ENERGY, bool WRITE, bool DRIFT, int MW>
__global__ void __launch_bounds__(MW * kWave) k_forces(SimArgs a, bool from_step) {
    if (from_step) {
        if (scalar_load(a.hdr + HDR_ERROR) & DEV_ORDER) return;
    } else if (!state_ok(a, false)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&a.hdr[HDR_ERROR], DEV_ORDER);
        return;
    }
    extern __shared__ float4 tile[];  // cell_lds_entries(a.tile_cap, a.waves) entries
    __shared__ Neighbourhood nb;
    // the slice reduction reuses the tile (320 floats per wavefront)
    force_cell<KICK, ENERGY, WRITE, DRIFT, false, 0, false, MW>(a, xcd_block_order(blockIdx.x, a.ncells), tile, nb,
                                                                reinterpret_cast<float*>(tile));
    if (WRITE && blockIdx.x == 0 && threadIdx.x == 0) a.hdr[HDR_STATE] = STATE_FORCES;
}

// A step between rebuilds (md_step_every): forces, kick, and the next step's
// half kick and drift into pos2/vel2.
template <bool ENERGY, int MW>
__global__ void __launch_bounds__(MW * kWave) k_forces_skin(SimArgs a) {
    if (scalar_load(a.hdr + HDR_ERROR) & DEV_ORDER) return;
    extern __shared__ float4 tile[];
    __shared__ Neighbourhood nb;
    force_cell<true, ENERGY, false, true, true, 0, false, MW>(a, xcd_block_order(blockIdx.x, a.ncells), tile, nb,
                                                              reinterpret_cast<float*>(tile));
}

// Pair-list steps: RECORD right after a rebuild, else walk the recorded lists;
// BIN: the drift bins for the next rebuild, else it goes to pos2/vel2.
template <bool ENERGY, bool RECORD, bool BIN>
__global__ void __launch_bounds__(kWave) k_forces_list(SimArgs a) {
    if (scalar_load(a.hdr + HDR_ERROR) & DEV_ORDER) return;
    extern __shared__ float4 tile[];
    __shared__ Neighbourhood nb;
    force_cell<true, ENERGY, false, true, !BIN, RECORD ? 1 : 2>(a, xcd_block_order(blockIdx.x, a.ncells), tile, nb,
                                                                reinterpret_cast<float*>(tile));
}

// md_step_nlist, right after a rebuild: forces, kick and the next drift as
// k_forces_list, and every atom's neighbour list within the list radius.
template <bool ENERGY, bool BIN>
__global__ void __launch_bounds__(kWave) k_forces_record(SimArgs a) {
    if (scalar_load(a.hdr + HDR_ERROR) & DEV_ORDER) return;
    extern __shared__ float4 tile[];  // a.tile_cap + kTilePad positions, then as many 4-byte list entries
    __shared__ Neighbourhood nb;
    force_cell<true, ENERGY, false, true, !BIN, 3>(a, xcd_block_order(blockIdx.x, a.ncells), tile, nb,
                                                   reinterpret_cast<float*>(tile), tile + (a.tile_cap + kTilePad));
}

// md_step_nlist between rebuilds: kListLanes lanes per atom (sorted slots,
// in the XCD order of the cell kernels) walk the atom's neighbour list, lane
// s taking entry groups s, s + kListLanes, ...: partner j at x_j + s L (s
// from the entry's image code), the truncated, shifted force of section 2
// for r < r_c; the lanes' partials are added in a fixed order, then the
// first wavefront applies the kick and the next half kick and drift as the
// cell passes do (BIN: wrap and bin for the next rebuild; else
// unwrapped into pos2/vel2 with the displacement check against the
// positions the lists were written at). The displacement is formed as
// (x_i - max(sL, 0)) - (x_j + min(sL, 0)): an image shift is taken off the
// coordinate that lies within a cell of the far box face, where the
// subtraction is exact, so d carries only the rounding of small numbers (as
// the frame translation of the cell passes does).
constexpr int kListBlock = 256;
constexpr int kListLanes = 4;
constexpr int kListAtoms = kListBlock / kListLanes;

template <bool BIN>
__global__ void __launch_bounds__(kListBlock) k_nlist_forces(SimArgs a) {
    if (a.hdr[HDR_ERROR] & DEV_ORDER) return;
    // max(s L, 0) and min(s L, 0) of each image code (the five code bits
    // index 32 entries; codes past 26 never occur and shift by nothing)
    constexpr int kCenter = 13;  // (0, 0, 0)
    __shared__ float4 shp[32], shm[32];
    if (threadIdx.x < 32) {
        const int code = threadIdx.x < 27 ? threadIdx.x : kCenter;
        const float sx = static_cast<float>(code % 3 - 1) * a.box, sy = static_cast<float>((code / 3) % 3 - 1) * a.box,
                    sz = static_cast<float>(code / 9 - 1) * a.box;
        shp[threadIdx.x] = make_float4(fmaxf(sx, 0.f), fmaxf(sy, 0.f), fmaxf(sz, 0.f), 0.f);
        shm[threadIdx.x] = make_float4(fminf(sx, 0.f), fminf(sy, 0.f), fminf(sz, 0.f), 0.f);
    }
    __syncthreads();
    const int lane = __lane_id();
    const char* pbase = reinterpret_cast<const char*>(a.pos0);
    const int last = a.n - 1;
    const int sl = threadIdx.x % kListLanes;
    const int i = xcd_block_order(blockIdx.x, gridDim.x) * kListAtoms + static_cast<int>(threadIdx.x) / kListLanes;
    const bool valid = i < a.n;
    float4 pi = make_float4(0.f, 0.f, 0.f, 0.f);
    int cnt = 0;
    if (valid) {
        pi = a.pos0[i];
        cnt = min(max(a.ncount[i], 0), a.nlist_cap);
    }
    // entries 4 g .. 4 g + 3 of every atom are one uint4, and the atoms' uint4
    // of one group are consecutive
    const uint4* col = reinterpret_cast<const uint4*>(a.nlist) + (valid ? i : 0);
    float fx = 0.f, fy = 0.f, fz = 0.f, u_loc = 0.f, w_loc = 0.f;
    // the capacity is a multiple of 4: whole uint4 loads. Each group's four
    // partners are requested together and the next group's entries are in
    // flight during this group's arithmetic; image shifts (pairs across a box
    // face, rare) are applied once all four partners have arrived.
    int g = sl;
    uint4 e4 = 4 * g < cnt ? col[static_cast<size_t>(a.n) * g] : make_uint4(0u, 0u, 0u, 0u);
    for (; 4 * g < cnt; g += kListLanes) {
        const uint32_t e[4] = {e4.x, e4.y, e4.z, e4.w};
        float4 q[4];
        int code[4];
        bool in[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            in[u] = 4 * g + u < cnt;
            // entries past the count are not this atom's: read the atom itself, masked
            const uint32_t ej = in[u] ? e[u] : (static_cast<uint32_t>(i) | (kCenter << kSlotBits));
            const uint32_t off = static_cast<uint32_t>(min(static_cast<int>(ej & kSlotMask), last)) << 4;
            q[u] = *reinterpret_cast<const float4*>(pbase + off);
            code[u] = static_cast<int>(ej >> kSlotBits);
        }
        const int gn = g + kListLanes;
        if (4 * gn < cnt) e4 = col[static_cast<size_t>(a.n) * gn];
        float xs[4], ys[4], zs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            xs[u] = pi.x;
            ys[u] = pi.y;
            zs[u] = pi.z;
        }
        const bool shifted = (code[0] != kCenter) | (code[1] != kCenter) | (code[2] != kCenter) | (code[3] != kCenter);
        if (__any(shifted)) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float4 hp = shp[code[u]], hm = shm[code[u]];
                q[u].x += hm.x;
                q[u].y += hm.y;
                q[u].z += hm.z;
                xs[u] -= hp.x;
                ys[u] -= hp.y;
                zs[u] -= hp.z;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) pair_force<false>(a, q[u], xs[u], ys[u], zs[u], in[u], fx, fy, fz, u_loc, w_loc);
    }
    // the atom's lanes are consecutive: sum (s0 + s1) + (s2 + s3)
#pragma unroll
    for (int off = 1; off < kListLanes; off <<= 1) {
        fx += __shfl_xor(fx, off);
        fy += __shfl_xor(fy, off);
        fz += __shfl_xor(fz, off);
    }
    // the epilogue on one lane per atom, all of them in the first wavefront: its
    // 64 consecutive atoms are the binning's runs, and their loads and stores
    // whole lines. With 16 atoms in each wavefront (four times the atomics and
    // their round trips) the pass took, at N = 256,000, 23.2 us with binning for
    // 14.8 and 12.4 without for 11.5 (14 entries an atom), 42.1 for 36.8 and 35.9
    // for 35.0 (88 entries, bound by the gathers' address units).
    __shared__ float fsum[3][kListAtoms];
    if (sl == 0) {
        const int l = static_cast<int>(threadIdx.x) / kListLanes;
        fsum[0][l] = fx;
        fsum[1][l] = fy;
        fsum[2][l] = fz;
    }
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    const float gx = fsum[0][lane], gy = fsum[1][lane], gz = fsum[2][lane];
    const int ia = xcd_block_order(blockIdx.x, gridDim.x) * kListAtoms + lane;
    const bool own = ia < a.n;
    bool bad = false;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f), p_next = v;
    if (own) {
        p_next = a.pos0[ia];
        v = a.vel0[ia];
        bad = !finite3(gx, gy, gz);
        v.x += a.hdt_m * gx;
        v.y += a.hdt_m * gy;
        v.z += a.hdt_m * gz;
    }
    if (BIN) {
        int c_next = -1;
        if (own) c_next = half_kick_drift(a, p_next, v, gx, gy, gz);
        bin_atom(a, p_next, v, c_next);  // all lanes
    } else if (own) {
        const float4 pref = a.posref[ia];
        half_kick_drift_unwrapped(a, p_next, v, gx, gy, gz);
        a.pos2[ia] = p_next;
        a.vel2[ia] = v;
        const float ex = p_next.x - pref.x, ey = p_next.y - pref.y, ez = p_next.z - pref.z;
        if (ex * ex + ey * ey + ez * ez > a.disp_half * a.disp_half) atomicOr(&a.hdr[HDR_ERROR], DEV_SKIN);
    }
    if (bad) atomicOr(&a.hdr[HDR_ERROR], DEV_NONFINITE);
}

// Batched forces: one workgroup per listed cell (global cell indices of the
// replicas of one tile class, XCD-ordered); the replica's own geometry comes
// from its descriptor.
template <bool KICK, bool ENERGY, bool WRITE, bool DRIFT, int MW>
__global__ void __launch_bounds__(MW * kWave)
    k_batch_forces(SimArgs base, const Replica* __restrict__ reps, const int* __restrict__ cell_rep,
                   const int* __restrict__ cells, int ncl) {
    if (base.hdr[HDR_ERROR] & DEV_ORDER) return;
    extern __shared__ float4 tile[];  // cell_lds_entries of the class's largest tile_cap
    __shared__ Neighbourhood nb;
    float* red = reinterpret_cast<float*>(tile);  // slice reduction, as in k_forces
    const int gc = cells[xcd_block_order(blockIdx.x, ncl)];
    const SimArgs a = replica_view(base, reps[cell_rep[gc]]);
    force_cell<KICK, ENERGY, WRITE, DRIFT, false, 0, false, MW>(a, gc - a.cbase, tile, nb, red);
    if (WRITE && blockIdx.x == 0 && threadIdx.x == 0) base.hdr[HDR_STATE] = STATE_FORCES;
}

// Fixed-order final sum of the per-block partials: U = 1/2 sum, W = 1/2 sum
// (every pair is visited from both sides), K as is.
constexpr int kRedBlock = 256;    // batched finals: one workgroup per replica
constexpr int kFinalBlock = 1024; // the single system's final sum
constexpr int kRedUnroll = 8;

// Lane t's running sums of the (U, W, K) partials of blocks t, t + BLOCK,
// t + 2 BLOCK, ... in that order; the loads of kRedUnroll blocks are issued
// before their sums, so the sequential order costs one round trip per
// BLOCK * kRedUnroll blocks.
template <int BLOCK>
__device__ __forceinline__ void sum_partials(const double* __restrict__ e, int n, int t, double& u, double& w,
                                             double& k) {
    for (int b0 = t; b0 < n; b0 += BLOCK * kRedUnroll) {
        double pu[kRedUnroll], pw[kRedUnroll], pk[kRedUnroll];
#pragma unroll
        for (int q = 0; q < kRedUnroll; ++q) {
            const int b = b0 + q * BLOCK;
            const bool ok = b < n;
            pu[q] = ok ? e[3 * b + 0] : 0.0;
            pw[q] = ok ? e[3 * b + 1] : 0.0;
            pk[q] = ok ? e[3 * b + 2] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < kRedUnroll; ++q) {
            if (b0 + q * BLOCK < n) {
                u += pu[q];
                w += pw[q];
                k += pk[q];
            }
        }
    }
}
// LOSS: out3[0] = kcoef K + wcoef W instead of (U, K, W). With kcoef and
// wcoef nonzero otherwise, also out3[3] = kcoef K and out3[4] = wcoef (2 K + W)
// (the temperature and the pressure, with kcoef = 2 / (3 N - 3) and
// wcoef = 1 / (3 V)).
template <bool LOSS>
__global__ void __launch_bounds__(kFinalBlock) k_energy_final(SimArgs a, double* out3, bool from_step, double kcoef,
                                                              double wcoef) {
    if (from_step && (a.hdr[HDR_ERROR] & DEV_ORDER)) return;
    const int t = threadIdx.x;
    double x[3] = {0.0, 0.0, 0.0};
    sum_partials<kFinalBlock>(a.epart, a.ncells, t, x[0], x[1], x[2]);
    block_sum<kFinalBlock>(x, t);
    if (t == 0) {
        if (LOSS) {
            out3[0] = kcoef * x[2] + wcoef * (0.5 * x[1]);
        } else {
            out3[0] = 0.5 * x[0];
            out3[1] = x[2];
            out3[2] = 0.5 * x[1];
            if (wcoef != 0.0) {
                out3[3] = kcoef * x[2];
                out3[4] = wcoef * (2.0 * x[2] + 0.5 * x[1]);
            }
        }
    }
}

// Batched final sums: one workgroup per replica, fixed order over its cells;
// out[3 b + 0..2] = U, K, W of replica b.
__global__ void __launch_bounds__(kRedBlock)
    k_batch_energy_final(SimArgs base, const Replica* __restrict__ reps, double* out) {
    if (base.hdr[HDR_ERROR] & DEV_ORDER) return;
    const Replica r = reps[blockIdx.x];
    const int t = threadIdx.x;
    double x[3] = {0.0, 0.0, 0.0};
    sum_partials<kRedBlock>(base.epart + 3 * static_cast<size_t>(r.cbase), r.ncells, t, x[0], x[1], x[2]);
    block_sum<kRedBlock>(x, t);
    if (t == 0) {
        out[3 * blockIdx.x + 0] = 0.5 * x[0];
        out[3 * blockIdx.x + 1] = x[2];
        out[3 * blockIdx.x + 2] = 0.5 * x[1];
    }
}

// Neighbour export through the force kernel's own staging, screen and walk.
// LIST 1 screens against the list radius and keeps the accept words, as the
// force pass right after a rebuild of md_step_list does; LIST 2 walks the
// words kept last, as its passes between rebuilds do.
template <int LIST>
__global__ void __launch_bounds__(kWave) k_neighbors(SimArgs a, ExportArgs ex) {
    if (!state_ok(a, false)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&a.hdr[HDR_ERROR], DEV_ORDER);
        return;
    }
    extern __shared__ float4 tile[];  // 2 x (tile_cap + kTilePad): frame positions, then untranslated ones
    __shared__ Neighbourhood nb;
    force_cell<false, false, false, false, false, LIST, true>(a, xcd_block_order(blockIdx.x, a.ncells), tile, nb,
                                                              reinterpret_cast<float*>(tile),
                                                              tile + (a.tile_cap + kTilePad), ex);
}

}  // namespace

hipError_t launch_forces(const SimArgs& a_in, bool kick, bool energy, bool write_force, bool from_step, bool drift,
                         int par, hipStream_t st) {
    SimArgs a = a_in;
    a.par = par;
    const dim3 g(a.ncells), b(kWave * a.waves);
    const size_t lds = sizeof(float4) * cell_lds_entries(a.tile_cap, a.waves);
#define MD_FORCES(K, E, W, D)                                                                          \
    do {                                                                                               \
        if (a.waves == 1) hipLaunchKernelGGL((k_forces<K, E, W, D, 1>), g, b, lds, st, a, from_step);  \
        else hipLaunchKernelGGL((k_forces<K, E, W, D, kMaxCellWaves>), g, b, lds, st, a, from_step);   \
    } while (0)
    if (kick && drift && !write_force) {
        if (energy) MD_FORCES(true, true, false, true);
        else MD_FORCES(true, false, false, true);
    } else if (kick && !drift && write_force) {
        if (energy) MD_FORCES(true, true, true, false);
        else MD_FORCES(true, false, true, false);
    } else if (!kick && !drift && energy && !write_force) {
        MD_FORCES(false, true, false, false);
    } else if (!kick && !drift && !energy && write_force) {
        MD_FORCES(false, false, true, false);
    } else {
        return hipErrorInvalidValue;
    }
#undef MD_FORCES
    return hipGetLastError();
}

hipError_t launch_forces_skin(const SimArgs& a, bool energy, hipStream_t st) {
    const dim3 g(a.ncells), b(kWave * a.waves);
    const size_t lds = sizeof(float4) * cell_lds_entries(a.tile_cap, a.waves);
    if (a.waves == 1) {
        if (energy) hipLaunchKernelGGL((k_forces_skin<true, 1>), g, b, lds, st, a);
        else hipLaunchKernelGGL((k_forces_skin<false, 1>), g, b, lds, st, a);
    } else {
        if (energy) hipLaunchKernelGGL((k_forces_skin<true, kMaxCellWaves>), g, b, lds, st, a);
        else hipLaunchKernelGGL((k_forces_skin<false, kMaxCellWaves>), g, b, lds, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_forces_list(const SimArgs& a_in, bool energy, bool record, bool bin, int par, hipStream_t st) {
    SimArgs a = a_in;
    a.par = par;
    a.waves = 1;  // the kept words are per lane of one wavefront
    const dim3 g(a.ncells), b(kWave);
    const size_t lds = sizeof(float4) * static_cast<size_t>(a.tile_cap + kTilePad);
#define MD_LIST(E, R, B) hipLaunchKernelGGL((k_forces_list<E, R, B>), g, b, lds, st, a)
    if (energy) {
        if (record) {
            if (bin) MD_LIST(true, true, true);
            else MD_LIST(true, true, false);
        } else {
            if (bin) MD_LIST(true, false, true);
            else MD_LIST(true, false, false);
        }
    } else {
        if (record) {
            if (bin) MD_LIST(false, true, true);
            else MD_LIST(false, true, false);
        } else {
            if (bin) MD_LIST(false, false, true);
            else MD_LIST(false, false, false);
        }
    }
#undef MD_LIST
    return hipGetLastError();
}

hipError_t launch_forces_record(const SimArgs& a_in, bool energy, bool bin, int par, hipStream_t st) {
    SimArgs a = a_in;
    a.par = par;
    const dim3 g(a.ncells), b(kWave);
    const size_t entries = static_cast<size_t>(a.tile_cap + kTilePad);
    const size_t lds = sizeof(float4) * entries + sizeof(uint32_t) * entries;
    if (energy) {
        if (bin) hipLaunchKernelGGL((k_forces_record<true, true>), g, b, lds, st, a);
        else hipLaunchKernelGGL((k_forces_record<true, false>), g, b, lds, st, a);
    } else {
        if (bin) hipLaunchKernelGGL((k_forces_record<false, true>), g, b, lds, st, a);
        else hipLaunchKernelGGL((k_forces_record<false, false>), g, b, lds, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_nlist_forces(const SimArgs& a_in, bool bin, int par, hipStream_t st) {
    SimArgs a = a_in;
    a.par = par;
    const dim3 g((a.n + kListAtoms - 1) / kListAtoms), b(kListBlock);
    if (bin) hipLaunchKernelGGL(k_nlist_forces<true>, g, b, 0, st, a);
    else hipLaunchKernelGGL(k_nlist_forces<false>, g, b, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_energy_final(const SimArgs& a, double* out3, hipStream_t st) {
    hipLaunchKernelGGL(k_energy_final<false>, dim3(1), dim3(kFinalBlock), 0, st, a, out3, true, 0.0, 0.0);
    return hipGetLastError();
}

hipError_t launch_thermo_final(const SimArgs& a, double t_coef, double p_coef, double* out5, hipStream_t st) {
    hipLaunchKernelGGL(k_energy_final<false>, dim3(1), dim3(kFinalBlock), 0, st, a, out5, true, t_coef, p_coef);
    return hipGetLastError();
}

hipError_t launch_loss_final(const SimArgs& a, double kcoef, double wcoef, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_energy_final<true>, dim3(1), dim3(kFinalBlock), 0, st, a, out, true, kcoef, wcoef);
    return hipGetLastError();
}

hipError_t launch_batch_forces(const SimArgs& base_in, const Replica* reps, const int* cell_rep, const int* cells,
                               int ncl, int tile_cap, int waves, bool kick, bool energy, bool write_force, bool drift,
                               int par, hipStream_t st) {
    SimArgs base = base_in;
    base.par = par;
    base.waves = waves;
    const dim3 g(ncl), b(kWave * base.waves);
    const size_t lds = sizeof(float4) * cell_lds_entries(tile_cap, base.waves);
#define MD_FORCES(K, E, W, D)                                                                                      \
    do {                                                                                                           \
        if (base.waves == 1)                                                                                       \
            hipLaunchKernelGGL((k_batch_forces<K, E, W, D, 1>), g, b, lds, st, base, reps, cell_rep, cells, ncl);  \
        else                                                                                                       \
            hipLaunchKernelGGL((k_batch_forces<K, E, W, D, kMaxCellWaves>), g, b, lds, st, base, reps, cell_rep,   \
                               cells, ncl);                                                                        \
    } while (0)
    if (kick && drift && !write_force) {
        if (energy) MD_FORCES(true, true, false, true);
        else MD_FORCES(true, false, false, true);
    } else if (kick && !drift && write_force) {
        if (energy) MD_FORCES(true, true, true, false);
        else MD_FORCES(true, false, true, false);
    } else if (!kick && !drift && energy && !write_force) {
        MD_FORCES(false, true, false, false);
    } else if (!kick && !drift && !energy && write_force) {
        MD_FORCES(false, false, true, false);
    } else {
        return hipErrorInvalidValue;
    }
#undef MD_FORCES
    return hipGetLastError();
}

hipError_t launch_batch_energy_final(const SimArgs& base, const Replica* reps, int count, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_energy_final, dim3(count), dim3(kRedBlock), 0, st, base, reps, out);
    return hipGetLastError();
}

hipError_t launch_neighbors(const SimArgs& a, int* counts, int* idx, int max_per_atom, int list, hipStream_t st) {
    hipError_t e = hipMemsetAsync(counts, 0, sizeof(int) * static_cast<size_t>(a.n), st);
    if (e != hipSuccess) return e;
    const ExportArgs ex{counts, idx, max_per_atom};
    const size_t lds = 2 * sizeof(float4) * static_cast<size_t>(a.tile_cap + kTilePad);
    if (list == 1) hipLaunchKernelGGL(k_neighbors<1>, dim3(a.ncells), dim3(kWave), lds, st, a, ex);
    else if (list == 2) hipLaunchKernelGGL(k_neighbors<2>, dim3(a.ncells), dim3(kWave), lds, st, a, ex);
    else hipLaunchKernelGGL(k_neighbors<0>, dim3(a.ncells), dim3(kWave), lds, st, a, ex);
    return hipGetLastError();
}

}  // namespace mdlj
