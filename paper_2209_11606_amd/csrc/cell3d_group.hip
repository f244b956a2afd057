// cell3d_group.hip -- the 3D cell kernel with several cells per wavefront and
// synchronised cuts.
//
// The method is the one of cell3d.hip: a cell is a set of dual triangles
// (one per vertex, three plane ids each) with a table of twin edges in LDS; a
// candidate plane (the bisector of Eq. 3) is tested against every vertex
// with a ballot, and a cut replaces the conflict region by a fan of new
// triangles around the new plane.  The candidates come from the grid blocks
// in nearest-first order (section 2.1.3) and the search ends by the radius
// bound (section 2.1.3).  Two kinds of cell are left to the spill pass, the
// one-cell kernel of cell3d.hip: a cell whose search radius still reaches
// four block sides after its nearest blocks, or whose search would run past
// the precomputed block offsets (an extended cell, section 3.1), whose 64
// lanes run the block bound's shell search there; and a cell with a side
// decision (a vertex test or an edge's degeneracy test) in the band of the
// exact predicate, which decides it there.  The exact expansions stay out
// of this kernel: they would hold registers that the cell state needs, for
// about one side test in 10^8 on random input.
//
// Mapping.  A cell is owned by a group of G lanes (G = 16 or 32, so 64/G
// cells share a wavefront).  Each group runs a small state machine:
//
//   NEW -> GATHER -> BATCH -> TEST -> (CUT -> TEST)* -> ... -> STATS -> NEW
//
// GATHER reads the particle counts of up to 64 blocks and BATCH loads up to
// 64 particles, keeps those inside the radius bound and sorts them by distance
// (a rank count over the keys), both with the whole wave for one cell at a
// time.  TEST takes the sorted candidates one at a time, and a conflict
// parks the group in CUT.  The cut itself (the costliest step) runs only once
// no group of the wave can advance without one, so that the cuts of the
// wave's cells run in the same instructions instead of one after another.  STATS (volume, centroid, counts, face
// orders, neighbours) is deferred in the same way.
//
// All masks are the group's bit fields (32 bits), reductions are DPP row
// operations plus one swizzle across the two rows of a 32-lane group.  Each
// group is one workgroup's slice of LDS; LDS hand-offs use a workgroup-scope
// fence (one wave per workgroup).
#include "cell_common.h"

namespace vc {

namespace {

template <int G>
struct Gw {
    static constexpr int CPW = 64 / G;
    static constexpr uint32_t FULL = G >= 32 ? 0xffffffffu : ((1u << G) - 1u);
};

// blocks of a cell's first gather (periodic 10^6, two cells per wave, step: 8
// blocks 10.05 ms, 12 9.84, 16 9.80, 24 9.73, 32 9.77)
constexpr int kFirstBlocks = 24;

// a negative phase is a failure (-ST_*)
enum { PH_NEW, PH_GATHER, PH_BATCH, PH_TEST, PH_CUT, PH_STATS, PH_DONE };

__device__ __forceinline__ void lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// the group's bits of a wave ballot
template <int G>
__device__ __forceinline__ uint32_t gbal(bool p, int gb)
{
    unsigned long long b = __builtin_amdgcn_ballot_w64(p);
    if (G == 32) return gb ? (uint32_t)(b >> 32) : (uint32_t)b;
    return (uint32_t)(b >> gb) & Gw<G>::FULL;
}

// lane i of a 32-lane group exchanges with lane i ^ 16
__device__ __forceinline__ int swz16(int v)
{
    return __builtin_amdgcn_ds_swizzle(v, 0x401f);
}

template <int G>
__device__ __forceinline__ uint32_t gmax_u32(uint32_t v)
{
    int x = (int)v;
    x = (int)max((uint32_t)x, (uint32_t)dpp_i32<DPP_QUAD_1032, 0xf>(x, x));
    x = (int)max((uint32_t)x, (uint32_t)dpp_i32<DPP_QUAD_2301, 0xf>(x, x));
    x = (int)max((uint32_t)x, (uint32_t)dpp_i32<DPP_ROW_HALF_MIRROR, 0xf>(x, x));
    x = (int)max((uint32_t)x, (uint32_t)dpp_i32<DPP_ROW_MIRROR, 0xf>(x, x));
    if (G >= 32) x = (int)max((uint32_t)x, (uint32_t)swz16(x));
    return (uint32_t)x;
}

template <int G>
__device__ __forceinline__ int gisum(int v)
{
    v = v + dpp_i32<DPP_QUAD_1032, 0xf>(0, v);
    v = v + dpp_i32<DPP_QUAD_2301, 0xf>(0, v);
    v = v + dpp_i32<DPP_ROW_HALF_MIRROR, 0xf>(0, v);
    v = v + dpp_i32<DPP_ROW_MIRROR, 0xf>(0, v);
    if (G >= 32) v = v + swz16(v);
    return v;
}

// fixed combination order: the same sum on every run
template <int G>
__device__ __forceinline__ double gsum(double v)
{
    v = v + dpp_f64<DPP_QUAD_1032, 0xf>(0.0, v);
    v = v + dpp_f64<DPP_QUAD_2301, 0xf>(0.0, v);
    v = v + dpp_f64<DPP_ROW_HALF_MIRROR, 0xf>(0.0, v);
    v = v + dpp_f64<DPP_ROW_MIRROR, 0xf>(0.0, v);
    if (G >= 32) {
        unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        unsigned lo = (unsigned)swz16((int)(unsigned)u), hi = (unsigned)swz16((int)(unsigned)(u >> 32));
        double w = __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
        // both rows add the same two partial sums in the same order
        v = (threadIdx.x & 16) ? w + v : v + w;
    }
    return v;
}

// search state of a group that only the phase steps read (kept in LDS to
// leave registers for the side tests and cuts)
struct GState {
    double p[3];            // the particle
    int bc[3];              // its block
    int fl[3];              // reflection of the block offsets per axis (+1 or -1)
    int si, id;             // sorted index, input index
    double ri;              // the particle's radius (radical tessellation), else 0
    int cur;                // next offset index
    int gtot, gc0;          // candidates of the gather, next batch start
    int tess;               // its tessellation
    uint32_t cnt[DC_N];     // counters other than candidates and tests
};

// A candidate of the batch.  dk orders it: the high word of |q|^2 less 2^-15
// of it (the batch's sorting resolution), with the image code in the low seven
// bits.
struct alignas(16) Cand {
    double q[3], h;  // the plane q.r = h
    double band;     // FP64 side-test band
    int32_t id;      // particle
    uint32_t dk;
};

// The group's LDS.  The radical instantiation has the same layout: its
// plane offsets already hold the radii, and the radii themselves fed only
// the exact predicate, which this kernel leaves to the one-cell kernel.
template <int G, int S, int MAXP, bool RAD>
struct SL {
    alignas(16) double pq[MAXP][4];  // planes n.r = h (n = q for a bisector, h = |q|^2 / 2)
    GState gs;
    int32_t plab[MAXP];
    uint8_t psh[MAXP];
    // edge k of slot t is number 4 t + k: nb[it] is the number of the same
    // edge in the triangle across it
    alignas(4) uint8_t nb[4 * G * S];
    union alignas(16) {
        struct {               // the search
            Cand cq[G];        // the batch's candidates, nearest first
            int32_t cpre[65];  // the gather's blocks: particles before, first particle less that,
            int32_t coff[64];  // image code
            uint8_t ccode[64];
            union {
                double off[6];                        // NEW: corner offsets
                struct {                              // BATCH: ranking keys, block of each lane
                    alignas(16) uint32_t key[G + 4];
                    uint8_t mark[64];
                } b;
                struct {                              // CUT: boundary edges a | b << 8 | number << 16,
                    uint32_t bedge[G * S];            // 4 x slot of the new triangle whose first plane is a
                    uint8_t first[MAXP];
                } c;
            } x;
        } w;
        struct {               // the statistics of the finished cell
            double pos[G * S][3];
            uint32_t tpl[G * S];
            int32_t forder[MAXP];
            int32_t fref[MAXP];
            int32_t fo[kFoLen];
        } st;
    } u;
};

// one cell and its search state, held by a group (values are the same on
// every lane of the group, apart from the per-lane slots)
template <int S, bool F32>
struct SCell {
    uint32_t tp[S];              // plane ids a | b << 8 | c << 16
    double vx[S], vy[S], vz[S];  // vertex, relative to the particle
    float fx[S], fy[S], fz[S];
    uint32_t live[S];            // live slots (group bit fields)
    uint32_t conf[S];            // conflict slots of the pending cut
    uint32_t used;               // plane slots in use (at most 32)
    uint32_t hw[S];              // squared vertex norm: its high word plus one; 0 for a free slot
    uint32_t rk;                 // their maximum over the cell
    double lim;                  // squared search radius (upper bound)
    uint32_t dlim;               // its high word, the low seven bits set: a candidate whose dk is above lies beyond
    int phase;
    int bn, bk;                  // candidates of the batch, next one
};

template <int MAXP>
__device__ __forceinline__ int free_plane(uint32_t used)
{
    static_assert(MAXP <= 32, "plane slots");
    constexpr uint32_t valid = MAXP >= 32 ? ~0u : ((1u << MAXP) - 1u);
    const uint32_t fr = ~used & valid;
    return fr ? __builtin_ctz(fr) : -1;
}

// Radius bound: the largest squared vertex norm, rounded up to 20 mantissa
// bits (the high word of the double plus one unit, kept per slot), so the
// group maximum is a 32-bit DPP reduction.  R and the search radius are upper
// bounds, which is all the radius test and the error bands need.
template <int G, int S, bool F32>
__device__ __forceinline__ void update_radius(SCell<S, F32> &c, const CellArgs &A, double ri)
{
    uint32_t m = c.hw[0];
#pragma unroll
    for (int s = 1; s < S; s++) m = max(m, c.hw[s]);
    m = gmax_u32<G>(m);
    c.rk = m;
    const double R2 = __builtin_bit_cast(double, (unsigned long long)m << 32);
    c.lim = A.rad ? search_lim(R2, radius_bound(m), A, ri) : 4.0 * R2 * kMargin;
    c.dlim = (uint32_t)(__builtin_bit_cast(unsigned long long, c.lim) >> 32) | 127u;
}

template <int G, int S, int MAXP, bool F32, bool RAD>
__device__ __forceinline__ void cell_fail(const CellArgs &A, SL<G, S, MAXP, RAD> &sh, SCell<S, F32> &c, int st, int gl)
{
    const int id = sh.gs.id;
    if (A.fo)
        for (int k = gl; k < kFoLen; k += G) A.fo[(int64_t)id * kFoLen + k] = 0;
    if (gl == 0) {
        if (A.vol) A.vol[id] = __builtin_nan("");
        if (A.cen) A.cen[3 * (int64_t)id] = A.cen[3 * (int64_t)id + 1] = A.cen[3 * (int64_t)id + 2] = __builtin_nan("");
        if (A.nv) A.nv[id] = 0;
        if (A.ne) A.ne[id] = 0;
        if (A.nf) A.nf[id] = 0;
        if (A.wbl) A.wbl[id] = 0;
        if (st == ST_DUP) {
            A.status[id] = 3;
        } else {
            A.status[id] = 1;
            int pos = atomicAdd(A.spill_count, 1);
            A.spill_list[pos] = sh.gs.si;
        }
    }
    if (st != ST_DUP) sh.gs.cnt[DC_SPILL]++;
    c.phase = PH_NEW;
}

// The search steps take all 64 lanes for one cell: a wave's cells seldom
// need particles at the same moment, and a step for one cell costs the wave
// the same with 64 lanes as with G.  The cell's values are wave-uniform here
// (its record is read through the scalar cache).  With G lanes a cell of the
// periodic 10^6 set took 8 batches and 3 gathers, nearly all of them with the
// other half of the wave idle; with 64, 4,771 -> 4,317 VALU instructions a
// cell and the step 10.71 -> 9.80 ms (two cells per wave).

typedef const __attribute__((address_space(4))) Offset *OffsetConst;
typedef const __attribute__((address_space(4))) Particle *ParticleConst;

// ---- NEW: claim the next cell and set up the box (Eq. 1-2) ----
// Returns the next phase; `in`: the lanes of the cell's group.
template <int G, int S, int MAXP, bool F32, bool RAD>
__device__ __forceinline__ int co_new(const CellArgs &A, SL<G, S, MAXP, RAD> &sh, SCell<S, F32> &c, Claim &q, int ncell,
                                      int lane, bool in)
{
    if (q.cell >= q.end && !claim(A, q, ncell)) return PH_DONE;
    const int cell = q.cell++;
    const int si = A.cell_list ? __builtin_amdgcn_readfirstlane(A.cell_list[cell]) : cell;
    ParticleConst me = (ParticleConst)(uintptr_t)(A.part + si);
    const double p[3] = {me->x, me->y, me->z};
    const int id = me->id, tess = me->tess;
    const double ri = A.rad ? A.rad[si] : 0.0;
    TessConst T = (TessConst)(uintptr_t)(A.tess + tess);
    sh.gs.si = si;
    sh.gs.id = id;
    sh.gs.ri = ri;
    sh.gs.tess = tess;
    sh.gs.cur = 0;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        // as block_coord and offset_flip
        const int g = T->G.g[d];
        const double lo = T->G.lo[d], bs = T->G.bs[d];
        const int k = min(max((int)floor((p[d] - lo) * T->G.inv_bs[d]), 0), g - 1);
        sh.gs.p[d] = p[d];
        sh.gs.bc[d] = k;
        sh.gs.fl[d] = (p[d] - (lo + k * bs)) * 2.0 > bs ? -1 : 1;
    }
    if (lane < 6) {
        // face 2d + side of the box (Eq. 1-2, clipped as in section 3.1.3),
        // as box_side
        const int d = lane >> 1, side = lane & 1;
        const bool d0 = d == 0, d1 = d == 1;
        const double pd = d0 ? p[0] : (d1 ? p[1] : p[2]), L = d0 ? T->G.L[0] : (d1 ? T->G.L[1] : T->G.L[2]);
        const double lo = d0 ? T->G.lo[0] : (d1 ? T->G.lo[1] : T->G.lo[2]);
        const double hi = d0 ? T->G.hi[0] : (d1 ? T->G.hi[1] : T->G.hi[2]);
        const bool per = (d0 ? T->G.per[0] : (d1 ? T->G.per[1] : T->G.per[2])) != 0;
        const double sg = side ? 1.0 : -1.0;
        double off = per ? 0.5 * L : (side ? hi - pd : -(lo - pd));
        double nd = per ? sg * L : sg, h = per ? 0.5 * (L * L) : off;
        int lab = per ? id : -(2 * d + side + 1), code = kNoShift;
        if (per) code += (side ? 1 : -1) * (d0 ? 1 : (d1 ? 5 : 25));
        const double clip = T->clip_half;
        if (clip > 0.0 && clip < off) {
            nd = sg;
            h = off = clip;
            lab = -(7 + 2 * d + side);
            code = kNoShift;
        }
        sh.plab[lane] = lab;
        sh.psh[lane] = (uint8_t)code;
        sh.pq[lane][0] = d0 ? nd : 0.0;
        sh.pq[lane][1] = d1 ? nd : 0.0;
        sh.pq[lane][2] = d == 2 ? nd : 0.0;
        sh.pq[lane][3] = h;
        sh.u.w.x.off[lane] = side ? off : -off;
    }
    lds_fence();
    if (in) {
        const int gl = lane % G;
#pragma unroll
        for (int s = 0; s < S; s++) {
            c.tp[s] = 0;
            c.vx[s] = c.vy[s] = c.vz[s] = 0.0;
            c.fx[s] = c.fy[s] = c.fz[s] = 0.0f;
            c.live[s] = 0;
            c.conf[s] = 0;
            c.hw[s] = 0;
        }
        c.live[0] = 0xffu;
        if (gl < 8) {
            const int bx = gl & 1, by = (gl >> 1) & 1, bz = (gl >> 2) & 1;
            const int X = bx, Y = 2 + by, Z = 4 + bz, neg = 3 - bx - by - bz;
            c.tp[0] = (neg & 1) ? (X | (Z << 8) | (Y << 16)) : (X | (Y << 8) | (Z << 16));
            c.vx[0] = sh.u.w.x.off[X];
            c.vy[0] = sh.u.w.x.off[Y];
            c.vz[0] = sh.u.w.x.off[Z];
            c.fx[0] = (float)c.vx[0];
            c.fy[0] = (float)c.vy[0];
            c.fz[0] = (float)c.vz[0];
            c.hw[0] = norm_key(c.vx[0], c.vy[0], c.vz[0]);
            // the corners across the edges of planes X Y, Y Z and Z X differ in z,
            // x and y; a corner and its neighbour list these planes in opposite
            // senses, so a corner's edges 0, 1, 2 are its neighbours' 2, 1, 0
            const int nz = 4 * (gl ^ 4), nx = 4 * (gl ^ 1), ny = 4 * (gl ^ 2);
            reinterpret_cast<uint32_t *>(sh.nb)[gl] =
                (uint32_t)(((neg & 1) ? ny : nz) + 2) | (uint32_t)(nx + 1) << 8 | (uint32_t)((neg & 1) ? nz : ny) << 16;
        }
        c.used = 0x3fu;
        update_radius<G, S, F32>(c, A, ri);
    }
    lds_fence();
    return PH_GATHER;
}

// ---- GATHER: particle counts of the next blocks of the offset list ----
// The first gather takes kFirstBlocks blocks, whose cuts bring the search
// radius near its final value; the next ones take 64 and keep those inside it.
// Returns the next phase.
template <int G, int S, int MAXP, bool RAD>
__device__ __forceinline__ int co_gather(const CellArgs &A, SL<G, S, MAXP, RAD> &sh, int lane, double lim)
{
    TessConst T = (TessConst)(uintptr_t)(A.tess + __builtin_amdgcn_readfirstlane(sh.gs.tess));
    const int cur = __builtin_amdgcn_readfirstlane(sh.gs.cur);
    // past the offset list: the shell search of the block bound is the
    // one-cell kernel's (the spill pass), as for the extended cells below
    if (cur >= A.noff) return -ST_CAP;
    // no block left in the offset list can hold a cutting particle
    if (((OffsetConst)(uintptr_t)A.offs)[cur].m * 0.25 * T->bsmin2 >= lim) return PH_STATS;
    // after the G nearest blocks the search radius still reaches four block
    // sides, past most of the offset list: an extended cell (section 3.1),
    // left to the one-cell kernel of the spill pass, which tests the list's
    // blocks against the balls and takes 64 blocks of a shell per step
    const bool far = lim > 16.0 * T->bsmin2;
    if (cur >= G && far) return -ST_CAP;
    const int width = cur == 0 ? min(kFirstBlocks, G) : (far ? G - cur : 64);
    const int o = cur + lane;
    bool ok = lane < width && o < A.noff;
    const Offset of = ok ? A.offs[o] : Offset{0, 0, 0, 0};
    const int dd[3] = {of.dx * sh.gs.fl[0], of.dy * sh.gs.fl[1], of.dz * sh.gs.fl[2]};
    // the blocks: periodic wrap by whole periods (at most two each way), walls
    int bb[3], sv[3];
    double d2b = 0.0;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const int g = T->G.g[d];
        const int t = sh.gs.bc[d] + dd[d];
        int w = t, s = 0;
        if (T->G.per[d]) {
            if (g >= kOffRadius) {
                // the list reaches kOffRadius blocks: one period at most
                s = t < 0 ? -1 : (t >= g ? 1 : 0);
                w = t - s * g;
            } else {
                for (int r = 0; r < 3; r++) {
                    const int q = w < 0 ? -1 : (w >= g ? 1 : 0);
                    s += q;
                    w -= q * g;
                }
                if (s > 2 || s < -2 || w < 0 || w >= g) ok = false;
            }
        } else if (t < 0 || t >= g) {
            ok = false;
        }
        bb[d] = w;
        sv[d] = s;
        const double blo = T->G.lo[d] + t * T->G.bs[d];
        const double e = fmax(0.0, fmax(blo - sh.gs.p[d], sh.gs.p[d] - (blo + T->G.bs[d])));
        d2b += e * e;
    }
    if (d2b >= lim) ok = false;
    int cntb = 0, beg = 0;
    if (ok) {
        const int blk = T->bbase + bb[0] + T->G.g[0] * (bb[1] + T->G.g[1] * bb[2]);
        beg = A.start[blk];
        cntb = A.start[blk + 1] - beg;
    }
    const int incl = wave_incl_scan(cntb);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    sh.gs.cnt[DC_BLOCKS] += __popcll(__builtin_amdgcn_ballot_w64(ok));
    sh.gs.cnt[DC_LOADED] += total;
    sh.gs.cur = cur + width;
    if (total == 0) return PH_GATHER;
    sh.u.w.cpre[lane] = incl - cntb;
    sh.u.w.cpre[64] = total;
    sh.u.w.coff[lane] = beg - (incl - cntb);
    sh.u.w.ccode[lane] = (uint8_t)(25 * (sv[2] + 2) + 5 * (sv[1] + 2) + (sv[0] + 2));
    sh.gs.gtot = total;
    sh.gs.gc0 = 0;
    lds_fence();
    return PH_BATCH;
}

// ---- BATCH: the next particles of the gather, sorted by distance ----
// 64 particles are loaded; those inside the search radius, at most G, are the
// batch (when more are inside, as before the first cuts, fewer particles are
// taken).  Returns the next phase and the size of the batch.
template <int G, int S, int MAXP, bool F32, bool RAD>
__device__ __forceinline__ int co_batch(const CellArgs &A, SL<G, S, MAXP, RAD> &sh, int lane, double lim, uint32_t rk,
                                        int &bn)
{
    const int c0 = __builtin_amdgcn_readfirstlane(sh.gs.gc0), tot = __builtin_amdgcn_readfirstlane(sh.gs.gtot);
    if (c0 >= tot) return PH_GATHER;
    // the block of each particle: blocks mark the lane of their first one,
    // and a lane's block is the last mark at or below it
    const int pre = sh.u.w.cpre[lane], nxt = sh.u.w.cpre[lane + 1];
    sh.u.w.x.b.mark[lane] = 0;
    lds_fence();
    if (nxt > pre && nxt > c0 && pre < c0 + 64) sh.u.w.x.b.mark[max(pre - c0, 0)] = (uint8_t)(lane + 1);
    lds_fence();
    const int b = max(wave_max_scan(sh.u.w.x.b.mark[lane]) - 1, 0);
    const int ci = c0 + lane;
    bool valid = ci < tot;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, d2 = 0.0, h = 0.0;
    int pid = 0, code = 0;
    if (valid) {
        const int idx = sh.u.w.coff[b] + ci;
        code = sh.u.w.ccode[b];
        const Particle o = A.part[idx];
        a0 = o.x - sh.gs.p[0];
        a1 = o.y - sh.gs.p[1];
        a2 = o.z - sh.gs.p[2];
        if (code != kNoShift) {
            TessConst T = (TessConst)(uintptr_t)(A.tess + __builtin_amdgcn_readfirstlane(sh.gs.tess));
            const int s0 = code % 5 - 2, s1 = code / 5 % 5 - 2, s2 = code / 25 - 2;
            if (s0) a0 = a0 + s0 * T->G.L[0];
            if (s1) a1 = a1 + s1 * T->G.L[1];
            if (s2) a2 = a2 + s2 * T->G.L[2];
        }
        d2 = a0 * a0 + a1 * a1 + a2 * a2;
        pid = o.id;
        if (A.rad) {
            // radical plane (section 2.1.1): |x|^2 - ri^2 <= |x - q|^2 - rj^2
            h = 0.5 * (d2 + radical_shift(sh.gs.ri, A.rad[idx]));
        } else {
            h = 0.5 * d2;
        }
        valid = d2 < lim && !(idx == sh.gs.si && code == kNoShift);
    }
    unsigned long long vm = __builtin_amdgcn_ballot_w64(valid);
    // radical: whether an empty cell on a coincident particle is a duplicate
    // or empty depends on which of the two shows first, by G particles at a time
    int width = RAD && __builtin_amdgcn_ballot_w64(valid && lane >= G && d2 == 0.0) ? G : 64;
    if (width < 64) vm &= Gw<G>::FULL;
    if (__popcll(vm) > G) {
        do {
            width >>= 1;
            vm &= (1ull << width) - 1;
        } while (width > G && __popcll(vm) > G);
        if (!RAD) valid = valid && lane < width;
    }
    if (RAD) valid = (vm >> lane) & 1;
    bn = __popcll(vm);
    sh.gs.gc0 = c0 + width;
    if (bn == 0) return PH_BATCH;
    // unique 32-bit keys: the high word of the distance (its exponent and
    // 20 mantissa bits) with the low five bits replaced by the place among
    // the batch's particles, so candidates closer than 2^-15 relative may
    // swap; TEST ends a batch only past that resolution
    const int at = lane_rank(vm);
    const uint32_t key = ((uint32_t)(__builtin_bit_cast(unsigned long long, d2) >> 32) & ~31u) | (uint32_t)at;
    // each key counts the smaller ones, four at a time
    if (valid) sh.u.w.x.b.key[at] = key;
    if (lane < 3) sh.u.w.x.b.key[bn + lane] = ~0u;
    lds_fence();
    int rank = 0;
    for (int j = 0; j < bn; j += 4) {
        const uint4 k4 = *reinterpret_cast<const uint4 *>(&sh.u.w.x.b.key[j]);
        rank += (k4.x < key) + (k4.y < key) + (k4.z < key) + (k4.w < key);
    }
    if (valid) {
        // side-test bands with the radius bound of now: R only shrinks, so
        // a band taken now stays wide enough for every later test
        const double R = radius_bound(rk);
        const double band = A.tau * ((fabs(a0) + fabs(a1) + fabs(a2)) * R + fabs(h));
        const uint32_t hd = max((uint32_t)(__builtin_bit_cast(unsigned long long, d2) >> 32), 32u) - 32u;
        sh.u.w.cq[rank] = Cand{{a0, a1, a2}, h, band, pid, (hd & ~127u) | (uint32_t)code};
    }
    lds_fence();
    // a candidate at distance zero (a coincident particle)
    return __builtin_amdgcn_ballot_w64(valid && d2 == 0.0) ? -ST_DUP : PH_TEST;
}

// ---- TEST: side of every vertex against the next candidates ----
// The group's candidates in turn, until one has a conflict (the group parks
// in CUT), one has a vertex in the exact band, or the batch ends.  Side masks
// are whole-wave compares (only the testing groups' lanes are active): the
// step is three FMAs and two compares per slot in use, and while no group of
// the wave has a vertex outside or in band nothing is taken per group.  A
// free slot holds the vertex 0, the particle, which lies inside a bisector
// (s = -h < 0), so it seldom shows there and the live slots are masked only
// where something shows.  Candidates and tests are counted once per run.
// The candidate's offset and bands were set by BATCH.
template <int G, int S, int MAXP, bool F32, bool RAD>
__device__ __forceinline__ void ph_test(const CellArgs &A, SL<G, S, MAXP, RAD> &sh, SCell<S, F32> &c, uint32_t *cnt,
                                        int gl, int gb)
{
    const int k0 = c.bk;
    int k = k0;
    unsigned long long wc[S], wi[S];
    // slots that some testing group uses
    bool inuse[S];
#pragma unroll
    for (int s = 0; s < S; s++) inuse[s] = s == 0 || __builtin_amdgcn_ballot_w64(c.live[s] != 0) != 0;
    int hit = 0;  // 1: conflict, 2: in-band vertex
    for (;;) {
        if (k >= c.bn) break;
        const Cand &cd = sh.u.w.cq[k];
        const double q0 = cd.q[0], q1 = cd.q[1], q2 = cd.q[2], h = cd.h, band = cd.band;
        // past this bound the rest of the batch is beyond the search radius
        // too (a candidate just beyond it is tested and cuts nothing)
        const bool beyond = cd.dk > c.dlim;
        // issue the candidate's three LDS reads together, ahead of the range test
        __asm__ volatile("" ::: "memory");
        if (beyond) break;
        if (F32) {
            const float g0 = (float)q0, g1 = (float)q1, g2 = (float)q2, gh = (float)h;
            const float band32 = (float)(band * A.kband32);
            unsigned long long wu[S], wun = 0;
#pragma unroll
            for (int s = 0; s < S; s++) {
                wc[s] = wu[s] = wi[s] = 0;
                if (!inuse[s]) continue;
                const float sv = fmaf(g0, c.fx[s], fmaf(g1, c.fy[s], fmaf(g2, c.fz[s], -gh)));
                wc[s] = __builtin_amdgcn_fcmpf(sv, band32, 2);             // sv > band
                wu[s] = __builtin_amdgcn_fcmpf(fabsf(sv), band32, 13);     // |sv| <= band or NaN
                wun |= wu[s];
            }
            if (wun) {
                int nre = 0;
#pragma unroll
                for (int s = 0; s < S; s++) {
                    if (!wu[s]) continue;
                    const double sv = fma(q0, c.vx[s], fma(q1, c.vy[s], fma(q2, c.vz[s], -h)));
                    wc[s] |= wu[s] & __builtin_amdgcn_fcmp(sv, band, 2);
                    wi[s] = wu[s] & __builtin_amdgcn_fcmp(fabs(sv), band, 13);
                    nre += __popc((uint32_t)(wu[s] >> gb) & c.live[s]);
                }
                uint32_t ib = 0;
#pragma unroll
                for (int s = 0; s < S; s++) ib |= (uint32_t)(wi[s] >> gb) & c.live[s];
                if (!ib) sh.gs.cnt[DC_RECHECK] += nre;
            }
        } else {
#pragma unroll
            for (int s = 0; s < S; s++) {
                wc[s] = wi[s] = 0;
                if (!inuse[s]) continue;
                const double sv = fma(q0, c.vx[s], fma(q1, c.vy[s], fma(q2, c.vz[s], -h)));
                wc[s] = __builtin_amdgcn_fcmp(sv, band, 2);         // sv > band
                wi[s] = __builtin_amdgcn_fcmp(fabs(sv), band, 13);  // |sv| <= band or NaN
            }
        }
        unsigned long long wany = 0, wib = 0;
#pragma unroll
        for (int s = 0; s < S; s++) {
            wany |= wc[s];
            wib |= wi[s];
        }
        if (wany | wib) {
            uint32_t ic = 0, ii = 0;
#pragma unroll
            for (int s = 0; s < S; s++) {
                ic |= (uint32_t)(wc[s] >> gb) & c.live[s];
                ii |= (uint32_t)(wi[s] >> gb) & c.live[s];
            }
            if (ic | ii) {
                hit = ii ? 2 : 1;
#pragma unroll
                for (int s = 0; s < S; s++) c.conf[s] = (uint32_t)(wc[s] >> gb) & c.live[s];
                break;
            }
        }
        k++;
    }
    c.bk = k;
    const int tested = k - k0 + (hit == 1);
    cnt[0] += tested + (hit == 2);
    int nlive = 0;
#pragma unroll
    for (int s = 0; s < S; s++) nlive += __popc(c.live[s]);
    cnt[1] += tested * nlive;
    if (hit == 0) {
        c.phase = PH_BATCH;
    } else if (hit == 2) {
        // an in-band vertex needs the exact predicate: the cell is left to the
        // one-cell kernel of the spill pass, which decides it exactly; the tests
        // and rechecks of this step are not counted (that kernel counts its own)
        c.phase = -ST_CAP;
    } else {
        c.phase = PH_CUT;
        if (A.rad) {
            // a radical plane can leave no vertex strictly inside: the cell
            // is empty (a Voronoi cell always keeps its particle inside)
            uint32_t inside = 0;
#pragma unroll
            for (int s = 0; s < S; s++) inside |= c.live[s] & ~c.conf[s];
            if (!inside) {
#pragma unroll
                for (int s = 0; s < S; s++) {
                    c.live[s] = 0;
                    c.conf[s] = 0;
                }
                c.phase = PH_STATS;
            }
        }
    }
}

// vertex of planes A, B, C by Cramer's rule, with the reciprocal of the
// determinant by two Newton steps: what the division gives wherever it was
// compared (volumes and centroids bit for bit those of `cramer` in 2.8 million
// cells of uniform, crystal, radical and mixed sets; boxes of sides 2^-250 to
// 2^256 scale exactly).  With the division the same sets take 0.3% to 0.9%
// longer.  Where the determinant or its reciprocal is not a normal number the
// vertex is not finite and the cell goes to the one-cell kernel.
__device__ __forceinline__ void cut_vertex(const double *A, const double *B, const double *C, double &x, double &y,
                                           double &z)
{
    const double bc0 = B[1] * C[2] - B[2] * C[1], bc1 = B[2] * C[0] - B[0] * C[2], bc2 = B[0] * C[1] - B[1] * C[0];
    const double ca0 = C[1] * A[2] - C[2] * A[1], ca1 = C[2] * A[0] - C[0] * A[2], ca2 = C[0] * A[1] - C[1] * A[0];
    const double ab0 = A[1] * B[2] - A[2] * B[1], ab1 = A[2] * B[0] - A[0] * B[2], ab2 = A[0] * B[1] - A[1] * B[0];
    const double det = A[0] * bc0 + A[1] * bc1 + A[2] * bc2;
    double inv = __builtin_amdgcn_rcp(det);
    inv = fma(inv, fma(-det, inv, 1.0), inv);
    inv = fma(inv, fma(-det, inv, 1.0), inv);
    x = (A[3] * bc0 + B[3] * ca0 + C[3] * ab0) * inv;
    y = (A[3] * bc1 + B[3] * ca1 + C[3] * ab1) * inv;
    z = (A[3] * bc2 + B[3] * ca2 + C[3] * ab2) * inv;
}

// ---- CUT: remove the conflict region, fan new triangles around the plane ----
// The kernel is bound by instruction issue and the cut is its costliest step,
// so the triangles across a slot's edges are kept by edge number (nb): a
// conflict slot reads its three twins in one word, where a table by pairs of
// plane ids took three reads and their addresses, and the new triangles are
// linked through the plane their first edge starts at.  The table is 256
// bytes a cell instead of 1,024.  With the norm key kept per slot and the
// lighter TEST step, periodic 10^6 cells: 5,503 -> 4,771 VALU instructions a
// cell, step 11.72 -> 10.71 ms.
template <int G, int S, int MAXP, bool F32, bool RAD>
__device__ __forceinline__ void ph_cut(const CellArgs &A, SL<G, S, MAXP, RAD> &sh, SCell<S, F32> &c, uint32_t *cnt,
                                       int gl, int gb, uint32_t below)
{
    const int k = c.bk;
    int p = free_plane<MAXP>(c.used);
    if (p < 0) {
        // the planes of the kept vertices (one that loses all of them is free)
        uint32_t u = 0;
#pragma unroll
        for (int s = 0; s < S; s++)
            if (((c.live[s] & ~c.conf[s]) >> gl) & 1)
#pragma unroll
                for (int j = 0; j < 3; j++) u |= 1u << ((c.tp[s] >> (8 * j)) & 0xff);
        // group OR of the plane masks
#pragma unroll
        for (int sh_ = 1; sh_ < G; sh_ <<= 1) u |= (uint32_t)__shfl_xor((int)u, sh_);
        c.used = u;
        p = free_plane<MAXP>(c.used);
        if (p < 0) {
            c.phase = -ST_CAP;
            return;
        }
    }
    // boundary edges of the conflict region (conflict triangle edges whose
    // twin triangle is kept), listed edge by edge of each slot
    const uint32_t *nbw = reinterpret_cast<const uint32_t *>(sh.nb);
    unsigned long long keep = 0;
#pragma unroll
    for (int s = 0; s < S; s++) keep |= (unsigned long long)(~c.conf[s] & Gw<G>::FULL) << (s * G);
    int m = 0;
#pragma unroll
    for (int s = 0; s < S; s++) {
        if (s > 0 && !__builtin_amdgcn_ballot_w64(c.conf[s] != 0)) continue;
        const uint32_t w = nbw[s * G + gl], t3 = c.tp[s], mine = (c.conf[s] >> gl) & 1;
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const uint32_t bd = (uint32_t)(keep >> ((w >> (8 * j + 2)) & (G * S - 1))) & mine;
            const uint32_t mb = gbal<G>(bd != 0, gb);
            const int o = m + __popc(mb & below);
            // bytes: planes a, b of the edge, its number in the kept triangle
            if (bd != 0 && o < G * S)
                sh.u.w.x.c.bedge[o] = __builtin_amdgcn_perm(w, t3, 0x0c000000 | (4 + j) << 16 | ((j + 1) % 3) << 8 | j);
            m += __popc(mb);
        }
    }
    uint32_t fr[S];
    int nfree = 0;
#pragma unroll
    for (int s = 0; s < S; s++) {
        fr[s] = (~c.live[s] | c.conf[s]) & Gw<G>::FULL;
        nfree += __popc(fr[s]);
    }
    if (m > nfree || (A.vcap > 0 && G * S - nfree + m > A.vcap)) {
        c.phase = -ST_CAP;
        return;
    }
    const Cand &cd = sh.u.w.cq[k];
    const double C[4] = {cd.q[0], cd.q[1], cd.q[2], cd.h};
    if (gl == 0) {
        sh.pq[p][0] = C[0];
        sh.pq[p][1] = C[1];
        sh.pq[p][2] = C[2];
        sh.pq[p][3] = C[3];
        sh.plab[p] = cd.id;
        sh.psh[p] = (uint8_t)(cd.dk & 127u);
    }
    lds_fence();
    // free slots in slot order take the new triangles (a, b, p) by rank; the
    // lane that takes one computes its vertex
    int before = 0;
    bool take[S];
    uint32_t ed[S];
#pragma unroll
    for (int s = 0; s < S; s++) {
        const int rk = before + __popc(fr[s] & below);
        // one compare: a slot that is not free ranks past every triangle
        take[s] = rk + (int)((~fr[s] >> gl & 1) << 16) < m;
        before += __popc(fr[s]);
        const uint32_t tk = gbal<G>(take[s], gb);
        if ((c.conf[s] >> gl) & 1) {
            // a freed slot holds the particle (TEST) until it is taken
            c.vx[s] = c.vy[s] = c.vz[s] = 0.0;
            if (F32) c.fx[s] = c.fy[s] = c.fz[s] = 0.0f;
            c.hw[s] = 0;
        }
        if (take[s]) {
            ed[s] = sh.u.w.x.c.bedge[rk];
            const int a = ed[s] & 0xff, b = (ed[s] >> 8) & 0xff;
            double x, y, z;
            cut_vertex(sh.pq[a], sh.pq[b], C, x, y, z);
            c.tp[s] = (ed[s] & 0xffff) | ((uint32_t)p << 16);
            c.vx[s] = x;
            c.vy[s] = y;
            c.vz[s] = z;
            if (F32) {
                c.fx[s] = (float)x;
                c.fy[s] = (float)y;
                c.fz[s] = (float)z;
            }
            c.hw[s] = norm_key(x, y, z);
            sh.u.w.x.c.first[a] = (uint8_t)(4 * (s * G + gl));
        }
        c.live[s] = (c.live[s] & ~c.conf[s]) | tk;
        c.conf[s] = 0;
    }
    lds_fence();
    // edges of the new triangle: (a, b) to the kept triangle, (b, p) to the
    // new one whose first plane is b, as that one's edge (p, b)
#pragma unroll
    for (int s = 0; s < S; s++) {
        if (take[s]) {
            const int t = 4 * (s * G + gl), e = ed[s] >> 16, nx = (sh.u.w.x.c.first[(ed[s] >> 8) & 0xff] & 0xfc) | 2;
            *reinterpret_cast<uint16_t *>(sh.nb + t) = (uint16_t)(e | nx << 8);
            sh.nb[nx] = (uint8_t)(t + 1);
            sh.nb[e] = (uint8_t)t;
        }
    }
    lds_fence();
    c.used |= 1u << p;
    update_radius<G, S, F32>(c, A, sh.gs.ri);
    sh.gs.cnt[DC_CUTS]++;
    sh.gs.cnt[DC_NEWV] += m;
    c.bk++;
    c.phase = c.lim < 1e300 ? PH_TEST : -ST_CAP;
}

// ---- STATS: volume, centroid, V/E/F, face orders, neighbours ----
template <int G, int S, int MAXP, bool F32, bool RAD>
__device__ __forceinline__ void ph_stats(const CellArgs &A, SL<G, S, MAXP, RAD> &sh, SCell<S, F32> &c, uint32_t *cnt,
                                         int gl, int gb, uint32_t below)
{
    const int id = sh.gs.id;
    uint32_t anylive = 0;
#pragma unroll
    for (int s = 0; s < S; s++) anylive |= c.live[s];
    if (!anylive) {
        // an empty radical cell: zero volume, no vertices or faces
        if (gl == 0) {
            if (A.vol) A.vol[id] = 0.0;
            if (A.cen) A.cen[3 * (int64_t)id] = A.cen[3 * (int64_t)id + 1] = A.cen[3 * (int64_t)id + 2] = 0.0;
            if (A.nv) A.nv[id] = 0;
            if (A.ne) A.ne[id] = 0;
            if (A.nf) A.nf[id] = 0;
            if (A.wbl) A.wbl[id] = 0;
            A.status[id] = (uint8_t)ST_EMPTY;
        }
        if (A.fo)
            for (int k = gl; k < kFoLen; k += G) A.fo[(int64_t)id * kFoLen + k] = 0;
        c.phase = PH_NEW;
        return;
    }
    lds_fence();
#pragma unroll
    for (int s = 0; s < S; s++) {
        int t = s * G + gl;
        bool lv = (c.live[s] >> gl) & 1;
        sh.u.st.tpl[t] = lv ? c.tp[s] : 0xffffffffu;
        sh.u.st.pos[t][0] = c.vx[s];
        sh.u.st.pos[t][1] = c.vy[s];
        sh.u.st.pos[t][2] = c.vz[s];
    }
    for (int k = gl; k < MAXP; k += G) {
        sh.u.st.forder[k] = 0;
        sh.u.st.fref[k] = 0x7fffffff;
    }
    for (int k = gl; k < kFoLen; k += G) sh.u.st.fo[k] = 0;
    lds_fence();
    for (int t = gl; t < S * G; t += G) {
        uint32_t t3 = sh.u.st.tpl[t];
        if (t3 == 0xffffffffu) continue;
        for (int j = 0; j < 3; j++) atomicMin(&sh.u.st.fref[(t3 >> (8 * j)) & 0xff], t);
    }
    lds_fence();
    // fan apex: the particle when it lies strictly inside the cell (every
    // face offset h > 0, always so for a Voronoi cell), else one vertex
    double o0 = 0.0, o1 = 0.0, o2 = 0.0;
    if (A.rad) {
        bool in = true;
#pragma unroll
        for (int s = 0; s < S; s++)
            if ((c.live[s] >> gl) & 1)
#pragma unroll
                for (int j = 0; j < 3; j++) in = in && sh.pq[(c.tp[s] >> (8 * j)) & 0xff][3] > 0.0;
        if (gbal<G>(!in, gb)) {
            int t0 = 0;
#pragma unroll
            for (int s = S - 1; s >= 0; s--)
                if (c.live[s]) t0 = s * G + __builtin_ctz(c.live[s]);
            o0 = sh.u.st.pos[t0][0];
            o1 = sh.u.st.pos[t0][1];
            o2 = sh.u.st.pos[t0][2];
        }
    }
    // one pass over the edges (a, b) of every live triangle: the edge's
    // degeneracy test and the face orders and fan terms that use it.  A
    // vertex whose opposite vertex across an edge lies on the vertex's
    // fourth plane is degenerate: the edge has zero length; a side clearly
    // inside decides it here, an in-band one is left to the exact
    // predicate of the one-cell kernel.  A fan
    // tetrahedron's volume is zero when its edge has zero length, so the
    // volume and moment sums take every edge; the face-order count skips
    // zero-length edges.
    const double R = radius_bound(c.rk);
    uint32_t ib = 0;
    double v6 = 0.0, m0 = 0.0, m1 = 0.0, m2 = 0.0;
    for (int j = 0; j < 3 * S; j++) {
        int t = (j / 3) * G + gl, k = j % 3;
        uint32_t t3 = sh.u.st.tpl[t];
        if (t3 == 0xffffffffu) continue;
        const int a = (t3 >> (8 * k)) & 0xff, e = sh.nb[4 * t + k];
        const int tw = (e >> 2) & (G * S - 1);
        // the twin's third plane: the one before its edge's first
        const int d = (sh.u.st.tpl[tw] >> ((e & 3) ? 8 * (e & 3) - 8 : 16)) & (MAXP - 1);
        const double *nd = sh.pq[d];
        const double *v0 = sh.u.st.pos[t];
        double sd = nd[0] * v0[0] + nd[1] * v0[1] + nd[2] * v0[2] - nd[3];
        double bd = A.tau * ((fabs(nd[0]) + fabs(nd[1]) + fabs(nd[2])) * R + fabs(nd[3]));
        if (!(sd < -bd)) ib |= 1u << j;
        else atomicAdd(&sh.u.st.forder[a], 1);
        const double *r0 = sh.u.st.pos[sh.u.st.fref[a]];
        const double *w0 = sh.u.st.pos[tw];
        const double r[3] = {r0[0] - o0, r0[1] - o1, r0[2] - o2};
        const double w[3] = {w0[0] - o0, w0[1] - o1, w0[2] - o2};
        const double v[3] = {v0[0] - o0, v0[1] - o1, v0[2] - o2};
        double det = r[0] * (w[1] * v[2] - w[2] * v[1]) - r[1] * (w[0] * v[2] - w[2] * v[0]) +
                     r[2] * (w[0] * v[1] - w[1] * v[0]);
        v6 += det;
        m0 += det * (r[0] + w[0] + v[0]);
        m1 += det * (r[1] + w[1] + v[1]);
        m2 += det * (r[2] + w[2] + v[2]);
    }
    if (gbal<G>(ib != 0, gb)) {
        // an edge whose length is in band: the exact predicate decides it
        // in the one-cell kernel of the spill pass (nothing of the cell has
        // been written yet)
        lds_fence();
        c.phase = -ST_CAP;
        return;
    }
    // no edge has zero length: every triangle is a vertex of its own
    int nvert = 0;
#pragma unroll
    for (int s = 0; s < S; s++) nvert += __popc(c.live[s]);
    lds_fence();
    int rk = 0, sumord = 0;
    bool foover = false;
    for (int k0 = 0; k0 < MAXP; k0 += G) {
        int k = k0 + gl;
        int ord = k < MAXP ? sh.u.st.forder[k] : 0;
        bool real = ord >= 3;
        uint32_t rb = gbal<G>(real, gb);
        int rank = rk + __popc(rb & below);
        if (real) {
            if (ord < kFoLen) atomicAdd(&sh.u.st.fo[ord], 1);
            if ((A.mask & (16 | 32)) && A.nbr && rank < kMaxNbr) {
                A.nbr[(int64_t)id * kMaxNbr + rank] = sh.plab[k];
                A.nsh[(int64_t)id * kMaxNbr + rank] = sh.psh[k];
            }
        }
        rk += __popc(rb);
        sumord += gisum<G>(real ? ord : 0);
        foover = foover || gbal<G>(real && ord >= kFoLen, gb) != 0u;
    }
    const int nface = rk;
    const double vol6 = gsum<G>(v6);
    const double M0 = gsum<G>(m0), M1 = gsum<G>(m1), M2 = gsum<G>(m2);
    lds_fence();
    if (nface > kMaxNbr) {
        cell_fail<G, S, MAXP, F32, RAD>(A, sh, c, ST_CAP, gl);
        return;
    }
    int wl = 0;
    if (A.wbg) {
        // (no edge here has zero length; the vertex positions are no longer
        // needed, and their LDS holds the vertex numbers)
        wl = wb_simple<G, S>(A.wbg + (int64_t)id * kWbStride, sumord, sh.u.st.tpl, TwinNumber<uint8_t>{sh.nb},
                             reinterpret_cast<uint8_t *>(&sh.u.st.pos[0][0]), gl, gb);
    }
    if (gl == 0) {
        if (A.wbl) A.wbl[id] = wl;
        double vol = vol6 / 6.0;
        if (A.vol) A.vol[id] = vol;
        if (A.cen) {
            A.cen[3 * (int64_t)id + 0] = o0 + M0 / (4.0 * vol6);
            A.cen[3 * (int64_t)id + 1] = o1 + M1 / (4.0 * vol6);
            A.cen[3 * (int64_t)id + 2] = o2 + M2 / (4.0 * vol6);
        }
        if (A.nv) A.nv[id] = nvert;
        if (A.ne) A.ne[id] = sumord / 2;
        if (A.nf) A.nf[id] = nface;
        A.status[id] = (uint8_t)(foover ? ST_FO_OVER : ST_OK);
        if (A.lim_out) A.lim_out[sh.gs.si] = c.lim;
    }
    if (A.fo)
        for (int k = gl; k < kFoLen; k += G) A.fo[(int64_t)id * kFoLen + k] = (uint8_t)min(sh.u.st.fo[k], 255);
    lds_fence();
    c.phase = PH_NEW;
}

// candidates and tests are counted in registers, the rest in the group's LDS
template <int G, int S, int MAXP, bool RAD>
__device__ __forceinline__ void flush_counters(const CellArgs &A, SL<G, S, MAXP, RAD> &sh, uint32_t &ncand,
                                               uint32_t &ntest, int gl)
{
    sh.gs.cnt[DC_CAND] += ncand;
    sh.gs.cnt[DC_TESTS] += ntest;
    ncand = ntest = 0;
    lds_fence();
    if (gl < DC_N) {
        uint32_t v = sh.gs.cnt[gl];
        if (v) atomicAdd(&A.diag[gl], (unsigned long long)v);
    }
    lds_fence();
    if (gl < DC_N) sh.gs.cnt[gl] = 0;
    lds_fence();
}

// Occupancy target in waves per SIMD, to which the register allocator is
// held.  The two-cells-per-wave form runs five waves: 96 registers, with 18
// spilled, and 7,968 bytes of LDS per wave (of the 8,192 that twenty waves per
// compute unit leave); a cell that needs more than 32 plane slots goes to the
// spill pass.  At four waves nothing is spilled and the periodic 10^6 step
// takes 9.25 ms against 8.69.
template <int G>
struct SyncWaves {
    static constexpr int value = G == 32 ? 5 : 2;
};

template <int G, int S, int MAXP, bool F32, bool RAD, bool WB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(SyncWaves<G>::value))) void k_cells_sync(CellArgs Ain)
{
    // the Voronoi instantiation carries no radical code, and one without
    // Weinberg records none of their code: those pointers are compile-time
    // nulls
    CellArgs A = Ain;
    if (!RAD) A.rad = nullptr;
    if (!WB) {
        A.wbg = nullptr;
        A.wbl = nullptr;
    }
    static_assert(((G * S) & (G * S - 1)) == 0, "slot count must be a power of two");
    static_assert(G * S <= 64, "edge numbers are bytes, and a cut's kept slots one 64-bit mask");
    static_assert(G == 16 || G == 32, "group width");
    __shared__ SL<G, S, MAXP, RAD> shv[Gw<G>::CPW];
    static_assert(G != 32 || sizeof(shv) <= 160 * 1024 / 20, "twenty waves a compute unit");
    const int lane = __lane_id();
    const int gl = lane % G, gb = lane - gl;
    SL<G, S, MAXP, RAD> &sh = shv[lane / G];
    uint32_t cnt[2] = {0, 0};  // candidates, vertex tests
    const int ncell = A.ncell;
    SCell<S, F32> c;
    c.phase = PH_NEW;
    if (gl < DC_N) sh.gs.cnt[gl] = 0;
    Claim q = first_claim(A, ncell);
    lds_fence();
#ifdef VC_PHASE_CLOCKS
    // wave-level shader-clock cycles and executions of each phase body
    unsigned long long pclk[kPhaseSlots] = {}, pcnt[kPhaseSlots] = {};
    unsigned long long t_prev = clock64();
#define VC_PHASE_MARK(k, ran)                    \
    do {                                         \
        const unsigned long long t_ = clock64(); \
        pclk[k] += t_ - t_prev;                  \
        pcnt[k] += (ran) ? 1 : 0;                \
        t_prev = t_;                             \
    } while (0)
#define VC_PHASE_RAN(ph) (__ballot(c.phase == (ph)) != 0)
#else
#define VC_PHASE_RAN(ph) false
#define VC_PHASE_MARK(k, ran) \
    do {                      \
        (void)(ran);          \
    } while (0)
#endif
    for (;;) {
        if (c.phase == PH_NEW &&
            (cnt[1] > (1u << 30) || sh.gs.cnt[DC_NEWV] > (1u << 30) || sh.gs.cnt[DC_LOADED] > (1u << 30)))
            flush_counters<G, S, MAXP, RAD>(A, sh, cnt[0], cnt[1], gl);
        // each cell that needs particles searches until it has a batch to
        // test or its search has ended
        for (unsigned long long need = __builtin_amdgcn_ballot_w64(c.phase <= PH_BATCH && c.phase >= 0); need;) {
            const int l0 = __builtin_ctzll(need) & ~(G - 1);
            need &= ~((unsigned long long)Gw<G>::FULL << l0);
            SL<G, S, MAXP, RAD> &sg = shv[l0 / G];
            int ph = __builtin_amdgcn_readlane(c.phase, l0), bn = 0;
            if (ph == PH_NEW) {
                ph = co_new<G, S, MAXP, F32, RAD>(A, sg, c, q, ncell, opaque(lane), gb == l0);
                VC_PHASE_MARK(0, true);
            }
            const double lim = readlane_f64(c.lim, l0);
            const uint32_t rk = (uint32_t)__builtin_amdgcn_readlane((int)c.rk, l0);
            while (ph == PH_GATHER || ph == PH_BATCH) {
                if (ph == PH_GATHER) {
                    ph = co_gather<G, S, MAXP, RAD>(A, sg, opaque(lane), lim);
                    VC_PHASE_MARK(1, true);
                }
                if (ph == PH_BATCH) {
                    ph = co_batch<G, S, MAXP, F32, RAD>(A, sg, opaque(lane), lim, rk, bn);
                    VC_PHASE_MARK(2, true);
                }
            }
            if (gb == l0) {
                c.phase = ph;
                c.bn = bn;
                c.bk = 0;
            }
        }
        if (!__builtin_amdgcn_ballot_w64(c.phase != PH_DONE)) break;
#ifdef VC_PHASE_CLOCKS
        const uint32_t t_cand = cnt[0];
#endif
        if (c.phase == PH_TEST) ph_test<G, S, MAXP, F32, RAD>(A, sh, c, cnt, gl, gb);
#ifdef VC_PHASE_CLOCKS
        pcnt[6] += cnt[0] - t_cand;
#endif
        VC_PHASE_MARK(3, true);
        // cuts and statistics wait until no group can advance without one
        if (!__ballot(c.phase <= PH_BATCH)) {
            const bool r_cut = VC_PHASE_RAN(PH_CUT);
            if (c.phase == PH_CUT) {
                // (only the radical form gains by giving up its lane constants here)
                const int l = RAD ? opaque(lane) : lane, gl = l % G, gb = l - gl;
                ph_cut<G, S, MAXP, F32, RAD>(A, shv[l / G], c, cnt, gl, gb, (1u << gl) - 1u);
            }
            VC_PHASE_MARK(4, r_cut);
            const bool r_st = VC_PHASE_RAN(PH_STATS);
            if (c.phase == PH_STATS) {
                const int l = opaque(lane), gl = l % G, gb = l - gl;
                SL<G, S, MAXP, RAD> &sh = shv[l / G];
                ph_stats<G, S, MAXP, F32, RAD>(A, sh, c, cnt, gl, gb, (1u << gl) - 1u);
            }
            VC_PHASE_MARK(5, r_st);
        }
        if (c.phase < 0) {
            const int l = opaque(lane), gl = l % G;
            SL<G, S, MAXP, RAD> &sh = shv[l / G];
            cell_fail<G, S, MAXP, F32, RAD>(A, sh, c, -c.phase, gl);
        }
        VC_PHASE_MARK(7, true);
    }
    flush_counters<G, S, MAXP, RAD>(A, sh, cnt[0], cnt[1], gl);
#ifdef VC_PHASE_CLOCKS
    if (lane == 0)
        for (int k = 0; k < kPhaseSlots; k++) {
            atomicAdd(&A.diag[kPhaseClk + k], pclk[k]);
            atomicAdd(&A.diag[kPhaseCnt + k], pcnt[k]);
        }
#endif
#undef VC_PHASE_MARK
#undef VC_PHASE_RAN
}

}  // namespace

hipError_t launch_cells_group(const CellArgs &a, int precision, int cpw, int waves, hipStream_t s)
{
    const bool rad = a.rad != nullptr, wb = a.wbg != nullptr, f32 = precision == 1;
#define VC_GROUP(G, S, P)                                                                        \
    do {                                                                                         \
        if (rad) {                                                                               \
            if (wb) {                                                                            \
                if (f32) k_cells_sync<G, S, P, true, true, true><<<waves, 64, 0, s>>>(a);        \
                else k_cells_sync<G, S, P, false, true, true><<<waves, 64, 0, s>>>(a);           \
            } else {                                                                             \
                if (f32) k_cells_sync<G, S, P, true, true, false><<<waves, 64, 0, s>>>(a);       \
                else k_cells_sync<G, S, P, false, true, false><<<waves, 64, 0, s>>>(a);          \
            }                                                                                    \
        } else {                                                                                 \
            if (wb) {                                                                            \
                if (f32) k_cells_sync<G, S, P, true, false, true><<<waves, 64, 0, s>>>(a);       \
                else k_cells_sync<G, S, P, false, false, true><<<waves, 64, 0, s>>>(a);          \
            } else {                                                                             \
                if (f32) k_cells_sync<G, S, P, true, false, false><<<waves, 64, 0, s>>>(a);      \
                else k_cells_sync<G, S, P, false, false, false><<<waves, 64, 0, s>>>(a);         \
            }                                                                                    \
        }                                                                                        \
    } while (0)
    if (cpw == 4) VC_GROUP(16, 4, 32);
    else if (cpw == 2) VC_GROUP(32, 2, 32);
    else return hipErrorInvalidValue;
#undef VC_GROUP
    return hipGetLastError();
}

}  // namespace vc
