// weinberg.hip -- Weinberg codes of finished 3D cells: the cell-topology
// code that VoroTop computes for every cell (section 5; Weinberg 1966).
//
// Input: the edge-graph record each cell kernel wrote for its cell (see
// wb_record): V vertices, their degrees, and each vertex's neighbours in one
// common rotational sense.  A walk takes every dart (directed edge) once:
// on reaching a vertex for the first time it leaves by the next dart in the
// rotation after the reversed arrival dart; on reaching a vertex seen before
// it goes back along the same edge unless that was done already, and else
// leaves by the first unused dart in the rotation after the reversed arrival
// dart.  Vertices are numbered 1, 2, ... as first reached; the walk's code is
// the number of the vertex each dart leaves, 2E numbers.  The cell's code is
// the smallest walk code over all 2E starting darts and both rotational
// senses; its symmetry count is the number of (dart, sense) pairs giving it.
//
// The 4E candidate walks run one per lane in lockstep: at each step the lanes
// still alive share the same code prefix, the smallest next number is kept and
// every lane with a larger one drops out; a round whose prefix exceeds the
// best code so far stops.  The first round runs all 2E steps; later rounds
// usually stop within a few.
//
// Two kernels: k_weinberg_small takes the cells of up to 64 vertices and 192
// darts (all but a few in practice), four cells to a wavefront, with each
// lane's walk state in registers (vertices seen: a 64-bit mask; darts taken:
// three) and one table entry per dart; the general kernel takes the rest, one
// wavefront per cell.
#include "cell_common.h"

namespace vc {
namespace {

struct WbLDS {
    uint8_t head[kWbMaxD];               // vertex each dart enters
    uint8_t tailv[kWbMaxD];              // vertex each dart leaves
    uint16_t rev[kWbMaxD];               // the opposite dart
    uint16_t base[kWbMaxV + 1];          // first dart of each vertex
    uint8_t deg[kWbMaxV];
    uint8_t best[kWbMaxD];               // smallest code so far
    uint8_t cur[kWbMaxD];                // the current round's code
    uint8_t lbl[kWbMaxV][64];            // per lane: vertex numbers of its walk
    uint32_t used[(kWbMaxD + 31) / 32][64];  // per lane: darts taken
};

__device__ __forceinline__ int wave_imin(int v)
{
    constexpr int kBig = 0x7fffffff;
    v = min(v, dpp_i32<DPP_QUAD_1032, 0xf>(kBig, v));
    v = min(v, dpp_i32<DPP_QUAD_2301, 0xf>(kBig, v));
    v = min(v, dpp_i32<DPP_ROW_HALF_MIRROR, 0xf>(kBig, v));
    v = min(v, dpp_i32<DPP_ROW_MIRROR, 0xf>(kBig, v));
    v = min(v, dpp_i32<DPP_ROW_BCAST15, 0xa>(kBig, v));
    v = min(v, dpp_i32<DPP_ROW_BCAST31, 0xc>(kBig, v));
    return __builtin_amdgcn_readlane(v, 63);
}

// next dart leaving the tail of d in the rotation (o = 0) or against it
__device__ __forceinline__ int wb_rot(const WbLDS &sh, int d, int o)
{
    const int v = sh.tailv[d], b = sh.base[v], n = sh.deg[v];
    if (o == 0) return d + 1 == b + n ? b : d + 1;
    return d == b ? b + n - 1 : d - 1;
}

__device__ __forceinline__ bool wb_used(const WbLDS &sh, int d, int lane)
{
    return (sh.used[d >> 5][lane] >> (d & 31)) & 1u;
}

constexpr int kSmV = 64, kSmD = 192;  // the small-cell kernel's limits

constexpr int kSmL = 16;              // lanes per cell
constexpr int kSmC = 64 / kSmL;       // cells per wave

constexpr int kSmB = 8;              // cells per wave whose codes are written together
constexpr int kSmDeg = 8;             // darts of a vertex

struct alignas(16) WbSmall {
    uint8_t tailv[kSmD];     // vertex each dart leaves
    uint8_t cand[kSmD];      // candidate starts of sense 0 (their opposites: of sense 1)
    uint8_t deg[kSmV];
    uint8_t base[kSmV];      // first dart of each vertex
    union {
        uint8_t rec[(3 + kSmV + kSmD + 15) / 16 * 16];  // the cell's record
        // per lane: each vertex's number in the walk (0: not reached), and
        // << 8 its darts taken, by their place in the lane's sense
        alignas(16) uint16_t vert[kSmV][kSmL];
    };
};

struct alignas(16) WbWave {
    // per dart of a cell: the vertex it enters, that vertex's first dart << 8
    // and degree << 16, and the opposite dart's place among its darts, counted
    // with the rotation << 20 and against it << 24
    uint32_t tab[kSmB][kSmD];
    int16_t start[kSmB];     // a start of the smallest code (dart, sense << 8), -1: no code here
    uint8_t len[kSmB];       // the code's length
    union {
        WbSmall c[kSmC];     // the cells at work
        struct {             // writing the codes: one lane per cell
            alignas(16) uint16_t vert[kSmV][kSmB];
            uint32_t code[kSmB][kSmD / 4];
        } w;
    };
};

// One step of a walk: dart x of its table enters a vertex whose entry is en
// (si: the shift of the lane's sense o in x).  Sets the vertex's new entry and
// its number lab (nl: the numbers given so far); returns the next dart.
__device__ __forceinline__ int wb_step(uint32_t x, uint32_t &en, int o, int si, int &nl, int &lab)
{
    const int b = (x >> 8) & 0xff, nw = (x >> 16) & 0xf, i = (x >> si) & 0xf;
    const uint32_t fr = ~(en >> 8) & ((1u << nw) - 1u);
    const bool seen = (en & 0xff) != 0;
    nl += seen ? 0 : 1;
    lab = seen ? (int)(en & 0xff) : nl;
    int j = i + __ffs((int)((fr | fr << nw) >> (i + 1)));
    j = j >= nw ? j - nw : j;
    if (seen && ((fr >> i) & 1)) j = i;
    en = (uint32_t)lab | (en & 0xff00u) | 0x100u << j;
    return b + (o ? nw - 1 - j : j);
}

__device__ __forceinline__ int wb_opposite(uint32_t x) { return ((x >> 8) & 0xff) + ((x >> 20) & 0xf); }

// smallest value of each row of 16 lanes, in all its lanes
__device__ __forceinline__ int row_imin(int v)
{
    v = min(v, dpp_i32<DPP_QUAD_1032, 0xf>(v, v));
    v = min(v, dpp_i32<DPP_QUAD_2301, 0xf>(v, v));
    v = min(v, dpp_i32<DPP_ROW_HALF_MIRROR, 0xf>(v, v));
    return min(v, dpp_i32<DPP_ROW_MIRROR, 0xf>(v, v));
}

// the cell's bits of a wave ballot
__device__ __forceinline__ uint32_t row_ballot(bool p, int gb)
{
    return (uint32_t)(__builtin_amdgcn_ballot_w64(p) >> gb) & 0xffffu;
}

// The cells whose record has at most kSmV vertices, kSmDeg darts each and kSmD
// in all (and the cells without a record: symmetry 0).  The others are listed in big (their
// count in queue[2]) for the general kernel.
//
// After some ten steps one walk of a cell is left.  So the walks first only
// decide the smallest start: 16 lanes hold the candidates of most cells at once
// (a dozen on the smallest faces), a wave runs four cells, and a round ends
// when one walk is left; the next round's candidates walk against it.  The
// codes of eight cells are then written together, one lane a cell.  What bounds it
// is instruction issue, so a step has no branch: the way on from a vertex is the opposite dart if the vertex was
// reached before and that dart is free, else the first free dart after it in
// the lane's sense (at a new vertex: the next one), one bit scan of the
// vertex's mask.  200,000 periodic cells: 1.98 ms with one cell to a wave, 1.70
// with four, 1.55 with the branch-free step, 1.15 with the codes written 16 at
// a time (seven waves a compute unit in the LDS), 1.00 with eight (nine waves).
// A wave takes ranges of chunk cells: its first by its number, the later ones
// from the queue.
__global__ __launch_bounds__(64) void k_weinberg_small(const uint8_t *__restrict__ wbg,
                                                       const int32_t *__restrict__ wbl,
                                                       const int64_t *__restrict__ off, int64_t n, int chunk,
                                                       uint8_t *__restrict__ codes, int32_t *__restrict__ sym,
                                                       uint8_t *__restrict__ chiral, int32_t *__restrict__ queue,
                                                       int32_t *__restrict__ big)
{
    __shared__ WbWave sw;
    const int lane = __lane_id(), gl = lane % kSmL, gb = lane - gl, row = lane / kSmL;
    WbSmall &sh = sw.c[row];
    const int64_t firsts = (int64_t)gridDim.x * chunk;
    for (int64_t first = (int64_t)blockIdx.x * chunk; first < n;) {
        const int64_t last = min(first + chunk, n);
        for (int64_t c0 = first; c0 < last; c0 += kSmC) {
            // every branch below is taken by all 16 lanes of a cell
            const int64_t id = c0 + row;
            const int at = (int)(c0 - first) % kSmB + row;
            uint32_t *tab = sw.tab[at];
            const bool here = id < last;
            const int D = here ? wbl[id] : 0;
            int V = 0, Drec = 0;
            if (D > 0) {
                const uint4 *src = reinterpret_cast<const uint4 *>(wbg + id * kWbStride);
                uint4 *dst = reinterpret_cast<uint4 *>(sh.rec);
                for (int k = gl; k < (int)(sizeof(sh.rec) / 16); k += kSmL) dst[k] = src[k];
                wb_fence();
                V = sh.rec[0];
                Drec = sh.rec[1] | (sh.rec[2] << 8);
            }
            // mine: within this kernel's limits
            bool mine = D <= 0 || (V <= kSmV && D <= kSmD);
            bool ok = mine && D > 0 && V >= 4 && Drec == D;
            int count = 0, senses = 0, nc = 0;
            if (ok) {
                // degrees and first darts (four vertices a lane, a scan of the
                // row), dart ends
                constexpr int PV = kSmV / kSmL;
                int dg[PV], sum = 0;
#pragma unroll
                for (int i = 0; i < PV; i++) {
                    dg[i] = PV * gl + i < V ? sh.rec[3 + PV * gl + i] : 0;
                    sum += dg[i];
                }
                int inc = sum;
                inc += dpp_i32<DPP_ROW_SHR1, 0xf>(0, inc);
                inc += dpp_i32<DPP_ROW_SHR2, 0xf>(0, inc);
                inc += dpp_i32<DPP_ROW_SHR4, 0xf>(0, inc);
                inc += dpp_i32<DPP_ROW_SHR8, 0xf>(0, inc);
                ok = __shfl(inc, gb + kSmL - 1) == D;
                if (ok) {
                    int b = inc - sum;
#pragma unroll
                    for (int i = 0; i < PV; i++) {
                        const int v = PV * gl + i;
                        sh.deg[v] = (uint8_t)dg[i];
                        sh.base[v] = (uint8_t)b;
                        for (int j = 0; j < dg[i]; j++) sh.tailv[b + j] = (uint8_t)v;
                        b += dg[i];
                    }
                }
            }
            if (ok) {
                wb_fence();
                // opposites
                bool bad = false, odd = false;
                for (int d = gl; d < D; d += kSmL) {
                    const int v = sh.tailv[d], w = sh.rec[3 + V + d];
                    int b = 0, nw = 1, r = -1;
                    if (w < V) {
                        b = sh.base[w];
                        nw = sh.deg[w];
                        for (int e = b; e < b + nw; e++)
                            if (sh.rec[3 + V + e] == v) r = e;
                    }
                    bad |= r < 0;
                    odd |= nw > kSmDeg;
                    const int i = max(r - b, 0);
                    tab[d] = (uint32_t)w | b << 8 | (nw & 0xf) << 16 | (i & 0xf) << 20 | ((nw - 1 - i) & 0xf) << 24;
                }
                ok = row_ballot(bad, gb) == 0;
                wb_fence();
                if (ok && !row_ballot(odd, gb))
                    for (int d = gl; d < D; d += kSmL) odd |= wb_opposite(tab[wb_opposite(tab[d])]) != d;
                // a vertex of more darts, or not a simple graph (the general
                // kernel tries every start)
                if (ok && row_ballot(odd, gb)) ok = mine = false;
            }
            if (ok) {
                // A walk's code starts 1, 2, ..., p, 1 where p is the size of the
                // face on its turning side (it turns that way at every new
                // vertex until it closes that face), so only the starts on a
                // smallest face can give the smallest code: the candidates.  All
                // faces are walked in step until the first closes; in sense 1
                // the face of a dart is that of its opposite in sense 0.
                constexpr int PD = kSmD / kSmL;
                int e[PD];
                uint32_t closed = 0;
#pragma unroll
                for (int j = 0; j < PD; j++) e[j] = gl + kSmL * j;
                for (int l = 0; l < 64; l++) {
#pragma unroll
                    for (int j = 0; j < PD; j++)
                        if (kSmL * j < D && gl + kSmL * j < D) {
                            const uint32_t x = tab[e[j]];
                            const int b = (x >> 8) & 0xff, nw = (x >> 16) & 0xf, i = (x >> 20) & 0xf;
                            e[j] = b + (i + 1 == nw ? 0 : i + 1);
                            closed |= (e[j] == gl + kSmL * j ? 1u : 0u) << j;
                        }
                    if (row_ballot(closed != 0, gb)) break;
                }
#pragma unroll
                for (int j = 0; j < PD; j++) {
                    const bool is = (closed >> j) & 1;
                    const uint32_t m = row_ballot(is, gb);
                    if (is) sh.cand[nc + __popc(m & ((1u << gl) - 1))] = (uint8_t)(gl + kSmL * j);
                    nc += __popc(m);
                }
                nc *= 2;
                if (nc == 0) ok = mine = false;
                wb_fence();
            }
            // the candidate walks, one per lane, senses in turn; each cell goes
            // through its rounds by itself, from the second on with a start of
            // the smallest code so far in lane 0
            int rep = -1;
            {
                bool run = ok, fresh = ok, alive = false;
                int s0 = 0, k = 0, dcur = 0, nl = 1, lab = 1, o = 0, si = 20, mystart = 0;
                while (__builtin_amdgcn_ballot_w64(run)) {
                    if (fresh) {
                        fresh = false;
                        const uint4 z = {0, 0, 0, 0};
                        for (int i = gl; i < 2 * V; i += kSmL) reinterpret_cast<uint4 *>(sh.vert)[i] = z;
                        wb_fence();
                        const int ci = s0 + gl;
                        alive = ci < nc;
                        o = ci & 1;
                        dcur = sh.cand[alive ? ci >> 1 : 0];
                        if (o) dcur = wb_opposite(tab[dcur]);
                        if (rep >= 0 && gl == 0) {
                            dcur = rep & 0xff;
                            o = rep >> 8;
                        }
                        mystart = dcur | o << 8;
                        si = 20 + 4 * o;
                        const int v = sh.tailv[dcur], i = dcur - sh.base[v];
                        sh.vert[v][gl] = (uint16_t)(1 | 0x100 << (o ? sh.deg[v] - 1 - i : i));
                        nl = lab = 1;
                        k = 0;
                    }
                    const int least = row_imin(alive ? lab : 0x7fffffff);  // by all lanes
                    alive = alive && lab == least;
                    const uint32_t am = row_ballot(alive, gb);
                    if (run && ((am & (am - 1)) == 0 || k == D - 1)) {
                        // one walk left, or several with the same code
                        const bool in0 = alive && o == 0;
                        const uint32_t even = row_ballot(in0, gb), old = rep >= 0 ? 1 : 0;
                        const bool kept = am & old;
                        count = (kept ? count : 0) + __popc(am & ~old);
                        senses = (kept ? senses : 0) | ((even & ~old) ? 1 : 0) | ((am & ~even & ~old) ? 2 : 0);
                        rep = __shfl(mystart, gb + __ffs((int)am) - 1);
                        s0 += kSmL - 1;  // candidates s0 + 1 and up are to come
                        run = fresh = s0 + 1 < nc;
                    } else if (run) {
                        k++;
                        const uint32_t x = tab[dcur];
                        uint32_t en = sh.vert[x & 0xff][gl];
                        dcur = wb_step(x, en, o, si, nl, lab);
                        sh.vert[x & 0xff][gl] = (uint16_t)en;
                    }
                }
                wb_fence();
            }
            if (gl == 0) {
                sw.start[at] = (int16_t)(ok ? rep : -1);
                sw.len[at] = (uint8_t)(ok ? D : 0);
            }
            if (!ok && mine && D > 0 && D <= kWbMaxD) {
                // an inconsistent record: its slot of the codes is zeroed
                uint8_t *out = codes + off[id];
                for (int k = gl; k < D; k += kSmL) out[k] = 0;
            }
            if (here && gl == 0) {
                if (mine) {
                    sym[id] = ok ? count : 0;
                    chiral[id] = ok && senses != 3;
                } else {
                    // beyond this kernel's limits: listed for the general kernel
                    big[atomicAdd(queue + 2, 1)] = (int)id;
                }
            }
            wb_fence();
            if (at - row + kSmC < kSmB && c0 + kSmC < last) continue;
            // the codes of the cells since c0 - (at - row)
            const int cells = at - row + kSmC;
            const int64_t id0 = c0 - (at - row);
            const uint4 z = {0, 0, 0, 0};
            for (int i = lane; i < (int)(sizeof(sw.w.vert) / 16); i += 64) reinterpret_cast<uint4 *>(sw.w.vert)[i] = z;
            wb_fence();
            const int st = lane < cells ? sw.start[lane] : -1, len = st >= 0 ? sw.len[lane] : 0;
            if (len) {
                const uint32_t *tb = sw.tab[lane];
                const int o = st >> 8, si = 20 + 4 * o;
                int dcur = st & 0xff, nl = 1, lab = 1;
                const uint32_t back = tb[wb_opposite(tb[dcur])];  // the start's opposite enters the start's tail
                sw.w.vert[back & 0xff][lane] = (uint16_t)(1 | 0x100 << ((back >> si) & 0xf));
                uint32_t acc = 0;
                for (int k = 0; k < len; k++) {
                    acc |= (uint32_t)lab << (8 * (k & 3));
                    if ((k & 3) == 3 || k == len - 1) {
                        sw.w.code[lane][k >> 2] = acc;
                        acc = 0;
                    }
                    const uint32_t x = tb[dcur];
                    uint32_t en = sw.w.vert[x & 0xff][lane];
                    dcur = wb_step(x, en, o, si, nl, lab);
                    sw.w.vert[x & 0xff][lane] = (uint16_t)en;
                }
            }
            wb_fence();
            for (int c = row; c < cells; c += kSmC) {
                if (sw.start[c] < 0) continue;
                uint8_t *out = codes + off[id0 + c];
                const uint8_t *code = reinterpret_cast<const uint8_t *>(sw.w.code[c]);
                for (int k = gl; k < sw.len[c]; k += kSmL) out[k] = code[k];
            }
            wb_fence();
        }
        int next = 0;
        if (lane == 0) next = atomicAdd(queue, chunk);
        first = firsts + __builtin_amdgcn_readfirstlane(next);
    }
}

// The cells listed by the small kernel (their count in queue[2]).
__global__ __launch_bounds__(64) void k_weinberg(const uint8_t *__restrict__ wbg, const int32_t *__restrict__ wbl,
                                                 const int64_t *__restrict__ off, const int32_t *__restrict__ big,
                                                 uint8_t *__restrict__ codes, int32_t *__restrict__ sym,
                                                 uint8_t *__restrict__ chiral, int32_t *__restrict__ queue)
{
    __shared__ WbLDS sh;
    const int lane = __lane_id();
    const int nbig = __builtin_amdgcn_readfirstlane(queue[2]);
    // Every branch below is taken by the whole wave (its condition is made
    // wave-uniform), and the loop body has no early exit: the next cell is
    // claimed only once the wave has reconverged.
    for (;;) {
        int item = 0;
        if (lane == 0) item = atomicAdd(queue + 1, 1);
        item = __builtin_amdgcn_readfirstlane(item);
        if (item >= nbig) break;
        const int64_t id = __builtin_amdgcn_readfirstlane(big[item]);
        const uint8_t *rec = wbg + id * kWbStride;
        const int D = __builtin_amdgcn_readfirstlane(wbl[id]);
        const int V = D > 0 ? __builtin_amdgcn_readfirstlane((int)rec[0]) : 0;
        const int Drec = D > 0 ? __builtin_amdgcn_readfirstlane((int)(rec[1] | (rec[2] << 8))) : 0;
        const bool mine = D > 0;
        bool ok = mine && D <= kWbMaxD && V >= 4 && V <= kWbMaxV && Drec == D;
        int count = 0, senses = 0;
        if (ok) {
            // vertex degrees, first darts (a wave scan), dart ends and opposites
            for (int v = lane; v < V; v += 64) sh.deg[v] = rec[3 + v];
            const int a = lane < V ? rec[3 + lane] : 0;
            int inc = a;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                const int y = __shfl_up(inc, m);
                if (lane >= m) inc += y;
            }
            if (lane < V) sh.base[lane] = (uint16_t)(inc - a);
            const int tot = __shfl(inc, 63);
            const int b = lane + 64 < V ? rec[3 + lane + 64] : 0;
            int inc2 = b;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                const int y = __shfl_up(inc2, m);
                if (lane >= m) inc2 += y;
            }
            if (lane + 64 < V) sh.base[lane + 64] = (uint16_t)(tot + inc2 - b);
            if (lane == 0) sh.base[V] = (uint16_t)D;
            wb_fence();
            for (int d = lane; d < D; d += 64) {
                sh.head[d] = rec[3 + V + d];
                int lo = 0, hi = V - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (sh.base[mid] <= d) lo = mid; else hi = mid - 1;
                }
                sh.tailv[d] = (uint8_t)lo;
            }
            wb_fence();
            bool bad = false;
            for (int d = lane; d < D; d += 64) {
                const int v = sh.tailv[d], w = sh.head[d];
                int r = -1;
                if (w < V)
                    for (int e = sh.base[w]; e < sh.base[w] + sh.deg[w]; e++)
                        if (sh.head[e] == v) r = e;
                bad |= r < 0;
                sh.rev[d] = (uint16_t)max(r, 0);
            }
            wb_fence();
            const int last = __builtin_amdgcn_readfirstlane((int)sh.base[V - 1] + (int)sh.deg[V - 1]);
            ok = __builtin_amdgcn_ballot_w64(bad) == 0 && last == D;
        }
        if (ok) {
            // the candidate walks, 64 per round: lane l of a round starting
            // at c0 walks from dart (c0 + l) / 2 in sense (c0 + l) % 2
            bool have = false;
            for (int c0 = 0; c0 < 2 * D; c0 += 64) {
                const int c = c0 + lane;
                bool alive = c < 2 * D;
                const int o = lane & 1;
                int dcur = alive ? c >> 1 : 0;
                for (int v = 0; v < V; v++) sh.lbl[v][lane] = 0;
                for (int w = 0; w < (D + 31) / 32; w++) sh.used[w][lane] = 0u;
                int nl = 1;
                if (alive) sh.lbl[sh.tailv[dcur]][lane] = 1;
                bool eq = have, better = !have, done = false;
                for (int k = 0; k < D; k++) {
                    const int sk = alive ? sh.lbl[sh.tailv[dcur]][lane] : 0x7fffffff;
                    const int m = wave_imin(sk);
                    if (m == 0x7fffffff) break;
                    if (eq) {
                        const int bk = __builtin_amdgcn_readfirstlane((int)sh.best[k]);
                        if (m > bk) break;
                        if (m < bk) {
                            eq = false;
                            better = true;
                        }
                    }
                    alive = alive && sk == m;
                    if (lane == 0) sh.cur[k] = (uint8_t)m;
                    if (k == D - 1) {
                        done = true;
                        break;
                    }
                    if (alive) {
                        sh.used[dcur >> 5][lane] |= 1u << (dcur & 31);
                        const int v = sh.head[dcur], r = sh.rev[dcur];
                        if (sh.lbl[v][lane] == 0) {
                            sh.lbl[v][lane] = (uint8_t)(++nl);
                            dcur = wb_rot(sh, r, o);
                        } else if (!wb_used(sh, r, lane)) {
                            dcur = r;
                        } else {
                            int e = wb_rot(sh, r, o);
                            for (int g = 0; g < 256 && wb_used(sh, e, lane); g++) e = wb_rot(sh, e, o);
                            dcur = e;
                        }
                    }
                }
                wb_fence();
                if (done) {
                    const unsigned long long am = __builtin_amdgcn_ballot_w64(alive);
                    const int sm = ((am & 0x5555555555555555ull) ? 1 : 0) | ((am & 0xaaaaaaaaaaaaaaaaull) ? 2 : 0);
                    if (better) {
                        for (int k = lane; k < D; k += 64) sh.best[k] = sh.cur[k];
                        count = __popcll(am);
                        senses = sm;
                        have = true;
                    } else if (eq) {
                        count += __popcll(am);
                        senses |= sm;
                    }
                }
                wb_fence();
            }
            uint8_t *out = codes + off[id];
            for (int k = lane; k < D; k += 64) out[k] = sh.best[k];
        } else if (mine && D <= kWbMaxD) {
            // an inconsistent record: its slot of the codes is zeroed
            uint8_t *out = codes + off[id];
            for (int k = lane; k < D; k += 64) out[k] = 0;
        }
        if (mine && lane == 0) {
            sym[id] = ok ? count : 0;
            chiral[id] = ok && senses != 3;
        }
        wb_fence();
    }
}

}  // namespace

hipError_t launch_weinberg(const uint8_t *wbg, const int32_t *wbl, const int64_t *off, int64_t n, uint8_t *codes,
                           int32_t *sym, uint8_t *chiral, int32_t *queue, int32_t *big, int waves, hipStream_t s)
{
    if (n > 0) {
        // nine waves of the small kernel are resident on a compute unit (LDS);
        // several ranges a wave even the load out
        const int64_t res = std::min<int64_t>(waves, (int64_t)device_cu_count() * 9);
        const int chunk = (int)std::max<int64_t>(kSmC, std::min<int64_t>(2 * kSmB, n / (res * 2) / kSmC * kSmC));
        const int small = (int)std::min<int64_t>(res, (n + chunk - 1) / chunk);
        k_weinberg_small<<<small, 64, 0, s>>>(wbg, wbl, off, n, chunk, codes, sym, chiral, queue, big);
        k_weinberg<<<std::max(1, waves / 16), 64, 0, s>>>(wbg, wbl, off, big, codes, sym, chiral, queue);
    }
    return hipGetLastError();
}

}  // namespace vc
