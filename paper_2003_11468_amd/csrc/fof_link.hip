// Link search + lock-free union-find for gfx950 (wave64).
//
// Cells are split by occupancy. A cell holding at least `dense_min`
// particles is "dense" and is processed by k_link_dense: one wavefront takes
// up to 64 of its particles (one per lane), stages the candidates of each
// neighbour cell in LDS, 64 at a time, and tests every staged candidate
// against all 64 lanes at once (the candidate address is uniform, so the LDS
// read is a broadcast). All other ("sparse") cells are processed per lane by
// k_link_sparse: each lane walks its own neighbour cells.
//
// Every unordered pair of adjacent cells is searched exactly once:
//   both sparse  -> k_link_sparse, from the cell whose half shell holds the other;
//   one dense    -> k_link_dense of the dense cell (it searches all 26 neighbours,
//                   its lower half only where the neighbour is sparse);
//   both dense   -> k_link_dense, from the cell whose half shell holds the other.
// The half shell of (cx, cy, cz) is the 13 offsets with dz > 0, or dz == 0 and
// dy > 0, or dz == dy == 0 and dx > 0. With at least 3 cells per axis the 27
// periodic neighbours are distinct cells.
//
// Periodic images: the neighbour offset fixes the image, so no distance is
// wrapped per pair. In FP32 the image shift is applied where it is exact: the
// home coordinate minus L when the home cell is the top one (Sterbenz), the
// neighbour coordinate minus L when the neighbour is the top one. Each axis
// difference is then one correctly rounded subtraction of two exact values.
// In double, the difference is rounded first and the shift of +-L added after
// it, which is the very operation sequence of the link predicate.
//
// Union-find: a merge hooks the root of lower priority under the other by a
// compare-and-swap: by index, the larger under the smaller, or by a fixed
// pseudo-random priority (randomised linking). Swaps on a root that others
// have hooked meanwhile fail and cost a chain of dependent accesses each, so
// links are gathered where they name the same roots (a tile of the
// per-particle search, a stage of the wavefront search, a chunk of queued
// pairs, a dense cell) and every distinct root is hooked once.
#include <type_traits>

#include "fof_device.h"

namespace fof {
namespace {

using namespace dev;

constexpr int kWaves = kBlock / 64;

__device__ __forceinline__ float lane0(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

__device__ __forceinline__ float qnan() { return __builtin_nanf(""); }

// Merge the groups that contain roots-or-members a and b; returns a node of the
// merged group (the root that stayed a root at the time of the merge).
__device__ __forceinline__ int unite_root(int *parent, int a, int b, bool random, int mode, unsigned &retries)
{
    while (true) {
        a = find_root(parent, a, mode, random);
        b = find_root(parent, b, mode, random);
        if (a == b) return a;
        const bool a_first = link_key(a, random) < link_key(b, random);
        const int lo = a_first ? a : b;
        const int hi = a_first ? b : a;
        int expected = hi;
        if (__hip_atomic_compare_exchange_strong(parent + hi, &expected, lo, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return lo;
        ++retries;
        a = expected;
        b = lo;
    }
}

constexpr unsigned kGlobalMergeBlocks = 2048;

// ------------------------------------------------------ domain decomposition --
// Domain mode (paper, Section 3.3, on one GPU): a box is cut into `domains`
// slabs along x. Union-find merges only links inside a slab; a link across
// slabs goes to the boundary list (the list the paper's ranks exchange), and
// the global merge after the search joins the groups it names.

// Slab of a particle at x in a box of side L.
__device__ __forceinline__ int slab_of(float x, int domains, double L)
{
    const int d = (int)((double)x * (double)domains / L);
    return d < domains ? d : domains - 1;
}

// Slab of sorted particle s.
__device__ __forceinline__ int domain_of(const Plan &p, int s)
{
    const int b = p.n_boxes == 1 ? 0 : find_box(p.box_p0, p.n_boxes, s);
    return slab_of(p.sorted[s].x, p.domains, box_of(p, b).L);
}

// Appends the pair to the boundary list; a pair that finds the list full is
// merged at once (the groups come out the same).
__device__ __forceinline__ void defer_boundary(const Plan &p, int a, int b, unsigned &retries)
{
    const unsigned at = atomicAdd(&p.counters->n_boundary, 1u);
    if ((int64_t)at < p.max_edges) p.bnd[at] = make_int2(a, b);
    else retries += unite(p.parent, a, b, p.link_random, p.find_mode);
}

// Merge of a linked pair found by the search: at once, or in domain mode
// through the boundary list when the pair crosses slabs.
__device__ __forceinline__ void merge_pair(const Plan &p, int a, int b, unsigned &retries)
{
    if (p.domains > 1 && domain_of(p, a) != domain_of(p, b)) defer_boundary(p, a, b, retries);
    else retries += unite(p.parent, a, b, p.link_random, p.find_mode);
}

__device__ __forceinline__ int lds_ld(int *a) { return __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ void lds_st(int *a, int v)
{
    __hip_atomic_store(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Root of sub-cell x in the LDS forest f (path halving; parents only point to
// smaller indices).
__device__ __forceinline__ int lds_find(int *f, int x)
{
    while (true) {
        const int px = lds_ld(f + x);
        if (px == x) return x;
        const int gx = lds_ld(f + px);
        if (gx == px) return px;
        lds_st(f + x, gx);
        x = gx;
    }
}

// Warshall's closure of 64 boolean rows, one per lane (bit v of lane u's row:
// u is joined to v; every row holds its own bit): for each k in `todo` (the
// lanes whose rows hold other bits), every row holding bit k takes in row k,
// read with readlane. Afterwards a row is its lane's component, so its lowest
// bit is the component's smallest member. No branch and no memory access.
__device__ __forceinline__ unsigned long long close_rows(unsigned long long row, unsigned long long todo)
{
    // the two words of each row apart, so that the test of bit k reads one
    // word (k below 32: the low one) and its sign-extended bit masks row k in
    unsigned lo = (unsigned)row, hi = (unsigned)(row >> 32);
    for (unsigned t = (unsigned)todo; t; t &= t - 1u) {
        const int k = __ffs(t) - 1;
        const unsigned klo = (unsigned)__builtin_amdgcn_readlane((int)lo, k);
        const unsigned khi = (unsigned)__builtin_amdgcn_readlane((int)hi, k);
        const unsigned m = (unsigned)__builtin_amdgcn_sbfe((int)lo, (unsigned)k, 1u);
        lo |= klo & m;
        hi |= khi & m;
    }
    for (unsigned t = (unsigned)(todo >> 32); t; t &= t - 1u) {
        const int k = __ffs(t) - 1;
        const unsigned klo = (unsigned)__builtin_amdgcn_readlane((int)lo, k + 32);
        const unsigned khi = (unsigned)__builtin_amdgcn_readlane((int)hi, k + 32);
        const unsigned m = (unsigned)__builtin_amdgcn_sbfe((int)hi, (unsigned)k, 1u);
        lo |= klo & m;
        hi |= khi & m;
    }
    return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ void lds_unite(int *f, int a, int b)
{
    while (true) {
        a = lds_find(f, a);
        b = lds_find(f, b);
        if (a == b) return;
        const int lo = min(a, b), hi = max(a, b);
        int expected = hi;
        if (__hip_atomic_compare_exchange_strong(f + hi, &expected, lo, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
            return;
        a = expected;
        b = lo;
    }
}

// --------------------------------------------------------- sparse (lane) --

// Periodic shift code of one axis for a candidate range: 0 none; 1 the
// neighbour cell is the top one reached across the low face (candidate - L is
// exact); 2 the home cell is the top one and the neighbour lies across the
// high face (home - L is exact). Codes of x, y, z sit in bits 0-1, 2-3, 4-5.
__device__ __forceinline__ float axis_diff(float h, float q, int code, float L32)
{
    const float hh = code == 2 ? h - L32 : h;
    const float qq = code == 1 ? q - L32 : q;
    return hh - qq;
}

__device__ __forceinline__ double axis_shift(int code, double L) { return code == 1 ? L : (code == 2 ? -L : 0.0); }

constexpr int kMaxRanges = 10;

// One candidate range of a home particle: slots [j0, j1) (empty when
// j1 <= j0) and their periodic shift code.
struct Span {
    int j0 = 0, j1 = 0, code = 0;
};

// The three cells (x = cx-1, cx, cx+1) of one neighbour row, given their
// boundaries (st[e], en[e]) and whether the row wraps at either end. Runs of
// sparse, memory-contiguous cells are merged into one range: at most two per
// row (the cells of a row follow each other in memory except across the
// wrap, which is at one end, and around a dense middle cell).
__device__ __forceinline__ void row_spans(const int st[3], const int en[3], const int xcode[3], int yz_code,
                                          int dense_min, Span &A, Span &B)
{
    int a = -1, b = -1, code = 0;
    bool first = true;
    auto emit = [&](int j0, int j1, int c) {
        if (first) A = Span{j0, j1, c};
        else B = Span{j0, j1, c};
        first = false;
    };
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const bool sparse = en[e] - st[e] < dense_min;
        const int c = xcode[e] | yz_code;
        if (sparse && en[e] > st[e]) {
            if (a >= 0 && st[e] == b && c == code) {
                b = en[e];
            } else {
                if (a >= 0) emit(a, b, code);
                a = st[e];
                b = en[e];
                code = c;
            }
        }
    }
    if (a >= 0) emit(a, b, code);
}

// Linked pairs of the sparse search are not merged where they are found: a
// union is a chain of dependent memory accesses, and inside the search it
// would stall the whole wavefront round after round. Each wave collects its
// pairs in LDS and appends them to a global edge list 64 at a time; the
// union kernel then merges all of them with one thread per pair.
constexpr int kEdgeBuf = 128;

// kInline: a wave merges its pairs itself, 64 at a time, instead (small runs,
// where the union kernel's launch costs more than the waiting).
template <bool kInline>
struct EdgeSink {
    int2 *buf;      // this wave's LDS buffer [kEdgeBuf]
    int count;      // wave-uniform fill level

    // Appends (s, j) for every lane with `has`; flushes once 64 are waiting.
    __device__ __forceinline__ void push(const Plan &p, bool has, int s, int j, unsigned &retries)
    {
        const unsigned long long m = __ballot(has);
        if (!m) return;
        if (has) {
            const int at = count + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            buf[at] = make_int2(s, j);
        }
        count += __popcll(m);
        __builtin_amdgcn_wave_barrier();
        if (count >= 64) flush(p, retries);
    }

    // Appends the buffer to this work-group's slice of the edge list (one
    // atomic on the slice counter); pairs that find the slice full are merged here.
    __device__ __forceinline__ void flush(const Plan &p, unsigned &retries)
    {
        if (count == 0) return;
        const int lane = lane_id();
        if constexpr (kInline) {
            for (int k = lane; k < count; k += 64)
                retries += unite(p.parent, buf[k].x, buf[k].y, p.link_random, p.find_mode);
            __builtin_amdgcn_wave_barrier();
            count = 0;
            return;
        }
        const int slice = blockIdx.x % kEdgeSlices;
        const int64_t cap = p.max_edges / kEdgeSlices;
        unsigned base = 0;
        if (lane == 0) base = atomicAdd(&p.edge_fill[slice], (unsigned)count);
        base = (unsigned)__shfl((int)base, 0, 64);
        for (int k = lane; k < count; k += 64) {
            const int2 e = buf[k];
            const int64_t at = (int64_t)base + k;
            if (at < cap) p.edges[slice * cap + at] = e;
            else merge_pair(p, e.x, e.y, retries);
        }
        __builtin_amdgcn_wave_barrier();
        count = 0;
    }
};

// Per-wave LDS for the sparse search: the candidate ranges ("units") of the
// wave's 64 home particles, flattened into one list of pairs by a prefix sum,
// so that every lane tests a pair in every step whatever the range lengths.
constexpr int kMaxUnits = 64 * kMaxRanges;

struct SparseLds {
    // one entry past the last unit holds the number of pairs, and one more is read ahead
    int2 unit[kMaxUnits + 2];   // {first pair of the unit (exclusive prefix), its first candidate}
    unsigned short tag[kMaxUnits + 2];   // shift code (bits 0-5) | home lane << 8
    float4 home[64];                 // the home particles
    int2 ebuf[kEdgeBuf];             // edge sink buffer
    unsigned long long adj[64];      // links inside the tile: bit v of adj[u] for home u, slot s0 + v
};

// Box parameters of the pair test, in registers.
struct BoxPair {
    double L, half, l2;
    float L32, lo32, hi32;
    __device__ __forceinline__ static BoxPair of(const BoxDev &bd)
    {
        return BoxPair{bd.L, bd.half, bd.l2, bd.L32, bd.lo32, bd.hi32};
    }
};

// The pair loop of the per-particle search over the wave's flattened units.
// Merge-path split: lane l takes the pairs [T l / 64, T (l + 1) / 64) of the
// wave's T pairs, finds the unit of its first pair by one binary search, then
// walks forward; every lane runs the same number of steps. kOneBox: every
// home particle of the tile lies in one box, whose parameters are `bp`.
template <bool kFP64, bool kStats, bool kOneBox, bool kInline>
__device__ __forceinline__ void sparse_pairs(const Plan &p, SparseLds &L, EdgeSink<kInline> &sink, int s0, int n_units,
                                             int n_pairs, int b, BoxPair bp, bool in_tile, unsigned long long &tests,
                                             unsigned long long &links, unsigned long long &band, unsigned &retries)
{
    const int lane = lane_id();
    const bool strict = p.strict != 0;
    const int q0 = (int)(((int64_t)n_pairs * lane) >> 6);
    const int q1 = (int)(((int64_t)n_pairs * (lane + 1)) >> 6);
    int u = 0;
    for (int step = n_units > 1 ? 1 << (31 - __clz(n_units - 1)) : 0; step > 0; step >>= 1) {
        const int nxt = u + step;
        if (nxt < n_units && L.unit[nxt].x <= q0) u = nxt;
    }
    int jq = L.unit[u].y + (q0 - L.unit[u].x);   // candidate of pair q
    int tag = L.tag[u], next_start = L.unit[u + 1].x;
    // the unit after this one, read ahead, so that a lane that steps into it
    // does not wait for LDS
    int ahead_j0 = L.unit[u + 1].y, ahead_next = L.unit[u + 2].x, ahead_tag = L.tag[u + 1];
    u += 2;
    // four steps at a time: their candidate loads are in flight together, and
    // their home particles are read while those are (lanes past their last
    // pair load their tile's first particle)
    constexpr int kAhead = 4;
    const int steps = (n_pairs + 63) >> 6;   // at least every lane's pairs
    int q = q0;
    for (int k = 0; k < steps; k += kAhead) {
        int jj[kAhead], tg[kAhead];
        float4 hh[kAhead], cc[kAhead];
        bool lv[kAhead];
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
            lv[a] = q < q1;
            if (lv[a] && q == next_start) {   // the next unit starts here
                jq = ahead_j0;
                tag = ahead_tag;
                next_start = ahead_next;
                const int v = min(u, kMaxUnits);   // a lane in its last unit reads past the list
                ahead_j0 = L.unit[v].y;
                ahead_next = L.unit[v + 1].x;
                ahead_tag = L.tag[v];
                ++u;
            }
            jj[a] = lv[a] ? jq : s0;
            tg[a] = tag;
            jq += lv[a] ? 1 : 0;
            q += lv[a] ? 1 : 0;
        }
#pragma unroll
        for (int a = 0; a < kAhead; ++a) cc[a] = p.sorted[jj[a]];
#pragma unroll
        for (int a = 0; a < kAhead; ++a) hh[a] = L.home[tg[a] >> 8];
        // no lane's pairs of these steps need a periodic shift (the common
        // case away from the box faces): plain differences, the same values
        bool plain = false;
        if constexpr (!kFP64) {
            int codes = 0;
#pragma unroll
            for (int a = 0; a < kAhead; ++a) codes |= tg[a];
            plain = __ballot((codes & 63) != 0) == 0;
        }
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
            const int hl = tg[a] >> 8, code = tg[a] & 63;
            BoxPair bx = bp;
            if constexpr (!kOneBox) bx = BoxPair::of(p.boxes[__shfl(b, hl, 64)]);
            const float4 c = cc[a], hp = hh[a];
            bool link;
            if constexpr (kFP64) {
                const double tx = ((double)hp.x - (double)c.x) + axis_shift(code & 3, bx.L);
                const double ty = ((double)hp.y - (double)c.y) + axis_shift((code >> 2) & 3, bx.L);
                const double tz = ((double)hp.z - (double)c.z) + axis_shift((code >> 4) & 3, bx.L);
                const double sxy = tx * tx + ty * ty;
                const double r2 = sxy + tz * tz;
                link = lv[a] & (strict ? (r2 < bx.l2) : (r2 <= bx.l2));
            } else {
                float dx, dy, dz;
                if (plain) {
                    dx = hp.x - c.x;
                    dy = hp.y - c.y;
                    dz = hp.z - c.z;
                } else {
                    dx = axis_diff(hp.x, c.x, code & 3, bx.L32);
                    dy = axis_diff(hp.y, c.y, (code >> 2) & 3, bx.L32);
                    dz = axis_diff(hp.z, c.z, (code >> 4) & 3, bx.L32);
                }
                const float rr = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                link = lv[a] & (rr < bx.lo32);
                // the guard band (rare), decided in double; one branch, the
                // compares flat (a NaN lands in the band and fails there)
                if (lv[a] & !(rr < bx.lo32) & !(rr > bx.hi32)) {
                    if (kStats) ++band;
                    link = link_fp64(hp.x, hp.y, hp.z, c.x, c.y, c.z, bx.L, bx.half, bx.l2, strict);
                }
            }
            if (kStats && lv[a]) ++tests;
            if (kStats && link) ++links;
            // a link inside the tile goes to the tile's bit matrix, the others to the edge list
            const unsigned v = (unsigned)(jj[a] - s0);
            const bool local = in_tile && v < 64u;
            if (link && local) {   // both directions: the rows are then the tile's undirected links
                atomicOr(&L.adj[hl], 1ull << v);
                atomicOr(&L.adj[v & 63u], 1ull << hl);
            }
            sink.push(p, link && !local, s0 + hl, jj[a], retries);
        }
    }
}

// The per-particle search by work-group `block` of `blocks`, on this wave's LDS.
template <bool kFP64, bool kStats, bool kInline>
__device__ __forceinline__ void sparse_search(const Plan &p, SparseLds &L, int block, int blocks)
{
    const int wid = threadIdx.x >> 6, lane = lane_id();
    EdgeSink<kInline> sink{L.ebuf, 0};
    unsigned long long tests = 0, links = 0, band = 0;
    unsigned retries = 0;
    // links inside a tile are joined by the search itself (index order only:
    // the hook goes under the smallest slot; not in domain mode, whose links
    // across slabs must go through the boundary list)
    const bool tile_union = p.tile_join != 0 && p.link_random == 0 && p.domains <= 1;
    BoxHint hint;   // consecutive tiles of a wave nearly always lie in one box
    const bool any_dense = p.counters->n_items != 0;
    int hook_x = -1, hook_r = 0, hook_old = 0;   // this lane's last tile hook
    auto check_hook = [&]() {
        if (hook_x >= 0 && hook_old != hook_x) retries += 1 + unite(p.parent, hook_x, hook_r, false, p.find_mode);
        hook_x = -1;
    };
    const int64_t n_tiles = (p.n + 63) / 64;
    // each XCD sweeps one contiguous range of tiles, so the neighbour rows of
    // consecutive tiles are reused from its own L2
    const XcdRange xr = xcd_range(n_tiles, kWaves, wid, block, blocks);
    for (int64_t tile = xr.first; tile < xr.end; tile += xr.stride) {
        // a tile whose slots all lie in dense cells has nothing to search here
        // (slots past the end count as dense)
        if (any_dense) {
            const int64_t left = p.n - tile * 64;
            const unsigned long long dm = p.tile_dense[tile] | (left < 64 ? ~0ull << left : 0ull);
            if (dm == ~0ull) continue;
        }
        const int64_t s64 = tile * 64 + lane;
        Span R[kMaxRanges];   // own cell, next cell, then two per neighbour row
        float4 pi = make_float4(0.f, 0.f, 0.f, 0.f);
        int b = 0;
        bool simple = true;
        if (s64 < p.n) {
            const int s = (int)s64;
            b = p.n_boxes == 1 ? 0 : find_box_hint(p.box_p0, p.n_boxes, s64, hint);
            const BoxDev &bd = box_of(p, b);
            pi = p.sorted[s];
            const int nc = bd.nc;
            const int cx = cell_coord(pi.x, bd.inv_h, nc);
            const int cy = cell_coord(pi.y, bd.inv_h, nc);
            const int cz = cell_coord(pi.z, bd.inv_h, nc);
            const int64_t c = bd.cell_base + ((int64_t)cz * nc + cy) * nc + cx;
            const int *cst = p.cstart;
            const int dense_min = p.dense_min;
            const int seg_shift = p.seg_shift;
            // Boundaries of the own row and the four neighbour rows (dy, dz) =
            // (1, 0), (-1, 1), (0, 1), (1, 1): with the own cell these hold the
            // 13 half-shell cells. Occupancy words (bits and rank base per 32
            // cells, a small array that stays in cache) give the rank of each
            // cell among the occupied ones, and cstart the boundaries.
            const uint2 *occ = p.occ;
            typedef unsigned uint4a8 __attribute__((ext_vector_type(4), aligned(8)));
            typedef int int4a4 __attribute__((ext_vector_type(4), aligned(4)));
            auto rank_in = [](unsigned bits, unsigned base, int64_t cell_index) {
                return (int)base + __popc(bits & ((1u << ((unsigned)cell_index & 31u)) - 1u));
            };
            auto span = [&](int64_t cell_index, int &s0, int &s1) {   // left at 0, 0 for an empty cell
                const uint2 w = occ[cell_index >> 5];
                if ((w.x >> ((unsigned)cell_index & 31u)) & 1u) {
                    const int r = rank_in(w.x, w.y, cell_index);
                    s0 = cst[r];
                    s1 = cst[r + 1];
                }
            };
            const int nxp = cx + 1 < nc ? cx + 1 : 0;
            const bool inner = cx >= 1 && cx + 1 < nc;
            const int rdy[4] = {1, -1, 0, 1}, rdz[4] = {0, 1, 1, 1};
            int64_t c0[4];
            int yz[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int ny = cy + rdy[r], nz = cz + rdz[r], code = 0;
                if (ny >= nc) { ny -= nc; code |= 2 << 2; }
                else if (ny < 0) { ny += nc; code |= 1 << 2; }
                if (nz >= nc) { nz -= nc; code |= 2 << 4; }
                yz[r] = code;
                c0[r] = bd.cell_base + ((int64_t)nz * nc + ny) * nc + (inner ? cx - 1 : 0);
            }
            // Two rounds of loads, each issued whole before any of its results
            // is used, with no branch among them: first the occupancy words of
            // the own cell and of each row (two words each, so cells across a
            // word boundary are covered), then, from the ranks, one 16-byte
            // read of cell starts for the own cell and for each row. Every
            // address is in range whatever the bits: a rank is at most n and
            // cstart has n + 4 entries; a word index is at most the last one
            // plus one, inside the two words of padding.
            const uint4a8 wo = *reinterpret_cast<const uint4a8 *>(occ + (c >> 5));
            uint4a8 wr[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) wr[r] = *reinterpret_cast<const uint4a8 *>(occ + (c0[r] >> 5));
            const int4a4 qo = *reinterpret_cast<const int4a4 *>(cst + rank_in(wo.x, wo.y, c));   // the own cell holds s
            int4a4 qr[4];
            unsigned mr[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                mr[r] = (unsigned)((((uint64_t)wr[r].x | ((uint64_t)wr[r].z << 32)) >> ((unsigned)c0[r] & 31u)) & 7u);
                qr[r] = *reinterpret_cast<const int4a4 *>(cst + rank_in(wr[r].x, wr[r].y, c0[r]));
            }
            const int own_start = qo.x, own_end = qo.y;
            // The plain case: no row wraps at an x face or crosses a segment,
            // so its cells follow each other and their bounds are in the 16
            // bytes already loaded: one range per row, two around a dense
            // middle cell. What it leaves out is most of a tile's setup, which
            // is bound by instruction issue.
            const bool searches = own_end - own_start < dense_min;   // dense cells are searched elsewhere
            simple = inner && !p.sample && ((c ^ (c + 1)) >> seg_shift) == 0;
            {
                const unsigned b1 = (unsigned)(c + 1) & 31u;
                const bool nxt = (((b1 ? wo.x : wo.z) >> b1) & 1u) && qo.z - qo.y < dense_min;
                R[0] = Span{s + 1, searches ? (nxt ? qo.z : qo.y) : 0, 0};
            }
            bool crowded = false;   // some row may hold a dense cell
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int4a4 q = qr[r];
                const unsigned occupied = __popc(mr[r]);
                const int end = occupied == 0 ? q.x : (occupied == 1 ? q.y : (occupied == 2 ? q.z : q.w));
                simple = simple && ((c0[r] ^ (c0[r] + 2)) >> seg_shift) == 0;
                crowded = crowded || end - q.x >= dense_min;
                R[2 + 2 * r] = Span{q.x, searches ? end : 0, yz[r]};
            }
            simple = simple || !searches;
            if (__ballot(crowded && searches && simple)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int4a4 q = qr[r];
                    const unsigned o1 = mr[r] & 1u, o2 = o1 + ((mr[r] >> 1) & 1u);
                    const int b1 = o1 ? q.y : q.x, b2 = o2 == 0 ? q.x : (o2 == 1 ? q.y : q.z);
                    const int b3 = R[2 + 2 * r].j1;   // below the row's start for a lane that does not search
                    const bool d0 = b1 - q.x >= dense_min, d1 = b2 - b1 >= dense_min, d2 = b3 - b2 >= dense_min;
                    const int end = d2 ? b2 : b3;
                    R[2 + 2 * r].j0 = d0 ? b1 : q.x;
                    R[2 + 2 * r].j1 = d1 ? min(b1, b3) : end;
                    R[3 + 2 * r] = Span{b2, d1 ? end : 0, yz[r]};
                }
            }
            // Lanes at an x face, of a row across segments, or of the first
            // pass of the giant-component skip (centre cells of the axis
            // neighbours (dy, dz) = (1, 0) and (0, 1) only): cell by cell.
            if (!simple) {
                int st[3], en[3];
                st[0] = en[0] = 0;
                span(c - cx + nxp, st[0], en[0]);
                R[0] = Span{s + 1, own_end, 0};
                R[1] = en[0] - st[0] < dense_min ? Span{st[0], en[0], cx + 1 < nc ? 0 : 2} : Span{};
                const int xcode[3] = {cx == 0 ? 1 : 0, 0, cx + 1 == nc ? 2 : 0};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    int ny = cy + rdy[r], nz = cz + rdz[r];
                    ny += ny >= nc ? -nc : (ny < 0 ? nc : 0);
                    nz += nz >= nc ? -nc : 0;
                    const int64_t row = bd.cell_base + ((int64_t)nz * nc + ny) * nc;
#pragma unroll
                    for (int e = 0; e < 3; ++e) {
                        int nx = cx - 1 + e;
                        nx += nx < 0 ? nc : (nx >= nc ? -nc : 0);
                        st[e] = en[e] = 0;
                        if (!p.sample || ((r == 0 || r == 2) && e == 1)) span(row + nx, st[e], en[e]);
                    }
                    const int code = R[2 + 2 * r].code;
                    R[2 + 2 * r] = R[3 + 2 * r] = Span{};
                    row_spans(st, en, xcode, code, dense_min, R[2 + 2 * r], R[3 + 2 * r]);
                }
            }
        }
        // flatten the units of the wave: unit and pair offsets by prefix sums
        // (mostly every other range is empty in all lanes)
        bool more = false;
#pragma unroll
        for (int r = 1; r < kMaxRanges; r += 2) more = more || R[r].j1 > R[r].j0;
        const bool all_simple = __ballot(more) == 0;
        int my_pairs = 0, my_units = 0;
        auto add_up = [&](const Span &x) {
            const int len = max(x.j1 - x.j0, 0);
            my_pairs += len;
            my_units += len > 0 ? 1 : 0;
        };
#pragma unroll
        for (int r = 0; r < kMaxRanges; r += 2) add_up(R[r]);
        if (!all_simple) {
#pragma unroll
            for (int r = 1; r < kMaxRanges; r += 2) add_up(R[r]);
        }
        const int unit_incl = wave_incl_scan(my_units);
        const int pair_incl = wave_incl_scan(my_pairs);
        const int n_units = __builtin_amdgcn_readlane(unit_incl, 63);
        const int n_pairs = __builtin_amdgcn_readlane(pair_incl, 63);
        if (n_pairs == 0) continue;
        {
            int u = unit_incl - my_units, pr = pair_incl - my_pairs;
            auto put = [&](const Span &x) {
                if (x.j1 > x.j0) {
                    L.unit[u] = make_int2(pr, x.j0);
                    L.tag[u] = x.code | (lane << 8);
                    pr += x.j1 - x.j0;
                    ++u;
                }
            };
#pragma unroll
            for (int r = 0; r < kMaxRanges; r += 2) put(R[r]);
            if (!all_simple) {
#pragma unroll
                for (int r = 1; r < kMaxRanges; r += 2) put(R[r]);
            }
            if (lane == 63) L.unit[n_units].x = n_pairs;
            L.home[lane] = pi;
        }
        __builtin_amdgcn_wave_barrier();
        check_hook();
        L.adj[lane] = 0ull;
        __builtin_amdgcn_wave_barrier();
        // a tile inside one box keeps that box's parameters in registers for
        // every pair; otherwise each pair reads the box of its home particle
        const int s0 = (int)(tile * 64);
        const int b0 = __builtin_amdgcn_readfirstlane(b);
        if (__ballot(b != b0) == 0)
            sparse_pairs<kFP64, kStats, true, kInline>(p, L, sink, s0, n_units, n_pairs, b, BoxPair::of(box_of(p, b0)),
                                              tile_union, tests, links, band, retries);
        else
            sparse_pairs<kFP64, kStats, false, kInline>(p, L, sink, s0, n_units, n_pairs, b, BoxPair{}, tile_union, tests,
                                               links, band, retries);
        __builtin_amdgcn_wave_barrier();
        if (tile_union) {
            // The components of the links inside the tile, by Warshall's
            // closure over the rows of the bit matrix (one per lane): row u
            // starts as u's links and u itself; for each slot k with links,
            // every row that holds k takes in row k. Afterwards row u is u's
            // component, and its lowest bit the component's smallest slot,
            // the node of smallest hooking key, under which u is hooked.
            // A particle may have been hooked by then: with kInline the waves
            // merge their pairs all through the search, otherwise only where
            // a full edge-list slice made a search merge its surplus at once.
            // So the hook is a compare-and-swap, and one that finds its slot
            // hooked already becomes an ordinary union.
            const unsigned long long tile_links = L.adj[lane];
            const unsigned long long todo = __ballot(tile_links != 0ull);
            if (todo) {
                const unsigned long long row = close_rows(tile_links | (1ull << lane), todo);
                const int r = __ffsll((long long)row) - 1;
                if (r != lane) {   // read back with the next tile, so the wave does not wait for it
                    hook_x = s0 + lane;
                    hook_r = s0 + r;
                    hook_old = atomicCAS(p.parent + hook_x, hook_x, hook_r);
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
    check_hook();
    sink.flush(p, retries);
    if (kStats) {
        tests = wave_sum_u64(tests);
        links = wave_sum_u64(links);
        band = wave_sum_u64(band);
        unsigned long long r = wave_sum_u64((unsigned long long)retries);
        if (lane == 0) {
            atomicAdd(&p.counters->sparse_tests, tests);
            atomicAdd(&p.counters->pair_tests, tests);
            atomicAdd(&p.counters->links, links);
            atomicAdd(&p.counters->band_hits, band);
            atomicAdd(&p.counters->cas_retries, r);
        }
    }
}

template <bool kFP64, bool kStats>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) k_link_sparse(Plan p)
{
    __shared__ SparseLds lds[kWaves];
    sparse_search<kFP64, kStats, false>(p, lds[threadIdx.x >> 6], blockIdx.x, gridDim.x);
}

constexpr int kUnionIlp = 4;   // queued pairs a lane merges at once
constexpr int kUnionChunk = kBlock * kUnionIlp;
constexpr int kUnionSlots = 4096;   // of the table of a chunk's roots, at most half filled
constexpr int kUnionRounds = 16;
static_assert(kUnionSlots >= 4 * kUnionChunk, "at most 2 roots per pair, and room to probe");

// Merges the queued pairs, no ordering needed. A work-group takes chunks of
// kUnionChunk consecutive pairs; the finds of a lane's 2 kUnionIlp end points
// advance together. Consecutive pairs come from the same few tiles, so many of
// them name the same roots: swapped one by one, as many swaps failed as there
// were pairs (each then a chain of finds of its own). So the chunk's roots go
// into a table in LDS, each takes the smallest root it is joined to there (the
// smaller label of every pair, until nothing changes), and each distinct root
// is hooked under its label by one compare-and-swap; one that finds the root
// moved goes on as an ordinary union, and so do pairs whose labels had not
// met after kUnionRounds rounds. 2.1e6 clustered particles (0.49M pairs) 91 ->
// 48 us, 256 boxes (15.8M) 0.80 -> 0.37 ms, 2.1e6 lattice sites, where all
// swaps meet on a few roots, 345 -> 194 .. 266 us with where the forest lies in
// memory (beside 194: 2 pairs per lane 60 us, 0.36 ms, 320 us; 8: 58, 0.42,
// 168).
// Slice s holds the pairs found on XCD s % 8 (the search's work-group b
// appends to slice b % 256, and work-groups go to XCDs round-robin), whose
// home particles are that XCD's contiguous range of cells; its kUnionParts
// work-groups run on the same XCD, so the finds of a slice stay in one L2.
// Domain mode and the depth-2 compression take the plain path, one pair at a
// time.
constexpr int kUnionParts = 16;
static_assert(kEdgeSlices % kXcds == 0, "slices split evenly over the XCDs");

// kRandom: randomised link order, whose labels compare by priority.
template <bool kStats, bool kRandom>
__global__ void __launch_bounds__(kBlock) k_union_edges(Plan p)
{
    using Label = std::conditional_t<kRandom, unsigned long long, int>;
    auto label_of = [](int x) {
        if constexpr (kRandom) return ((unsigned long long)link_key(x, true) << 32) | (unsigned)x;
        else return x;
    };
    auto node_of = [](Label l) { return (int)(unsigned)l; };
    const int xcd = blockIdx.x % kXcds, g = blockIdx.x / kXcds;
    const int slice = (g % (kEdgeSlices / kXcds)) * kXcds + xcd;
    const int part = g / (kEdgeSlices / kXcds);
    const int64_t cap = p.max_edges / kEdgeSlices;
    const unsigned fill = p.edge_fill[slice];
    const int64_t ne = (int64_t)fill < cap ? (int64_t)fill : cap;
    const int2 *edges = p.edges + slice * cap;
    unsigned retries = 0;
    if (p.domains > 1 || p.find_mode != 0) {
        const int64_t stride = (int64_t)kUnionParts * kBlock;
        for (int64_t k = (int64_t)part * kBlock + threadIdx.x; k < ne; k += stride) {
            const int2 e = edges[k];
            merge_pair(p, e.x, e.y, retries);
        }
    } else if ((int64_t)part * kUnionChunk < ne) {
        __shared__ int root[kUnionSlots];
        __shared__ Label label[kUnionSlots];
        __shared__ int moved[2];
        for (int k = threadIdx.x; k < kUnionSlots; k += kBlock) root[k] = -1;
        if (threadIdx.x < 2) moved[threadIdx.x] = 0;
        __syncthreads();
        for (int64_t c0 = (int64_t)part * kUnionChunk; c0 < ne; c0 += (int64_t)kUnionParts * kUnionChunk) {
            int x[2 * kUnionIlp], at[2 * kUnionIlp];
            bool done[2 * kUnionIlp];
            unsigned owned = 0u;   // end points whose table entry this lane made
#pragma unroll
            for (int u = 0; u < kUnionIlp; ++u) {
                const int64_t k = c0 + u * kBlock + threadIdx.x;
                const bool in = k < ne;
                const int2 e = in ? edges[k] : make_int2(0, 0);
                x[2 * u] = e.x;
                x[2 * u + 1] = e.y;
                done[2 * u] = done[2 * u + 1] = !in;
            }
            find_many<2 * kUnionIlp>(p.parent, x, done);
#pragma unroll
            for (int v = 0; v < 2 * kUnionIlp; ++v) {
                at[v] = -1;
                if (x[v] == x[v ^ 1]) continue;   // in one group already (or past the end)
                int h = (int)(((unsigned)x[v] * 0x9e3779b9u) >> (32 - 12));
                while (true) {
                    const int old = atomicCAS(&root[h], -1, x[v]);
                    if (old == -1) {
                        label[h] = label_of(x[v]);
                        owned |= 1u << v;
                    }
                    if (old == -1 || old == x[v]) break;
                    h = (h + 1) & (kUnionSlots - 1);
                }
                at[v] = h;
            }
            __syncthreads();
            for (int round = 0; round < kUnionRounds; ++round) {
                bool any = false;
#pragma unroll
                for (int u = 0; u < kUnionIlp; ++u) {
                    const int i = at[2 * u], j = at[2 * u + 1];
                    if (i < 0) continue;
                    const Label li = __hip_atomic_load(&label[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    const Label lj = __hip_atomic_load(&label[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (li == lj) continue;
                    atomicMin(li > lj ? &label[i] : &label[j], min(li, lj));
                    any = true;
                }
                if (any) moved[round & 1] = 1;
                __syncthreads();
                const bool again = moved[round & 1] != 0;
                if (threadIdx.x == 0) moved[(round & 1) ^ 1] = 0;   // read by no one before the next barrier
                if (!again) break;
                __syncthreads();
            }
            // hooks of the owned roots, their swaps in flight together
            int got[2 * kUnionIlp], to[2 * kUnionIlp];
#pragma unroll
            for (int v = 0; v < 2 * kUnionIlp; ++v) {
                got[v] = x[v];
                to[v] = (owned >> v) & 1u ? node_of(label[at[v]]) : x[v];
            }
            bool rest[kUnionIlp];
#pragma unroll
            for (int u = 0; u < kUnionIlp; ++u)
                rest[u] = at[2 * u] >= 0 && label[at[2 * u]] != label[at[2 * u + 1]];
#pragma unroll
            for (int v = 0; v < 2 * kUnionIlp; ++v)
                if (to[v] != x[v])
                    __hip_atomic_compare_exchange_strong(p.parent + x[v], &got[v], to[v], __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();   // every label read
#pragma unroll
            for (int v = 0; v < 2 * kUnionIlp; ++v)
                if ((owned >> v) & 1u) root[at[v]] = -1;
            if (threadIdx.x < 2) moved[threadIdx.x] = 0;
            __syncthreads();
#pragma unroll
            for (int v = 0; v < 2 * kUnionIlp; ++v)
                if (got[v] != x[v]) retries += 1 + unite(p.parent, got[v], to[v], kRandom);
#pragma unroll
            for (int u = 0; u < kUnionIlp; ++u)
                if (rest[u]) retries += unite(p.parent, x[2 * u], x[2 * u + 1], kRandom);
        }
    }
    if (kStats) {
        unsigned long long r = wave_sum_u64((unsigned long long)retries);
        if (lane_id() == 0 && r) atomicAdd(&p.counters->cas_retries, r);
        // queued pairs, for the statistics
        if (part == 0 && threadIdx.x == 0) atomicAdd(&p.counters->n_edges, fill);
    }
}

// ---------------------------------------------------------- dense (wave) --
//
// One work item = up to 64 particles of a dense cell, one per lane ("home"
// particles). Candidates are staged in LDS, 64 at a time, and every staged
// candidate is tested against all home lanes at once (its LDS address is
// uniform, so the read is a broadcast). A stage is filled from a list of
// candidate ranges (the cell itself, or several neighbour cells at once), so
// that small neighbour cells do not each cost a round of loads:
//  - the cell itself (only candidates above the home particle count);
//  - every neighbour cell the item searches (the upper half shell, and the
//    lower half where the neighbour is sparse) whose periodic image needs no
//    shift of the home coordinate, together in one list;
//  - FP32 only: each neighbour reached across a high face of the box, where
//    the home coordinate is shifted by -L (exact there), on its own.
// When every home lane knows the same root, candidates of that root are
// already in their group and are dropped while the stage is filled.

struct StageF {
    float4 v[64];            // x, y, z (candidate-side periodic shift applied), cached root (bits)
    int slot[64];            // sorted slot of the candidate
};

struct StageD {
    double x[64], y[64], z[64];
    double sx[64], sy[64], sz[64];   // periodic shift, added after the rounded difference
    int root[64];
    int slot[64];
};

template <bool kFP64>
struct Stage;
template <>
struct Stage<false> {
    using T = StageF;
};
template <>
struct Stage<true> {
    using T = StageD;
};

// Candidate ranges of one stage fill: range r covers slots
// [j0[r], j0[r] + pre[r + 1] - pre[r]) with periodic shift code code[r]
// (bits 0-1, 2-3, 4-5 for x, y, z: 1 = the neighbour is the top cell across
// the low face, its FP32 coordinate minus L is exact; 2 = the neighbour lies
// across the high face, handled on the home side in FP32). In double the
// shift (+L for 1, -L for 2) is added after the rounded difference.
struct RangeList {
    int pre[28];
    int j0[27];
    int code[27];
};

// Box parameters the inner loops need, held in registers.
struct BoxRegs {
    double L, half, l2;
    float lo32, hi32, L32;
    bool strict;
};

// The slow path of one staged candidate kk for the lanes in `cand`: an FP32
// result below lo32 links; one inside the band is re-decided in double from
// the original coordinates; a link merges the groups unless they are already
// known to be one. kGeneral: domain mode (a link across slabs goes to the
// boundary list) and randomised linking, decided at run time; the plain
// instance has neither, which keeps its registers and code size down.
//
// Known roots: root_i is the root last seen for the home particle; known0
// and known1 are two more nodes of its group (the two roots of its last
// merge). A candidate whose cached root is any of them is in the group
// already (groups only grow), so the pair needs no union whatever its
// distance. Without statistics the caller drops such candidates before the
// distance decides anything.
template <bool kFP64, bool kStats, bool kGeneral>
__device__ __forceinline__ void dense_hit(const Plan &p, const BoxRegs &br, const typename Stage<kFP64>::T &st,
                                          int kk, bool cand, float r, float4 pi, int &root_i, int &known0,
                                          int &known1, unsigned long long &links, unsigned long long &band,
                                          unsigned &retries)
{
    if (!cand) return;
    const int j = st.slot[kk];
    bool link = true;
    if constexpr (!kFP64) {
        if (!(r < br.lo32)) {
            if (kStats) ++band;
            const float4 oj = p.sorted[j];
            link = link_fp64(pi.x, pi.y, pi.z, oj.x, oj.y, oj.z, br.L, br.half, br.l2, br.strict);
        }
    }
    if (link) {
        if (kStats) ++links;
        int rj;
        if constexpr (kFP64) rj = st.root[kk];
        else rj = __float_as_int(st.v[kk].w);
        if (rj != root_i && rj != known0 && rj != known1) {
            if (kGeneral && p.domains > 1 && domain_of(p, j) != slab_of(pi.x, p.domains, br.L)) {
                defer_boundary(p, root_i, rj, retries);
            } else {
                const int old = root_i;
                root_i = unite_root(p.parent, root_i, rj, kGeneral && p.link_random, p.find_mode, retries);
                known0 = rj;
                known1 = old;
            }
        }
    }
}

// FP32 squared distance of the home lane to a staged candidate.
__device__ __forceinline__ float dist2_f32(const float4 cj, float hx, float hy, float hz)
{
    const float dx = hx - cj.x, dy = hy - cj.y, dz = hz - cj.z;
    return fmaf(dz, dz, fmaf(dy, dy, dx * dx));
}

// The double predicate of the home lane and staged candidate kk, with the
// candidate's periodic shift added after the rounded difference.
__device__ __forceinline__ bool link_f64_staged(const StageD &st, int kk, double dxi, double dyi, double dzi,
                                                const BoxRegs &br)
{
    const double tx = (dxi - st.x[kk]) + st.sx[kk];
    const double ty = (dyi - st.y[kk]) + st.sy[kk];
    const double tz = (dzi - st.z[kk]) + st.sz[kk];
    const double sxy = tx * tx + ty * ty;
    const double r2 = sxy + tz * tz;
    return br.strict ? (r2 < br.l2) : (r2 <= br.l2);
}

// Tests the staged candidates [0, cnt) against the wave's home particles.
// An item of at most 32 (or 16) home particles holds copies of them in both
// halves (all four quarters) of the wave: lane l is home particle l % H and
// tests candidate kk + l / H, so one step tests G = 64 / H candidates.
// kSelf: the candidates come from the home cell; only slots above the home
// particle's count. Without statistics a candidate whose cached root is
// known to be in the home particle's group is dropped together with the
// distance test's verdict.
template <bool kFP64, bool kStats, bool kGeneral, bool kSelf>
__device__ __forceinline__ void dense_batch(const Plan &p, const BoxRegs &br, const typename Stage<kFP64>::T &st,
                                            int cnt, int G, int q, int i, bool vi, float4 pi, float hx, float hy,
                                            float hz, double dxi, double dyi, double dzi, int &root_i, int &known0,
                                            int &known1, unsigned long long &links, unsigned long long &band,
                                            unsigned &retries)
{
    // non-short-circuit forms: the compares run flat, with no branch around them
    auto fresh = [&](int rj) { return kStats || ((rj != root_i) & (rj != known0)); };
    int kk = 0;
    if constexpr (!kFP64) {
        const int G4 = 4 * G;
        for (; kk + G4 <= cnt; kk += G4) {
            const int k0 = kk + q, k1 = k0 + G, k2 = k1 + G, k3 = k2 + G;
            const float4 q0 = st.v[k0], q1 = st.v[k1], q2 = st.v[k2], q3 = st.v[k3];
            const float r0 = dist2_f32(q0, hx, hy, hz);
            const float r1 = dist2_f32(q1, hx, hy, hz);
            const float r2 = dist2_f32(q2, hx, hy, hz);
            const float r3 = dist2_f32(q3, hx, hy, hz);
            bool c0 = (r0 <= br.hi32) & fresh(__float_as_int(q0.w));
            bool c1 = (r1 <= br.hi32) & fresh(__float_as_int(q1.w));
            bool c2 = (r2 <= br.hi32) & fresh(__float_as_int(q2.w));
            bool c3 = (r3 <= br.hi32) & fresh(__float_as_int(q3.w));
            if constexpr (kSelf) {
                c0 = c0 & (st.slot[k0] > i);
                c1 = c1 & (st.slot[k1] > i);
                c2 = c2 & (st.slot[k2] > i);
                c3 = c3 & (st.slot[k3] > i);
            }
            if (__ballot(c0 || c1 || c2 || c3)) {
                dense_hit<kFP64, kStats, kGeneral>(p, br, st, k0, c0, r0, pi, root_i, known0, known1, links, band,
                                                   retries);
                dense_hit<kFP64, kStats, kGeneral>(p, br, st, k1, c1, r1, pi, root_i, known0, known1, links, band,
                                                   retries);
                dense_hit<kFP64, kStats, kGeneral>(p, br, st, k2, c2, r2, pi, root_i, known0, known1, links, band,
                                                   retries);
                dense_hit<kFP64, kStats, kGeneral>(p, br, st, k3, c3, r3, pi, root_i, known0, known1, links, band,
                                                   retries);
            }
        }
    }
    for (; kk < cnt; kk += G) {
        const int k = kk + q;
        const bool in = k < cnt;
        const int kr = in ? k : 0;   // a valid stage entry for lanes past the end
        bool c;
        float r = 0.f;
        if constexpr (kFP64) {
            c = in && vi && fresh(st.root[kr]) && link_f64_staged(st, kr, dxi, dyi, dzi, br);
        } else {
            const float4 cq = st.v[kr];
            r = dist2_f32(cq, hx, hy, hz);
            c = in && r <= br.hi32 && fresh(__float_as_int(cq.w));   // false for invalid (NaN) lanes
        }
        if constexpr (kSelf) c = c && st.slot[kr] > i;
        if (__ballot(c))
            dense_hit<kFP64, kStats, kGeneral>(p, br, st, kr, c, r, pi, root_i, known0, known1, links, band, retries);
    }
}

// Tests the staged candidates [0, cnt) against the wave's home particles, in
// the copies of dense_batch, and merges the groups of the linked pairs once
// for the whole stage. While testing, a home lane gathers in `row` the home
// particles that share a linked candidate with it (the ballot of a candidate's
// links is their set), and lane c in `cand` the home particles linked to
// candidate c. Then every set of joined home particles (one, when they are one
// group already; otherwise the closure of the rows) takes the smallest root
// among its own and its candidates' as target, and each of the other roots is
// hooked under it, all in parallel: one round of compare-and-swaps per stage,
// where merging at every hit was a chain of finds and swaps for each group
// met. A swap that fails (its root has been hooked meanwhile) goes on as an
// ordinary union. The target is smaller than every node hooked under it, so
// the forest stays valid even when it is no root any more. 256 boxes (232k
// items): the kernel 1.10 -> 0.86 ms; 3.3e4 clustered particles 43 -> 27 us.
template <bool kFP64, bool kSelf>
__device__ __forceinline__ void dense_join(const Plan &p, const BoxRegs &br, typename Stage<kFP64>::T &st, int cnt,
                                           int H, int G, int q, int i, bool vi, float4 pi, float hx, float hy,
                                           float hz, double dxi, double dyi, double dzi, int &root_i,
                                           unsigned &retries)
{
    const int lane = lane_id();
    const unsigned long long copy = H == 64 ? ~0ull : (1ull << H) - 1ull;
    unsigned long long row = 0ull, cand = 0ull;
    auto take = [&](int kk, bool link) {
        const unsigned long long m = __ballot(link);
        if (!m) return;
        if (H == 64) {
            row |= link ? m : 0ull;
            cand = lane == kk ? m : cand;
        } else {
            const int d = lane - kk;
            row |= link ? (m >> (q * H)) & copy : 0ull;
            cand = (unsigned)d < (unsigned)G ? (m >> (d * H)) & copy : cand;
        }
    };
    auto in_band = [&](int k, float r) {   // decided in double
        bool link = r < br.lo32;
        const bool band = !(r < br.lo32) & (r <= br.hi32);
        if (__ballot(band)) {
            if (band) {
                const float4 oj = p.sorted[st.slot[k]];
                link = link_fp64(pi.x, pi.y, pi.z, oj.x, oj.y, oj.z, br.L, br.half, br.l2, br.strict);
            }
        }
        return link;
    };
    int kk = 0;
    if constexpr (!kFP64) {
        const int G4 = 4 * G;
        for (; kk + G4 <= cnt; kk += G4) {
            float r[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) r[u] = dist2_f32(st.v[kk + u * G + q], hx, hy, hz);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = kk + u * G + q;
                bool link = in_band(k, r[u]);
                if constexpr (kSelf) link = link & (st.slot[k] > i);
                take(kk + u * G, link);
            }
        }
    }
    for (; kk < cnt; kk += G) {
        const bool in = kk + q < cnt;
        const int k = in ? kk + q : 0;   // a valid stage entry for lanes past the end
        bool link;
        if constexpr (kFP64) link = vi && link_f64_staged(st, k, dxi, dyi, dzi, br);
        else link = in_band(k, dist2_f32(st.v[k], hx, hy, hz));   // false for invalid (NaN) lanes
        link = link & in;
        if constexpr (kSelf) link = link & (st.slot[k] > i);
        take(kk, link);
    }
    if (__ballot((row | cand) != 0ull) == 0) return;
    if (H <= 32) row |= __shfl_xor(row, 32, 64);
    if (H <= 16) row |= __shfl_xor(row, 16, 64);
    int lead = 0;   // first home lane of this lane's set (copies agree)
    const int rh = __builtin_amdgcn_readfirstlane(root_i);
    if (__ballot(vi && root_i != rh)) {
        const int h = lane & (H - 1);
        row |= 1ull << h;
        row = close_rows(row, __ballot(row != (1ull << h)) & copy);
        lead = __ffsll((long long)row) - 1;
    }
    int rj = INT_MAX;
    if (lane < cnt) {
        if constexpr (kFP64) rj = st.root[lane];
        else rj = __float_as_int(st.v[lane].w);
    }
    const bool linked = cand != 0ull;   // candidate `lane`
    const int lead_c = __shfl(lead, linked ? __ffsll((long long)cand) - 1 : 0, 64);
    int *target = st.slot;   // the candidates' slots are no longer needed
    __builtin_amdgcn_wave_barrier();
    target[lane] = INT_MAX;
    __builtin_amdgcn_wave_barrier();
    if (vi && lane < H) atomicMin(&target[lead], root_i);
    if (linked) atomicMin(&target[lead_c], rj);
    __builtin_amdgcn_wave_barrier();
    const int th = vi ? target[lead] : root_i, tc = linked ? target[lead_c] : rj;
    // one lane per root: the set's first lane and the lanes of other roots; of
    // neighbouring candidates of one root (a cell's are consecutive) the first
    const int lead_root = __shfl(root_i, lead, 64);
    const int before_root = __shfl_up(rj, 1, 64), before_lead = __shfl_up(linked ? lead_c : -1, 1, 64);
    const bool hook_h = vi && lane < H && root_i != th && (lane == lead || root_i != lead_root);
    const bool hook_c = linked && rj != tc && !(lane > 0 && before_root == rj && before_lead == lead_c);
    int got_h = root_i, got_c = rj;
    if (hook_h)
        __hip_atomic_compare_exchange_strong(p.parent + root_i, &got_h, th, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    if (hook_c)
        __hip_atomic_compare_exchange_strong(p.parent + rj, &got_c, tc, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    if (hook_h && got_h != root_i) retries += 1 + unite(p.parent, got_h, th, false, p.find_mode);
    if (hook_c && got_c != rj) retries += 1 + unite(p.parent, got_c, tc, false, p.find_mode);
    root_i = th;
}

// Fills stages from the ranges in `rl` (lane l < 27 holds range l's length
// in `len`, its first slot in `j0`, its shift code in `code`) and tests them
// against the home lanes (home coordinates hx, hy, hz, already shifted where
// the group needs it).
template <bool kFP64, bool kStats, bool kGeneral, bool kSelf>
__device__ __forceinline__ void dense_ranges(const Plan &p, const BoxRegs &br, typename Stage<kFP64>::T &st,
                                             RangeList &rl, int len, int j0, int code, int G, int q, int i, bool vi,
                                             float4 pi, float hx, float hy, float hz, int n_home, int &root_i,
                                             int &known0,
                                             int &known1, unsigned long long &tests, unsigned long long &links,
                                             unsigned long long &band, unsigned &retries)
{
    const int lane = lane_id();
    const int incl = wave_incl_scan(lane < 27 ? len : 0);
    const int total = __shfl(incl, 63, 64);
    if (total == 0) return;
    if (lane < 27) {
        rl.pre[lane + 1] = incl;
        rl.j0[lane] = j0;
        rl.code[lane] = code;
    }
    if (lane == 0) rl.pre[0] = 0;
    __builtin_amdgcn_wave_barrier();
    const bool rnd = kGeneral && p.link_random;
    const double dxi = (double)pi.x, dyi = (double)pi.y, dzi = (double)pi.z;
#pragma unroll 1
    for (int t0 = 0; t0 < total; t0 += 64) {
        const int t = t0 + lane;
        const bool vj = t < total;
        int r = 0;
        if (vj) {
#pragma unroll
            for (int step = 16; step > 0; step >>= 1)
                if (r + step < 27 && rl.pre[r + step] <= t) r += step;
        }
        const int j = vj ? rl.j0[r] + (t - rl.pre[r]) : 0;
        const int cj = vj ? rl.code[r] : 0;
        const float4 cq = vj ? p.sorted[j] : make_float4(qnan(), qnan(), qnan(), 0.f);
        // the home particle's cached root, checked once per stage fill
        // (other waves may have merged its group meanwhile)
        const int pr = (!kStats && vi) ? ld_rel(p.parent + root_i) : root_i;
        const int rj = vj ? find_root(p.parent, j, p.find_mode, rnd) : -2;
        bool keep = vj;
        if constexpr (!kStats) {
            if (pr != root_i) root_i = find_root(p.parent, pr, p.find_mode, rnd);
            // one root for every home lane: candidates of that root are in its group
            const int rh = __builtin_amdgcn_readfirstlane(root_i);   // lane 0 is a home particle
            if (__ballot(vi && root_i != rh) == 0) keep = keep && rj != rh;
        }
        const unsigned long long km = __ballot(keep);
        const int cnt = __popcll(km);
        if (kStats) tests += (unsigned long long)min(64, total - t0) * (unsigned long long)n_home;
        if (cnt == 0) continue;
        __builtin_amdgcn_wave_barrier();   // the previous stage has been read
        if (keep) {
            const int at = __builtin_amdgcn_mbcnt_hi((unsigned)(km >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)km, 0u));
            st.slot[at] = j;
            if constexpr (kFP64) {
                st.x[at] = (double)cq.x;
                st.y[at] = (double)cq.y;
                st.z[at] = (double)cq.z;
                st.sx[at] = axis_shift(cj & 3, br.L);
                st.sy[at] = axis_shift((cj >> 2) & 3, br.L);
                st.sz[at] = axis_shift((cj >> 4) & 3, br.L);
                st.root[at] = rj;
            } else {
                st.v[at] = make_float4((cj & 3) == 1 ? cq.x - br.L32 : cq.x,
                                       ((cj >> 2) & 3) == 1 ? cq.y - br.L32 : cq.y,
                                       ((cj >> 4) & 3) == 1 ? cq.z - br.L32 : cq.z, __int_as_float(rj));
            }
        }
        __builtin_amdgcn_wave_barrier();
        if constexpr (kStats || kGeneral)
            dense_batch<kFP64, kStats, kGeneral, kSelf>(p, br, st, cnt, G, q, i, vi, pi, hx, hy, hz, dxi, dyi, dzi,
                                                        root_i, known0, known1, links, band, retries);
        else
            dense_join<kFP64, kSelf>(p, br, st, cnt, 64 / G, G, q, i, vi, pi, hx, hy, hz, dxi, dyi, dzi, root_i,
                                     retries);
    }
    __builtin_amdgcn_wave_barrier();   // rl and the stage are reused by the next call
}

constexpr int kMaxSplit = 2;
constexpr int kDenseSample = 16;   // particles of a large one-group neighbour searched first

template <bool kFP64, bool kStats, bool kGeneral>
__global__ void __launch_bounds__(kBlock) k_link_dense(Plan p)
{
    using StageT = typename Stage<kFP64>::T;
    __shared__ StageT stage[kWaves];
    __shared__ RangeList ranges[kWaves];
    const int wid = threadIdx.x >> 6, lane = lane_id();
    StageT &st = stage[wid];
    RangeList &rl = ranges[wid];
    unsigned long long tests = 0, links = 0, band = 0;
    unsigned retries = 0;
    const int n_items = (int)p.counters->n_items;
    // Few items leave most of the grid's waves idle, and each is a chain of
    // dependent loads: an item's neighbours are then split over up to
    // 2^kMaxSplit waves (runs of 1e3 .. 1e5 clustered particles take 3 to 10 %
    // less; over 8 waves 1e4 particles take 10 % more, since more waves merge
    // the same few groups).
    int split = 0;
    while (split < kMaxSplit && ((int64_t)n_items << (split + 1)) <= (int64_t)gridDim.x * kWaves) ++split;
    const XcdRange xr = xcd_range((int64_t)n_items << split, kWaves, wid);   // items come in cell order
    for (int64_t vit = xr.first; vit < xr.end; vit += xr.stride) {
        const int64_t it = vit >> split;
        const int part = (int)vit & ((1 << split) - 1);
        const int4 item = p.items[it];
        const int first = __builtin_amdgcn_readfirstlane(item.x);
        const int rem = __builtin_amdgcn_readfirstlane(item.y) & ~kItemFirst;
        const int ce = first + rem;   // end of the cell
        const int n_home = min(64, rem);
        // home particles per copy (H) and copies (G = 64 / H)
        const int H = n_home > 32 ? 64 : (n_home > 16 ? 32 : 16);
        const int G = 64 / H, q = lane / H;
        const int i = first + (lane & (H - 1));
        const bool vi = i < ce;
        const float4 pi = vi ? p.sorted[i] : make_float4(qnan(), qnan(), qnan(), 0.f);
        const int b = __builtin_amdgcn_readfirstlane(item.z);
        const BoxDev &bd = box_of(p, b);
        const int nc = bd.nc;
        const int64_t cb = bd.cell_base;
        BoxRegs br;
        br.L = bd.L;
        br.half = bd.half;
        br.l2 = bd.l2;
        br.lo32 = bd.lo32;
        br.hi32 = bd.hi32;
        br.L32 = bd.L32;
        br.strict = p.strict != 0;
        // the cell, from its first home particle (lane 0)
        const int cx = cell_coord(lane0(pi.x), bd.inv_h, nc);
        const int cy = cell_coord(lane0(pi.y), bd.inv_h, nc);
        const int cz = cell_coord(lane0(pi.z), bd.inv_h, nc);
        int root_i = vi ? find_root(p.parent, i, p.find_mode, kGeneral && p.link_random) : -1;
        // the 27 neighbour cells, one per lane (lanes 0-26, neighbour
        // nb = 9 (dz + 1) + 3 (dy + 1) + dx + 1), looked up at once; code:
        // per axis 1 = the neighbour is the top cell across the low face,
        // 2 = the home cell is the top one and the neighbour across the high face
        int nb_j0 = 0, nb_j1 = 0, code = 0;
        if (lane < 27) {
            int nx = cx + lane % 3 - 1, ny = cy + (lane / 3) % 3 - 1, nz = cz + lane / 9 - 1;
            if (nx < 0) { nx += nc; code |= 1; } else if (nx >= nc) { nx -= nc; code |= 2; }
            if (ny < 0) { ny += nc; code |= 1 << 2; } else if (ny >= nc) { ny -= nc; code |= 2 << 2; }
            if (nz < 0) { nz += nc; code |= 1 << 4; } else if (nz >= nc) { nz -= nc; code |= 2 << 4; }
            const int2 sp = cell_span(p, cb + ((int64_t)nz * nc + ny) * nc + nx);
            nb_j0 = sp.x;
            nb_j1 = sp.y;
        }
        int known0 = -3, known1 = -3;   // never a node
        // neighbours searched from here: the upper half shell, and the lower
        // half where the neighbour is sparse (a dense one searches the pair)
        const int nlen = nb_j1 - nb_j0;
        bool searched = lane < 27 && lane != 13 && nlen > 0 && (lane > 13 || nlen < p.dense_min) &&
                        (lane & ((1 << split) - 1)) == part;
        int joined = 0;   // what the pre-merge has done: the home cell's flags
        bool one_group = false;   // this lane's neighbour is a dense cell found to be one group
        if constexpr (!kStats) {
            // A dense cell found to be one group leaves nothing to link when
            // its group is the home particles' (all of one group themselves):
            // inside a halo that is nearly every neighbour, and the item ends
            // here instead of staging all their particles.
            const bool flagged = lane < 27 && (lane == 13 || (searched && nlen >= p.dense_min));
            const int fl = flagged ? __float_as_int(p.sorted[nb_j0].w) : 0;
            joined = __builtin_amdgcn_readlane(fl, 13);
            const int rh = __builtin_amdgcn_readfirstlane(root_i);   // lane 0 is a home particle
            one_group = searched && (fl & kCellOneGroup);
            if (__ballot(vi && root_i != rh) == 0 && one_group)
                searched = find_root(p.parent, nb_j0, p.find_mode, kGeneral && p.link_random) != rh;
        }
        const bool home_shift = (code & 0x2a) != 0;   // some axis has code 2
        const bool together = searched && (kFP64 || !home_shift);

        // the cell itself, unless the pre-merge has linked it whole
        if (part == 0 && !(joined & kCellJoined))
            dense_ranges<kFP64, kStats, kGeneral, true>(p, br, st, rl, lane == 13 ? ce - first : 0, first, 0, G, q, i,
                                                        vi, pi, pi.x, pi.y, pi.z, n_home, root_i, known0, known1,
                                                        tests, links, band, retries);
        // Every neighbour that needs no shift of the home coordinate, at once;
        // of a large cell that is one group only the first kDenseSample
        // particles (they are in no particular order): one link joins the two
        // cells, and the rest of it is searched after that only if none of
        // these linked.
        const bool large = together && one_group && nlen > 2 * kDenseSample;
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            int j0 = nb_j0, len = together ? (large ? kDenseSample : nlen) : 0;
            if (pass == 1) {
                if (__ballot(large) == 0) break;
                if (vi) root_i = find_root(p.parent, root_i, p.find_mode, kGeneral && p.link_random);
                const int rh = __builtin_amdgcn_readfirstlane(root_i);
                bool rest = large;
                if (__ballot(vi && root_i != rh) == 0 && large)
                    rest = find_root(p.parent, nb_j0, p.find_mode, kGeneral && p.link_random) != rh;
                j0 = nb_j0 + kDenseSample;
                len = rest ? nlen - kDenseSample : 0;
            }
            dense_ranges<kFP64, kStats, kGeneral, false>(p, br, st, rl, len, j0, code, G, q, i, vi, pi, pi.x, pi.y,
                                                         pi.z, n_home, root_i, known0, known1, tests, links, band,
                                                         retries);
        }
        if constexpr (!kFP64) {
            // neighbours across a high face, one at a time
            unsigned long long rest = __ballot(searched && !together);
            while (rest) {
                const int nb = __ffsll((long long)rest) - 1;
                rest &= rest - 1;
                const int cd = __shfl(code, nb, 64);
                const float hx = (cd & 3) == 2 ? pi.x - br.L32 : pi.x;
                const float hy = ((cd >> 2) & 3) == 2 ? pi.y - br.L32 : pi.y;
                const float hz = ((cd >> 4) & 3) == 2 ? pi.z - br.L32 : pi.z;
                dense_ranges<kFP64, kStats, kGeneral, false>(p, br, st, rl, lane == nb ? nlen : 0, nb_j0, code, G, q,
                                                             i, vi, pi, hx, hy, hz, n_home, root_i, known0, known1,
                                                             tests, links, band, retries);
            }
        }
    }
    if (kStats) {
        links = wave_sum_u64(links);
        band = wave_sum_u64(band);
        unsigned long long r = wave_sum_u64((unsigned long long)retries);
        if (lane == 0) {
            atomicAdd(&p.counters->pair_tests, tests);
            atomicAdd(&p.counters->links, links);
            atomicAdd(&p.counters->band_hits, band);
            atomicAdd(&p.counters->cas_retries, r);
        }
    }
}

// Pre-merge of dense cells (before the pair search), one wavefront per dense
// cell. A cell of at most 64 particles is linked whole in registers
// (cell_rows, close_rows), so the pair search has nothing left to do inside
// it; cells found to be one group are marked, and the pair search passes over
// marked neighbours of the home particles' own group. Both kernels are bound
// by the latency of their dependent loads, so what counts is how few an item
// needs: on 256 boxes of 1e3 to 1e6 particles (232k items) the pre-merge went
// from 0.44 to 0.33 ms, and the pair search from 1.58 to 1.10 ms by what it
// spares there; on 1e5 particles, where a few halo cores were the tail, the
// search from 157 to 54 us. A larger cell is split into k^3 sub-cells small enough that any two
// particles of one sub-cell are linked. When the sub-cells are smaller still (sub_adj:
// any two particles of two sub-cells that touch, across a face, an edge or a
// corner, are linked), every two touching occupied sub-cells are joined: up to
// 64 occupied ones by the closure of their rows of touching ones, more on a
// grid of up to 128 by growing components of one mask, else by a union-find in
// LDS. Every particle is then hooked straight under the particle of highest
// hooking priority (smallest key) of its sub-cell or joined set: only particles joined by chains of linked pairs
// are merged, so the groups are unchanged, and the pair search meets few
// groups per dense cell (its staging drops the candidates of the home
// particles' own group). The particles of dense cells are still their own
// roots when this runs (the per-particle search and its union pass never
// link them) and each dense cell has one wavefront, so the hooks are plain
// stores.
constexpr int kMaxSub = 512;

// Coordinates of sub-cell t on a k^3 grid (t < k^3 <= kMaxSub): the float
// quotients of t + 1/2 lie at least 1/(2 k^2) from an integer, far above
// their rounding error, so truncation gives the integer quotients.
__device__ __forceinline__ void sub_xyz(int t, int k, float inv_k, float inv_k2, int &sx, int &sy, int &sz)
{
    sz = (int)(((float)t + 0.5f) * inv_k2);
    const int r = t - sz * k * k;
    sy = (int)(((float)r + 0.5f) * inv_k);
    sx = r - sy * k;
}

// Links of each lane's particle with particles j0 .. j1 - 1 of the wave's n
// (read with readlane): bit j - j0 of the result. kExact: decided in double;
// else in FP32, `band` set when a result lies in the guard band.
template <bool kExact>
__device__ __forceinline__ unsigned cell_row_word(const BoxDev &bd, int j0, int j1, bool strict, float x, float y,
                                                  float z, bool &band)
{
    unsigned w = 0u;
    for (int j = j0; j < j1; ++j) {
        const float xj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), j));
        const float yj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(y), j));
        const float zj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), j));
        bool link;
        if constexpr (kExact) {
            link = link_fp64(x, y, z, xj, yj, zj, bd.L, bd.half, bd.l2, strict);
        } else {
            const float dx = x - xj, dy = y - yj, dz = z - zj;
            const float rr = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            link = rr < bd.lo32;
            band = band | (!(rr < bd.lo32) & !(rr > bd.hi32));
        }
        w |= link ? 1u << (j - j0) : 0u;
    }
    return w;
}

// Links among the n <= 64 particles of one cell, one per lane: bit v of lane
// u's row is set when u and v are linked (or u == v). About 12 vector
// instructions per particle and no memory access; a result in the FP32 guard
// band (rare) has the whole cell decided in double. The differences of a pair
// are exact negatives either way round, so the rows are symmetric.
template <bool kFP64>
__device__ __forceinline__ unsigned long long cell_rows(const BoxDev &bd, int n, bool strict, float x, float y,
                                                        float z)
{
    const int n0 = min(n, 32);
    unsigned lo = 0u, hi = 0u;
    bool band = kFP64;
    if constexpr (!kFP64) {
        lo = cell_row_word<false>(bd, 0, n0, strict, x, y, z, band);
        hi = cell_row_word<false>(bd, 32, n, strict, x, y, z, band);
    }
    if (__ballot(band & (lane_id() < n))) {
        lo = cell_row_word<true>(bd, 0, n0, strict, x, y, z, band);
        hi = cell_row_word<true>(bd, 32, n, strict, x, y, z, band);
    }
    return ((((unsigned long long)hi) << 32) | lo) | (1ull << lane_id());
}

// Per-wave LDS of the pre-merge.
struct PremergeLds {
    unsigned long long rep[kMaxSub];   // per sub-cell: (hooking key << 32 | particle) of its first
                                       // particle, ~0 when empty
    int join[kMaxSub];                 // forest over the sub-cells (sub_adj)
    int used[kMaxSub];                 // the occupied sub-cells (sub_adj)
};

// The pre-merge by work-group `block` of `blocks`, on this wave's LDS.
template <bool kFP64>
__device__ __forceinline__ void premerge_cells(const Plan &p, PremergeLds &L, int block, int blocks)
{
    const int wid = threadIdx.x >> 6, lane = lane_id();
    unsigned long long *rp = L.rep;
    int *jf = L.join;
    int *ul = L.used;
    const bool rnd = p.link_random != 0;
    constexpr unsigned long long kEmpty = ~0ull;
    const int n_items = (int)p.counters->n_items;
    const XcdRange xr = xcd_range(n_items, kWaves, wid, block, blocks);
    for (int64_t it = xr.first; it < xr.end; it += xr.stride) {
        const int4 item = p.items[it];
        const int cs = __builtin_amdgcn_readfirstlane(item.x);
        const int tail = __builtin_amdgcn_readfirstlane(item.y);
        if (!(tail & kItemFirst)) continue;   // the cell's first item does the whole cell
        const int count = tail & ~kItemFirst;
        const int b = __builtin_amdgcn_readfirstlane(item.z);
        const BoxDev &bd = box_of(p, b);
        if (count <= 64) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (lane < count) v = p.sorted[cs + lane];
            const unsigned long long row =
                close_rows(cell_rows<kFP64>(bd, count, p.strict != 0, v.x, v.y, v.z), ~0ull >> (64 - count));
            int r = cs + __ffsll((long long)row) - 1;   // smallest index of the group
            if (rnd) {   // smallest hooking key instead, by the group's lowest lane
                const int at = r - cs;
                rp[lane] = kEmpty;
                __builtin_amdgcn_wave_barrier();
                if (lane < count) atomicMin(&rp[at], ((unsigned long long)link_key(cs + lane, true) << 32) |
                                                         (unsigned)(cs + lane));
                __builtin_amdgcn_wave_barrier();
                r = (int)(unsigned)(rp[at] & 0xffffffffull);
                __builtin_amdgcn_wave_barrier();
            }
            if (lane < count && r != cs + lane) p.parent[cs + lane] = r;
            const bool one = __ballot(lane < count && !(row & 1ull)) == 0;
            if (lane == 0) p.sorted[cs].w = __int_as_float(kCellJoined | (one ? kCellOneGroup : 0));
            continue;
        }
        const int k = bd.sub_k;
        if (k == 0) {
            if (lane == 0) p.sorted[cs].w = 0.f;
            continue;
        }
        const bool adj = bd.sub_adj != 0;
        const float inv_k = 1.0f / (float)k, inv_k2 = 1.0f / (float)(k * k);
        const int ce = cs + count;
        bool one = false;   // all joined into one set
        const float4 p0 = p.sorted[cs];   // the cell, from its first particle
        const int cx = cell_coord(p0.x, bd.inv_h, bd.nc), cy = cell_coord(p0.y, bd.inv_h, bd.nc),
                  cz = cell_coord(p0.z, bd.inv_h, bd.nc);
        const int nsub = k * k * k;
        for (int t = lane; t < nsub; t += 64) {
            rp[t] = kEmpty;
            jf[t] = t;
        }
        __builtin_amdgcn_wave_barrier();
        auto sub_of = [&](const float4 &q) {
            const double fx = (double)q.x * bd.inv_h - cx, fy = (double)q.y * bd.inv_h - cy,
                         fz = (double)q.z * bd.inv_h - cz;
            const int sx = min(max((int)floor(fx * k), 0), k - 1);
            const int sy = min(max((int)floor(fy * k), 0), k - 1);
            const int sz = min(max((int)floor(fz * k), 0), k - 1);
            return (sz * k + sy) * k + sx;
        };
        // kAhead particles per lane at a time, their loads in flight together;
        // the sub-cells of the first ones are kept for the hooks below
        constexpr int kAhead = 8;
        int kept[kAhead];
        auto sub_cells_from = [&](int base, int(&sub)[kAhead]) {
            float4 v[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int j = base + u * 64 + lane;
                v[u] = p.sorted[j < ce ? j : cs];
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) sub[u] = sub_of(v[u]);
        };
        sub_cells_from(cs, kept);
        for (int base = cs; base < ce; base += 64 * kAhead) {
            int sub[kAhead];
            if (base == cs) {
#pragma unroll
                for (int u = 0; u < kAhead; ++u) sub[u] = kept[u];
            } else {
                sub_cells_from(base, sub);
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int j = base + u * 64 + lane;
                if (j < ce) atomicMin(&rp[sub[u]], ((unsigned long long)link_key(j, rnd) << 32) | (unsigned)j);
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (adj) {
            // the occupied sub-cells, listed (there are at most as many as
            // particles), then each joined with the touching occupied ones
            // among the 13 of its 26 neighbours that come after it
            int n_used = 0;
            for (int t0 = 0; t0 < nsub; t0 += 64) {
                const int t = t0 + lane;
                const bool occ = t < nsub && rp[t] != kEmpty;
                const unsigned long long m = __ballot(occ);
                if (occ) ul[n_used + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u))] = t;
                n_used += __popcll(m);
            }
            __builtin_amdgcn_wave_barrier();
            if (n_used <= 64) {
                // at most 64 occupied sub-cells: lane q holds a row of bits, the
                // listed sub-cells touching sub-cell ul[q], and the components
                // come from the closure of the rows; jf maps a listed sub-cell
                // to its place in the list, then to its component's first one
                if (lane < n_used) jf[ul[lane]] = lane;
                __builtin_amdgcn_wave_barrier();
                unsigned long long row = 0ull;
                int t = 0;
                if (lane < n_used) {
                    t = ul[lane];
                    int sx, sy, sz;
                    sub_xyz(t, k, inv_k, inv_k2, sx, sy, sz);
                    row = 1ull << lane;
#pragma unroll
                    for (int o = 0; o < 27; ++o) {   // no branch: an outside neighbour reads sub-cell t
                        const int ux = sx + o % 3 - 1, uy = sy + (o / 3) % 3 - 1, uz = sz + o / 9 - 1;
                        const bool in = (unsigned)ux < (unsigned)k && (unsigned)uy < (unsigned)k &&
                                        (unsigned)uz < (unsigned)k;
                        const int u = in ? (uz * k + uy) * k + ux : t;
                        row |= (rp[u] != kEmpty ? 1ull : 0ull) << jf[u];
                    }
                }
                row = close_rows(row, __ballot(lane < n_used && row != (1ull << lane)));
                one = __ballot(lane < n_used && !(row & 1ull)) == 0;
                __builtin_amdgcn_wave_barrier();   // every map entry read
                if (lane < n_used) {
                    const int rt = ul[__ffsll((long long)row) - 1];
                    jf[t] = rt;
                    if (rt != t) atomicMin(&rp[rt], rp[t]);
                }
            } else if (nsub <= 128) {
                // up to 128 sub-cells (cells of up to 1.44 l_x: k = 5), as one
                // 128-bit mask in scalar registers: the component of the first
                // occupied sub-cell left grows by its 26 neighbours until it is
                // stable. So many occupied sub-cells are nearly always one
                // component, after a handful of steps; a union-find in LDS
                // over them took 14 us per cell.
                typedef unsigned __int128 Mask;
                Mask left = 0, x_inner0 = 0, x_inner1 = 0, y_inner0 = 0, y_inner1 = 0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int t = h * 64 + lane;
                    int sx, sy, sz;
                    sub_xyz(t, k, inv_k, inv_k2, sx, sy, sz);
                    auto half = [&](bool v) { return (Mask)__ballot(v) << (64 * h); };
                    left |= half(t < nsub && rp[t] != kEmpty);
                    x_inner0 |= half(sx > 0);
                    x_inner1 |= half(sx + 1 < k);
                    y_inner0 |= half(sy > 0);
                    y_inner1 |= half(sy + 1 < k);
                }
                const Mask occupied = left;
                int sets = 0;
                while (left) {
                    const unsigned long long l0 = (unsigned long long)left;
                    const int first = l0 ? __ffsll((long long)l0) - 1
                                         : 63 + __ffsll((long long)(unsigned long long)(left >> 64));
                    Mask m = (Mask)1 << first, before;
                    do {
                        before = m;
                        m |= ((m & x_inner1) << 1) | ((m & x_inner0) >> 1);
                        m |= ((m & y_inner1) << k) | ((m & y_inner0) >> k);
                        m |= (m << (k * k)) | (m >> (k * k));
                        m &= occupied;
                    } while (m != before);
                    left &= ~m;
                    ++sets;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int t = h * 64 + lane;
                        if ((unsigned)(m >> t) & 1u) {
                            jf[t] = first;
                            if (t != first) atomicMin(&rp[first], rp[t]);
                        }
                    }
                }
                one = sets == 1;
            } else {
                for (int q = lane; q < n_used; q += 64) {
                    const int t = ul[q];
                    int sx, sy, sz;
                    sub_xyz(t, k, inv_k, inv_k2, sx, sy, sz);
                    for (int o = 14; o < 27; ++o) {
                        const int ux = sx + o % 3 - 1, uy = sy + (o / 3) % 3 - 1, uz = sz + o / 9 - 1;
                        if (ux < 0 || ux >= k || uy < 0 || uy >= k || uz >= k) continue;
                        const int u = (uz * k + uy) * k + ux;
                        if (rp[u] != kEmpty) lds_unite(jf, t, u);
                    }
                }
                __builtin_amdgcn_wave_barrier();
                // the particle of smallest key of each joined set, at its root sub-cell
                const int r0 = lds_find(jf, ul[0]);
                bool same = true;
                for (int q = lane; q < n_used; q += 64) {
                    const int t = ul[q];
                    const int r = lds_find(jf, t);
                    same = same && r == r0;
                    if (r != t) atomicMin(&rp[r], rp[t]);
                }
                one = __ballot(!same) == 0;
            }
            __builtin_amdgcn_wave_barrier();
        }
        for (int base = cs; base < ce; base += 64 * kAhead) {
            int sub[kAhead];
            if (base == cs) {
#pragma unroll
                for (int u = 0; u < kAhead; ++u) sub[u] = kept[u];
            } else {
                sub_cells_from(base, sub);
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int j = base + u * 64 + lane;
                if (j >= ce) continue;
                const int r = (int)(unsigned)(rp[adj ? lds_find(jf, sub[u]) : sub[u]] & 0xffffffffull);
                if (r != j) p.parent[j] = r;   // a key smaller than j's: a valid hook of a root
            }
        }
        if (lane == 0) p.sorted[cs].w = __int_as_float(one ? kCellJoined | kCellOneGroup : 0);
        __builtin_amdgcn_wave_barrier();
    }
}

template <bool kFP64>
__global__ void __launch_bounds__(kBlock) k_dense_premerge(Plan p)
{
    __shared__ PremergeLds lds[kWaves];
    premerge_cells<kFP64>(p, lds[threadIdx.x >> 6], blockIdx.x, gridDim.x);
}

// Small runs (Plan::fused_link): the per-particle search, merging its own
// links, and the pre-merge side by side in one launch (they touch disjoint
// sets of particles) instead of three. The first `search` work-groups search.
template <bool kFP64>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) k_link_small(Plan p, int search)
{
    union Lds {
        SparseLds sparse[kWaves];
        PremergeLds pre[kWaves];
    };
    __shared__ __align__(16) unsigned char raw[sizeof(Lds)];
    Lds &lds = *reinterpret_cast<Lds *>(raw);
    const int wid = threadIdx.x >> 6, block = blockIdx.x;
    if (block < search) sparse_search<kFP64, false, true>(p, lds.sparse[wid], block, search);
    else premerge_cells<kFP64>(p, lds.pre[wid], block - search, gridDim.x - search);
}

// Global merge of domain mode, after the search. Workspace: the segment-order
// staging buffer (free after the build) holds flag/number [n + 1], the
// merge forest [n] and the group of each number [n].
//   roots: replace each boundary pair by the roots of its two groups and flag them
//   (an exclusive prefix over the flags numbers the flagged groups densely:
//    the paper's global-ID map, order-preserving so the smallest root of a
//    merged set also has the smallest number)
//   init:  a one-node tree per numbered group
//   union: union-find over the numbered pairs
//   apply: hook each merged group's root under its set's smallest root
__device__ __forceinline__ int *gm_flag(const Plan &p) { return reinterpret_cast<int *>(p.staging2); }
__device__ __forceinline__ int *gm_parent(const Plan &p) { return gm_flag(p) + p.n + 1; }
__device__ __forceinline__ int *gm_group(const Plan &p) { return gm_flag(p) + 2 * p.n + 1; }
__device__ __forceinline__ int64_t gm_pairs(const Plan &p)
{
    const int64_t nb = p.counters->n_boundary;
    return nb < p.max_edges ? nb : p.max_edges;
}

__global__ void __launch_bounds__(kBlock) k_gm_clear(Plan p)
{
    int *flag = gm_flag(p);
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i <= p.n; i += (int64_t)gridDim.x * kBlock) flag[i] = 0;
}

__global__ void __launch_bounds__(kBlock) k_gm_roots(Plan p)
{
    int *flag = gm_flag(p);
    const int64_t nb = gm_pairs(p);
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < nb; k += (int64_t)gridDim.x * kBlock) {
        const int2 e = p.bnd[k];
        const int ra = find_halve(p.parent, e.x), rb = find_halve(p.parent, e.y);
        p.bnd[k] = make_int2(ra, rb);
        flag[ra] = 1;
        flag[rb] = 1;
    }
}

__global__ void __launch_bounds__(kBlock) k_gm_init(Plan p)
{
    const int *num = gm_flag(p);   // exclusive prefix of the flags
    int *gp = gm_parent(p), *grp = gm_group(p);
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < p.n; r += (int64_t)gridDim.x * kBlock) {
        const int k = num[r];
        if (num[r + 1] != k) {
            gp[k] = k;
            grp[k] = (int)r;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) p.counters->n_bgroups = (unsigned)num[p.n];
}

__global__ void __launch_bounds__(kBlock) k_gm_union(Plan p)
{
    const int *num = gm_flag(p);
    int *gp = gm_parent(p);
    const int64_t nb = gm_pairs(p);
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < nb; k += (int64_t)gridDim.x * kBlock) {
        const int2 e = p.bnd[k];
        (void)unite(gp, num[e.x], num[e.y], false);
    }
}

__global__ void __launch_bounds__(kBlock) k_gm_apply(Plan p)
{
    const int *num = gm_flag(p);
    int *gp = gm_parent(p);
    const int *grp = gm_group(p);
    const int m = num[p.n];
    for (int k = blockIdx.x * kBlock + threadIdx.x; k < m; k += gridDim.x * kBlock) {
        const int r = find_halve(gp, k);
        if (r != k) p.parent[grp[k]] = grp[r];   // grp[r] < grp[k]: numbers keep the order of the roots
    }
}

// ------------------------------------------------- giant-component skip --
// In the manner of Afforest (Sutton et al., IPDPS 2018): after a first pass
// that links every particle to its axis-neighbour cells only (the per-particle
// search with Plan::sample set) and the dense-cell search, the largest group
// of a sample of roots is taken as "giant". The rest of the links is then
// searched over the whole periodic shell, both ways, but only from particles
// outside the giant group: a pair with one end inside is found from the other
// end, and a pair with both ends inside needs no union. Every linked pair of
// sparse cells is thereby merged; dense cells keep their own search.

__global__ void __launch_bounds__(kBlock) k_edge_reset(Plan p)
{
    if (threadIdx.x < kEdgeSlices) p.edge_fill[threadIdx.x] = 0;
}

constexpr int kGiantSamples = 4096;
constexpr int kGiantBlock = 1024;

// One work-group: the roots of kGiantSamples evenly spaced particles, sorted
// in LDS (bitonic), and the value of the longest run of equal roots.
__global__ void __launch_bounds__(kGiantBlock) k_giant(Plan p)
{
    __shared__ int r[kGiantSamples];
    __shared__ unsigned long long best;
    const int tid = (int)threadIdx.x;
    const bool rnd = p.link_random != 0;
    for (int k = tid; k < kGiantSamples; k += kGiantBlock)
        r[k] = find_root(p.parent, (int)((int64_t)k * p.n / kGiantSamples), p.find_mode, rnd);
    if (tid == 0) best = 0;
    __syncthreads();
    for (int k = 2; k <= kGiantSamples; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int idx = tid; idx < kGiantSamples; idx += kGiantBlock) {
                const int ixj = idx ^ j;
                if (ixj > idx) {
                    const int a = r[idx], b = r[ixj];
                    if ((a > b) == ((idx & k) == 0)) {
                        r[idx] = b;
                        r[ixj] = a;
                    }
                }
            }
            __syncthreads();
        }
    for (int idx = tid; idx < kGiantSamples; idx += kGiantBlock) {
        if (idx > 0 && r[idx - 1] == r[idx]) continue;   // not the start of a run
        int lo = idx, hi = kGiantSamples;                 // first entry above r[idx]
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (r[mid] <= r[idx]) lo = mid + 1;
            else hi = mid;
        }
        atomicMax(&best, ((unsigned long long)(lo - idx) << 32) | (unsigned)r[idx]);
    }
    __syncthreads();
    if (tid == 0) p.counters->giant = (int)(unsigned)(best & 0xffffffffull);
}

// The pair test of the per-particle search: FP32 with the image shift applied
// where it is exact (shift codes as for candidate ranges), re-decided in
// double inside the band; or the double predicate with the shift added after
// the rounded difference.
template <bool kFP64, bool kStats>
__device__ __forceinline__ bool pair_link(const float4 h, const float4 c, int code, const BoxPair &bx, bool strict,
                                          unsigned long long &band)
{
    if constexpr (kFP64) {
        const double tx = ((double)h.x - (double)c.x) + axis_shift(code & 3, bx.L);
        const double ty = ((double)h.y - (double)c.y) + axis_shift((code >> 2) & 3, bx.L);
        const double tz = ((double)h.z - (double)c.z) + axis_shift((code >> 4) & 3, bx.L);
        const double sxy = tx * tx + ty * ty;
        const double r2 = sxy + tz * tz;
        return strict ? (r2 < bx.l2) : (r2 <= bx.l2);
    } else {
        const float dx = axis_diff(h.x, c.x, code & 3, bx.L32);
        const float dy = axis_diff(h.y, c.y, (code >> 2) & 3, bx.L32);
        const float dz = axis_diff(h.z, c.z, (code >> 4) & 3, bx.L32);
        const float rr = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        if (rr < bx.lo32) return true;
        if (rr > bx.hi32) return false;
        if (kStats) ++band;
        return link_fp64(h.x, h.y, h.z, c.x, c.y, c.z, bx.L, bx.half, bx.l2, strict);
    }
}

// The second pass: one home particle per lane, skipped when it lies in the
// giant group or in a dense cell; otherwise every sparse cell of its periodic
// shell (all 27, both ways, the home particle itself excluded), each cell's
// candidates in lockstep over the wave so that the edge sink is reached by
// every lane together.
template <bool kFP64, bool kStats>
__global__ void __launch_bounds__(kBlock) k_link_rest(Plan p)
{
    __shared__ int2 ebuf[kWaves][kEdgeBuf];
    const int wid = threadIdx.x >> 6, lane = lane_id();
    EdgeSink<false> sink{ebuf[wid], 0};
    unsigned long long tests = 0, links = 0, band = 0;
    unsigned retries = 0;
    const bool rnd = p.link_random != 0;
    const bool strict = p.strict != 0;
    BoxHint hint;
    const int64_t n_tiles = (p.n + 63) / 64;
    const XcdRange xr = xcd_range(n_tiles, kWaves, wid);
    for (int64_t tile = xr.first; tile < xr.end; tile += xr.stride) {
        const int64_t s64 = tile * 64 + lane;
        bool active = s64 < p.n;
        const int s = active ? (int)s64 : 0;
        const int g = find_root(p.parent, p.counters->giant, p.find_mode, rnd);
        if (active) active = find_root(p.parent, s, p.find_mode, rnd) != g;
        int cx = 0, cy = 0, cz = 0, nc = 3;
        int64_t cb = 0;
        float4 h = make_float4(0.f, 0.f, 0.f, 0.f);
        BoxPair bx{};
        const int b = p.n_boxes == 1 ? 0 : find_box_hint(p.box_p0, p.n_boxes, s, hint);
        if (active) {
            const BoxDev &bd = box_of(p, b);
            bx = BoxPair::of(bd);
            h = p.sorted[s];
            nc = bd.nc;
            cb = bd.cell_base;
            cx = cell_coord(h.x, bd.inv_h, nc);
            cy = cell_coord(h.y, bd.inv_h, nc);
            cz = cell_coord(h.z, bd.inv_h, nc);
            const int2 own = cell_span(p, cb + ((int64_t)cz * nc + cy) * nc + cx);
            if (own.y - own.x >= p.dense_min) active = false;   // the dense search covers its pairs
        }
        if (__ballot(active) == 0) continue;
#pragma unroll 1
        for (int nb = 0; nb < 27; ++nb) {
            int j0 = 0, len = 0, code = 0;
            if (active) {
                int nx = cx + nb % 3 - 1, ny = cy + (nb / 3) % 3 - 1, nz = cz + nb / 9 - 1;
                if (nx < 0) { nx += nc; code |= 1; } else if (nx >= nc) { nx -= nc; code |= 2; }
                if (ny < 0) { ny += nc; code |= 1 << 2; } else if (ny >= nc) { ny -= nc; code |= 2 << 2; }
                if (nz < 0) { nz += nc; code |= 1 << 4; } else if (nz >= nc) { nz -= nc; code |= 2 << 4; }
                const int2 sp = cell_span(p, cb + ((int64_t)nz * nc + ny) * nc + nx);
                if (sp.y - sp.x < p.dense_min) {
                    j0 = sp.x;
                    len = sp.y - sp.x;
                }
            }
            int most = len;
            for (int d = 32; d >= 1; d >>= 1) most = max(most, __shfl_xor(most, d, 64));
            for (int t = 0; t < most; ++t) {
                const int j = j0 + t;
                const bool valid = t < len && j != s;
                bool link = false;
                if (valid) {
                    const float4 c = p.sorted[j];
                    link = pair_link<kFP64, kStats>(h, c, code, bx, strict, band);
                    if (kStats) {
                        ++tests;
                        if (link) ++links;
                    }
                }
                sink.push(p, link, s, j, retries);
            }
        }
    }
    sink.flush(p, retries);
    if (kStats) {
        tests = wave_sum_u64(tests);
        links = wave_sum_u64(links);
        band = wave_sum_u64(band);
        unsigned long long r = wave_sum_u64((unsigned long long)retries);
        if (lane == 0) {
            atomicAdd(&p.counters->sparse_tests, tests);
            atomicAdd(&p.counters->pair_tests, tests);
            atomicAdd(&p.counters->links, links);
            atomicAdd(&p.counters->band_hits, band);
            atomicAdd(&p.counters->cas_retries, r);
        }
    }
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

template <bool kFP64, bool kStats>
hipError_t launch_link_t(const Plan &p, hipStream_t stream, KernelTimer *t, const Fork *fk)
{
    Plan first = p;
    first.sample = p.giant_skip;   // the giant-component skip starts from the axis links
    if constexpr (!kStats)
        if (p.fused_link && !t) {
            const unsigned search = xcd_grid((p.n + 64 * kWaves - 1) / (64 * kWaves));
            const unsigned items = xcd_grid((p.n / p.dense_min + kWaves) / kWaves);
            const unsigned pre = items < 256u ? items : 256u;
            hipLaunchKernelGGL((k_link_small<kFP64>), dim3(search + pre), dim3(kBlock), 0, stream, p, (int)search);
            const unsigned dense = min(items << kMaxSplit, (unsigned)p.dense_blocks);
            if (p.link_random)
                hipLaunchKernelGGL((k_link_dense<kFP64, false, true>), dim3(dense), dim3(kBlock), 0, stream, p);
            else
                hipLaunchKernelGGL((k_link_dense<kFP64, false, false>), dim3(dense), dim3(kBlock), 0, stream, p);
            return hipSuccess;
        }
    if (t) t->mark(K_LINK_SPARSE, false, stream);
    hipLaunchKernelGGL((k_link_sparse<kFP64, kStats>), dim3((unsigned)p.sparse_blocks), dim3(kBlock), 0, stream,
                       first);
    if (t) t->mark(K_LINK_SPARSE, true, stream);
    // the sub-cell pre-merge would merge across slab faces: not in domain mode
    const bool premerge = p.domains <= 1 && p.premerge;
    // The pre-merge reads and writes the parents of particles in dense cells
    // only, the union pass those of particles in sparse cells only (the
    // per-particle search pairs sparse cells with sparse cells): given a
    // second stream the two run side by side, the pre-merge waiting for the
    // cell sort alone, and the wavefront search waits for both. Not with
    // per-kernel timers, whose events time each kernel alone.
    const bool beside = premerge && fk && fk->side && !t;
    if (beside) {
        hipError_t e = hipEventRecord(fk->fork, stream);
        if (e == hipSuccess) e = hipStreamWaitEvent(fk->side, fk->fork, 0);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_dense_premerge<kFP64>), dim3((unsigned)p.dense_blocks), dim3(kBlock), 0, fk->side, p);
        e = hipEventRecord(fk->join, fk->side);
        if (e != hipSuccess) return e;
    }
    auto union_edges = [&]() {
        const dim3 grid(kUnionParts * kEdgeSlices), block(kBlock);
        if (t) t->mark(K_UNION_EDGES, false, stream);
        if (p.link_random) hipLaunchKernelGGL((k_union_edges<kStats, true>), grid, block, 0, stream, p);
        else hipLaunchKernelGGL((k_union_edges<kStats, false>), grid, block, 0, stream, p);
        if (t) t->mark(K_UNION_EDGES, true, stream);
    };
    union_edges();
    if (beside) {
        const hipError_t e = hipStreamWaitEvent(stream, fk->join, 0);
        if (e != hipSuccess) return e;
    } else if (premerge) {
        if (t) t->mark(K_PREMERGE, false, stream);
        hipLaunchKernelGGL((k_dense_premerge<kFP64>), dim3((unsigned)p.dense_blocks), dim3(kBlock), 0, stream, p);
        if (t) t->mark(K_PREMERGE, true, stream);
    }
    if (t) t->mark(K_LINK_DENSE, false, stream);
    if (p.domains > 1 || p.link_random)
        hipLaunchKernelGGL((k_link_dense<kFP64, kStats, true>), dim3((unsigned)p.dense_blocks), dim3(kBlock), 0,
                           stream, p);
    else
        hipLaunchKernelGGL((k_link_dense<kFP64, kStats, false>), dim3((unsigned)p.dense_blocks), dim3(kBlock), 0,
                           stream, p);
    if (t) t->mark(K_LINK_DENSE, true, stream);
    if (p.giant_skip) {
        // the rest of the sparse pairs, from the particles outside the giant
        // group (timed with the per-particle search and the union pass)
        hipLaunchKernelGGL(k_edge_reset, dim3(1), dim3(kBlock), 0, stream, p);
        hipLaunchKernelGGL(k_giant, dim3(1), dim3(kGiantBlock), 0, stream, p);
        if (t) t->mark(K_LINK_SPARSE, false, stream);
        hipLaunchKernelGGL((k_link_rest<kFP64, kStats>), dim3((unsigned)p.sparse_blocks), dim3(kBlock), 0, stream,
                           p);
        if (t) t->mark(K_LINK_SPARSE, true, stream);
        union_edges();
    }
    if (p.domains > 1) {
        // global merge, timed with the union pass
        if (t) t->mark(K_UNION_EDGES, false, stream);
        const unsigned g = kGlobalMergeBlocks;
        hipLaunchKernelGGL(k_gm_clear, dim3(g), dim3(kBlock), 0, stream, p);
        hipLaunchKernelGGL(k_gm_roots, dim3(g), dim3(kBlock), 0, stream, p);
        scan_exclusive(reinterpret_cast<int *>(p.staging2), p.n + 1, p.scan_part, stream);
        hipLaunchKernelGGL(k_gm_init, dim3(g), dim3(kBlock), 0, stream, p);
        hipLaunchKernelGGL(k_gm_union, dim3(g), dim3(kBlock), 0, stream, p);
        hipLaunchKernelGGL(k_gm_apply, dim3(g), dim3(kBlock), 0, stream, p);
        if (t) t->mark(K_UNION_EDGES, true, stream);
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_link(const Plan &p, hipStream_t stream, KernelTimer *t, const Fork *fk)
{
    if (p.n == 0) return hipSuccess;
    const bool fp64 = p.predicate == 0;
    hipError_t e;
    if (fp64) e = p.stats ? launch_link_t<true, true>(p, stream, t, fk) : launch_link_t<true, false>(p, stream, t, fk);
    else e = p.stats ? launch_link_t<false, true>(p, stream, t, fk) : launch_link_t<false, false>(p, stream, t, fk);
    return e != hipSuccess ? e : hipGetLastError();
}

int64_t max_dense_items(int64_t n, int dense_min)
{
    const int64_t t = dense_min > 0 ? dense_min : 1;
    return n / 64 + n / t + 64;
}

}  // namespace fof
