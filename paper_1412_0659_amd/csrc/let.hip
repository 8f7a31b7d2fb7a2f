// Boundary trees and local essential trees (LETs) of spatial domains
// (Sec. III.B.2: each domain cuts its tree down to the cells on the edge of
// its particle set; a remote domain checks whether that boundary tree holds
// enough cells for its own targets, and otherwise receives the specific set
// of cells and particles its targets reach; the received trees become
// branches of one tree that the force walk reads).
//
// Boundary tree of a domain: from the root through cells of more than ncrit
// particles, stopping at cells of at most ncrit particles, at leaves and at
// a level L (the deepest at which the tree has at most max_cells cells).
// Its terminal cells cover every particle once; their tight particle boxes,
// widened by a margin, stand for the domain's targets.
//
// LET of a source tree for a target domain: every target box walks the
// source tree with the force walk's own traversal and opening test, and marks
// the cells it accepts and those it opens.  Any target group lies inside one
// terminal box, and the margin keeps its FP32 box distance to any cell at
// least the box's, so a group opens only cells that its box opens: the reached
// cells (opened cells with all their children, opened leaves with their
// particles) are exactly what the group walks need, and walking them gives bit
// for bit the interaction lists of the full source tree.  When no box opens a
// terminal cell of the source's boundary tree, the boundary tree itself serves
// as the LET.
//
// All sources of a target go through each step together (a source is a grid
// row), their cells and particles one after another in the scratch arrays, so
// that one scan numbers the kept cells and particles of all of them and the
// host waits once: 12 launches for up to 16 sources.  Source by source, with a
// pass up the levels to find the opened cells, it took 40 launches and two
// waits per source.  Four domains of a 262144-particle disk, trees and forces:
// 5.87 -> 2.51 ms, the construction now about 0.2 ms per target, half of it
// k_let_mark (97 us, a walk whose longest box bounds it).
#include <algorithm>

#include "walk_common.h"

namespace bh {

uint32_t cell_count(const bh_ctx *c, hipStream_t st) {
    uint32_t nc = 0;
    if (hipStreamSynchronize(st) != hipSuccess ||
        hipMemcpy(&nc, c->cells.ls + kLevels, sizeof(uint32_t), hipMemcpyDeviceToHost) !=
            hipSuccess)
        return 0;
    return nc;
}

// ---- boundary tree ----------------------------------------------------------

__global__ __launch_bounds__(256) void k_bnd_flags(Cells c, uint32_t ncrit, uint32_t *flag,
                                                   uint32_t *lvl) {
    const uint32_t nc = c.ls[kLevels];
    const uint32_t lane = threadIdx.x & 63u;
    // every thread of a wave runs the same trips, so the counts can be
    // combined across the wave (cells are level-ordered: most waves see one level)
    for (uint32_t base = blockIdx.x * 256 + (threadIdx.x & ~63u); base < nc;
         base += gridDim.x * 256) {
        const uint32_t i = base + lane;
        bool inb = false;
        uint32_t lev = kLevels;
        if (i < nc) {
            inb = i == 0u || c.count[c.parent[i]] > ncrit;
            flag[i] = inb ? 1u : 0u;
            lev = c.level[i];
        }
        const uint32_t lev0 = shfl(lev, 0);
        if (ballot(lev != lev0 && i < nc) == 0ull) {
            const uint32_t k = (uint32_t)__popcll(ballot(inb));
            if (lane == 0 && k) atomicAdd(&lvl[lev0], k);
        } else if (inb) {
            atomicAdd(&lvl[lev], 1u);
        }
    }
}

// FP32 bounding box of every cell's particles, from the deepest level up:
// a leaf over its particles, an internal cell over its children (min and
// max are exact, so this equals the box over the particles)
__global__ __launch_bounds__(256) void k_cbox_leaf(Cells c, const float4 *__restrict__ xyzm,
                                                   float4 *__restrict__ cmin,
                                                   float4 *__restrict__ cmax) {
    const uint32_t nc = c.ls[kLevels];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < nc; i += gridDim.x * 256) {
        if (c.nchild[i] != 0u) continue;
        const uint32_t b = c.begin[i], e = b + c.count[i];
        float4 mn = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
        float4 mx = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.f);
        for (uint32_t j = b; j < e; ++j) {
            const float4 p = xyzm[j];
            mn.x = fminf(mn.x, p.x); mn.y = fminf(mn.y, p.y); mn.z = fminf(mn.z, p.z);
            mx.x = fmaxf(mx.x, p.x); mx.y = fmaxf(mx.y, p.y); mx.z = fmaxf(mx.z, p.z);
        }
        cmin[i] = mn;
        cmax[i] = mx;
    }
}

__global__ __launch_bounds__(256) void k_cbox_up(Cells c, int l, float4 *cmin, float4 *cmax) {
    const uint32_t first = c.ls[l], last = c.ls[l + 1];
    for (uint32_t i = first + blockIdx.x * 256 + threadIdx.x; i < last; i += gridDim.x * 256) {
        const uint32_t nch = c.nchild[i];
        if (nch == 0u) continue;
        const uint32_t k0 = c.child0[i];
        float4 mn = cmin[k0], mx = cmax[k0];
        for (uint32_t k = k0 + 1; k < k0 + nch; ++k) {
            const float4 a = cmin[k], b = cmax[k];
            mn.x = fminf(mn.x, a.x); mn.y = fminf(mn.y, a.y); mn.z = fminf(mn.z, a.z);
            mx.x = fmaxf(mx.x, b.x); mx.y = fmaxf(mx.y, b.y); mx.z = fmaxf(mx.z, b.z);
        }
        cmin[i] = mn;
        cmax[i] = mx;
    }
}

__global__ __launch_bounds__(256) void k_bnd_terminal(Cells c, uint32_t level, uint32_t ncrit,
                                                      uint32_t *flag, uint32_t *tscan) {
    const uint32_t nc = c.ls[kLevels];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i <= nc; i += gridDim.x * 256) {
        if (i == nc) {
            flag[nc] = 0u;
            tscan[nc] = 0u;
            continue;
        }
        const uint32_t lev = c.level[i];
        const bool inb = (flag[i] & 1u) != 0u && lev <= level;
        const bool small = c.count[i] <= ncrit || c.nchild[i] == 0u;
        const bool term = inb && (lev == level || small);
        flag[i] = (inb ? 1u : 0u) | (term ? 2u : 0u);
        tscan[i] = term ? 1u : 0u;
    }
}

__global__ __launch_bounds__(256) void k_bnd_ids(const uint32_t *__restrict__ flag,
                                                 const uint32_t *__restrict__ tscan, uint32_t nc,
                                                 uint32_t *__restrict__ ids) {
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < nc; i += gridDim.x * 256)
        if (flag[i] & 2u) ids[tscan[i]] = i;
}

// tight FP32 box of each terminal cell: centre (min + max) / 2, half size
// (max - min) / 2 + margin
__global__ __launch_bounds__(256) void k_bnd_box(const uint32_t *__restrict__ ids, uint32_t nterm,
                                                 const float4 *__restrict__ cmin,
                                                 const float4 *__restrict__ cmax, float margin,
                                                 float4 *__restrict__ box) {
    for (uint32_t k = blockIdx.x * 256 + threadIdx.x; k < nterm; k += gridDim.x * 256) {
        const uint32_t cell = ids[k];
        const float4 mn = cmin[cell], mx = cmax[cell];
        box[2 * (size_t)k] = make_float4((mn.x + mx.x) * 0.5f, (mn.y + mx.y) * 0.5f,
                                         (mn.z + mx.z) * 0.5f, 0.f);
        box[2 * (size_t)k + 1] =
            make_float4((mx.x - mn.x) * 0.5f + margin, (mx.y - mn.y) * 0.5f + margin,
                        (mx.z - mn.z) * 0.5f + margin, 0.f);
    }
}

void launch_bnd_flags(bh_ctx *c, hipStream_t st) {
    launch_fill_u32(c->bnd.lvl, 0u, kLevels, st);
    hipLaunchKernelGGL(k_bnd_flags, dim3(kGrid), dim3(256), 0, st, c->cells,
                       (uint32_t)c->p.ncrit, c->bnd.flag, c->bnd.lvl);
}

void launch_bnd_terminal(bh_ctx *c, int level, hipStream_t st) {
    hipLaunchKernelGGL(k_bnd_terminal, dim3(kGrid), dim3(256), 0, st, c->cells, (uint32_t)level,
                       (uint32_t)c->p.ncrit, c->bnd.flag, c->bnd.scan);
}

void launch_bnd_boxes(bh_ctx *c, uint32_t nc, uint32_t nterm, hipStream_t st) {
    Boundary &b = c->bnd;
    hipLaunchKernelGGL(k_bnd_ids, dim3(kGrid), dim3(256), 0, st, (const uint32_t *)b.flag,
                       (const uint32_t *)b.scan, nc, b.ids);
    if (nterm == 0) return;
    hipLaunchKernelGGL(k_cbox_leaf, dim3(kGrid * 2), dim3(256), 0, st, c->cells,
                       (const float4 *)c->xyzm, b.cmin, b.cmax);
    for (int l = kLevels - 2; l >= 0; --l)
        hipLaunchKernelGGL(k_cbox_up, dim3(kGrid), dim3(256), 0, st, c->cells, l, b.cmin, b.cmax);
    uint32_t nb = cdiv(nterm, 256);
    if (nb > 4096) nb = 4096;
    hipLaunchKernelGGL(k_bnd_box, dim3(nb), dim3(256), 0, st, (const uint32_t *)b.ids, nterm,
                       (const float4 *)b.cmin, (const float4 *)b.cmax, b.margin, b.box);
}

// ---- local essential tree ---------------------------------------------------

// A source as the kernels see it, and where its cells and particles lie in the
// scratch arrays.
struct LetSrc {
    float4 *wA;
    const float2 *size;
    const uint2 *wN;
    const float4 *P0, *P1, *P2, *xyzm;
    const uint32_t *begin, *count, *child0, *nchild, *bflag;
    uint32_t nc, n, c0, p0;
};
constexpr int kLetBatch = 16;
struct LetBatch {
    LetSrc s[kLetBatch];
    uint32_t first, nsrc;  // this batch's first source, sources of all batches
    uint32_t cells, parts; // of all sources
    uint32_t *acc, *opn, *pmark, *word;  // [cells], [cells], [parts], [nsrc]
    uint32_t *keep;                      // [cells + parts + 1], then its scan
};

// opening radii of the batch's sources for theta
__global__ __launch_bounds__(256) void k_let_prep(LetBatch b, float theta) {
    const LetSrc &s = b.s[blockIdx.y];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < s.nc; i += gridDim.x * 256)
        s.wA[i].w = open_radius2(s.size[i], theta);
}

// One wave per (source, target box): the force walk's traversal of the
// source tree; accepted and opened cells are marked.
__global__ __launch_bounds__(64) void k_let_mark(LetBatch b, uint32_t batch,
                                                 const float4 *__restrict__ tbox, uint32_t nbox,
                                                 uint32_t *spill_base, uint32_t *status) {
    __shared__ TravLds L;
    const uint32_t lane = threadIdx.x;
    uint32_t *spill = spill_base + (size_t)blockIdx.x * kStackMax;
    for (uint32_t task = blockIdx.x; task < batch * nbox; task += gridDim.x) {
        const uint32_t q = task / nbox, k = task - q * nbox;
        const LetSrc &s = b.s[q];
        uint32_t *acc = b.acc + s.c0, *opn = b.opn + s.c0;
        const TreeView tv{s.wA, s.wN, (uint32_t)kRing, status, opn};
        const float4 bc = tbox[2 * (size_t)k], bh = tbox[2 * (size_t)k + 1];
        GroupBox g;
        g.cx = bc.x; g.cy = bc.y; g.cz = bc.z;
        g.hx = bh.x; g.hy = bh.y; g.hz = bh.z;
        uint32_t npc = 0, npp = 0;
        traverse<true>(
            tv, g, lane, L, spill, npc, npp,
            [&](uint32_t n) {
                for (uint32_t i = lane; i < n; i += 64u) acc[L.pcidx[i]] = 1u;
            },
            [&](uint32_t n) {
                for (uint32_t i = lane; i < n; i += 64u) opn[L.ppidx[i]] = 1u;
            });
    }
}

// Marks of the opened leaves' particles; word of a source: some box opened a
// terminal cell of its boundary tree.
__global__ __launch_bounds__(256) void k_let_opened(LetBatch b) {
    const LetSrc &s = b.s[blockIdx.y];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < s.nc; i += gridDim.x * 256) {
        if (!b.opn[s.c0 + i]) continue;
        if (s.bflag[i] & 2u) b.word[b.first + blockIdx.y] = 1u;
        if (s.nchild[i] != 0u) continue;
        const uint32_t j0 = s.p0 + s.begin[i], j1 = j0 + s.count[i];
        for (uint32_t j = j0; j < j1; ++j) b.pmark[j] = 1u;
    }
}

__global__ __launch_bounds__(256) void k_let_keep(LetBatch b) {
    const LetSrc &s = b.s[blockIdx.y];
    const bool boundary_only = b.word[b.first + blockIdx.y] == 0u;
    const uint32_t step = gridDim.x * 256, i0 = blockIdx.x * 256 + threadIdx.x;
    for (uint32_t i = i0; i < s.nc; i += step)
        b.keep[s.c0 + i] =
            boundary_only ? (s.bflag[i] & 1u) : (b.acc[s.c0 + i] | b.opn[s.c0 + i]);
    for (uint32_t j = i0; j < s.n; j += step)
        b.keep[b.cells + s.p0 + j] = boundary_only ? 0u : b.pmark[s.p0 + j];
    if (i0 == 0u) b.keep[b.cells + b.parts] = 0u;
}

struct LetOut {
    float4 *wA, *P0, *P1, *P2;
    uint2 *wN;
    uint32_t *origin;
    float4 *xyzm;
};

// Virtual cells above the sources' roots: levels of lv cells each.
struct LetVirtual {
    uint32_t lv[4];
    uint32_t nlv, nv;
};

// Kept source cells -> LET slots: the root of source k at nv + k, the other
// cells behind all roots in scan order.  An expanded cell keeps its children
// (internal) or its particles (leaf); every other kept cell becomes a leaf
// with none.
__global__ __launch_bounds__(256) void k_let_emit(LetBatch b, LetVirtual v, LetOut o) {
    const LetSrc &s = b.s[blockIdx.y];
    const uint32_t src = b.first + blockIdx.y;
    const bool boundary_only = b.word[src] == 0u;
    const uint32_t *scan = b.keep, *pscan = b.keep + b.cells;
    const uint32_t r0 = scan[s.c0], kept = scan[b.cells];
    // (scan counts the earlier sources' roots, this one's and the cell itself)
    auto slot_of = [&](uint32_t rank) { return v.nv + b.nsrc + rank - (src + 1u); };
    const uint32_t step = gridDim.x * 256, i0 = blockIdx.x * 256 + threadIdx.x;
    for (uint32_t i = i0; i < s.nc; i += step) {
        const bool opn = b.opn[s.c0 + i] != 0u;
        const bool keep = boundary_only ? (s.bflag[i] & 1u) != 0u : opn || b.acc[s.c0 + i] != 0u;
        if (!keep) continue;
        const uint32_t r = scan[s.c0 + i];
        const uint32_t slot = r == r0 ? v.nv + src : slot_of(r);
        const bool expand = boundary_only ? (s.bflag[i] & 3u) == 1u : opn;
        const uint32_t nch = s.nchild[i];
        uint2 N = make_uint2(0u, kLeafBit);
        if (expand && nch) N = make_uint2(slot_of(scan[s.c0 + s.child0[i]]), nch);
        else if (expand) N = make_uint2(pscan[s.p0 + s.begin[i]] - kept, s.count[i] | kLeafBit);
        o.wA[slot] = s.wA[i];
        o.P0[slot] = s.P0[i];
        o.P1[slot] = s.P1[i];
        o.P2[slot] = s.P2[i];
        o.wN[slot] = N;
        o.origin[2 * (size_t)slot] = src;
        o.origin[2 * (size_t)slot + 1] = i;
    }
    if (!boundary_only)
        for (uint32_t j = i0; j < s.n; j += step)
            if (b.pmark[s.p0 + j]) o.xyzm[pscan[s.p0 + j] - kept] = s.xyzm[j];
    if (src != 0u) return;
    // the virtual cells: never accepted (r_open^2 = +inf), children contiguous
    uint32_t off = 0;
    for (uint32_t q = 0; q + 1u < v.nlv; ++q) {
        const uint32_t next = off + v.lv[q];
        for (uint32_t i = i0; i < v.lv[q]; i += step) {
            const uint32_t slot = off + i;
            o.wA[slot] = make_float4(0.f, 0.f, 0.f, INFINITY);
            o.P0[slot] = o.P1[slot] = o.P2[slot] = make_float4(0.f, 0.f, 0.f, 0.f);
            o.wN[slot] = make_uint2(next + 8u * i, min(8u, v.lv[q + 1u] - 8u * i));
            o.origin[2 * (size_t)slot] = kNone;
            o.origin[2 * (size_t)slot + 1] = kNone;
        }
        off = next;
    }
}

// per source: boundary tree sufficed, cells, particles; then the totals
__global__ __launch_bounds__(64) void k_let_info(LetBatch b, uint32_t batch, uint32_t *info) {
    const uint32_t *scan = b.keep, *pscan = b.keep + b.cells;
    if (threadIdx.x < batch) {
        const LetSrc &s = b.s[threadIdx.x];
        const uint32_t k = b.first + threadIdx.x;
        info[3 * k] = b.word[k] == 0u ? 1u : 0u;
        info[3 * k + 1] = scan[s.c0 + s.nc] - scan[s.c0];
        info[3 * k + 2] = pscan[s.p0 + s.n] - pscan[s.p0];
    }
    if (threadIdx.x == 0) {
        info[3 * b.nsrc] = scan[b.cells];
        info[3 * b.nsrc + 1] = pscan[b.parts] - scan[b.cells];
    }
}

void launch_let(bh_ctx *tgt, bh_ctx *const *srcs, int nsrc, float theta, const int64_t lv[4],
                int nlv, uint32_t nv, hipStream_t st) {
    Let &t = tgt->let;
    uint32_t cells = 0, parts = 0, most = 1;
    for (int k = 0; k < nsrc; ++k) {
        cells += srcs[k]->bnd.ncell;
        parts += (uint32_t)srcs[k]->n;
        most = std::max({most, srcs[k]->bnd.ncell, (uint32_t)srcs[k]->n});
    }
    launch_fill_u32(t.marks, 0u, 2ull * cells + parts + (uint32_t)nsrc, st);
    const dim3 block(256);
    const uint32_t rows = std::min(cdiv(most, 256), 1024u);
    auto each_batch = [&](auto &&step) {
        uint32_t c0 = 0, p0 = 0;
        for (int first = 0; first < nsrc; first += kLetBatch) {
            LetBatch b{};
            const uint32_t batch = (uint32_t)std::min(kLetBatch, nsrc - first);
            for (uint32_t k = 0; k < batch; ++k) {
                const bh_ctx *s = srcs[first + (int)k];
                const Cells &q = s->cells;
                b.s[k] = LetSrc{q.wA, q.size, q.wN, q.P0, q.P1, q.P2, s->xyzm, q.begin, q.count,
                                q.child0, q.nchild, s->bnd.flag, s->bnd.ncell, (uint32_t)s->n,
                                c0, p0};
                c0 += s->bnd.ncell;
                p0 += (uint32_t)s->n;
            }
            b.first = (uint32_t)first;
            b.nsrc = (uint32_t)nsrc;
            b.cells = cells;
            b.parts = parts;
            b.acc = t.marks;
            b.opn = b.acc + cells;
            b.pmark = b.opn + cells;
            b.word = b.pmark + parts;
            b.keep = t.keep;
            step(b, batch);
        }
    };
    const uint32_t nbox = tgt->bnd.nterm;
    each_batch([&](const LetBatch &b, uint32_t batch) {
        hipLaunchKernelGGL(k_let_prep, dim3(rows, batch), block, 0, st, b, theta);
        const uint64_t tasks = (uint64_t)batch * nbox;
        if (tasks)
            hipLaunchKernelGGL(k_let_mark,
                               dim3((uint32_t)std::min<uint64_t>(tasks, (uint64_t)tgt->walk_grid)),
                               dim3(64), 0, st, b, batch, (const float4 *)tgt->bnd.box, nbox,
                               tgt->spill, tgt->status);
        hipLaunchKernelGGL(k_let_opened, dim3(rows, batch), block, 0, st, b);
        hipLaunchKernelGGL(k_let_keep, dim3(rows, batch), block, 0, st, b);
    });
    launch_exclusive_scan(t.keep, t.keep, cells + parts + 1u, t.spart, st);
    LetVirtual v{};
    for (int q = 0; q < 4; ++q) v.lv[q] = (uint32_t)lv[q];
    v.nlv = (uint32_t)nlv;
    v.nv = nv;
    const LetOut o{t.wA, t.P0, t.P1, t.P2, t.wN, t.origin, t.xyzm};
    each_batch([&](const LetBatch &b, uint32_t batch) {
        hipLaunchKernelGGL(k_let_emit, dim3(rows, batch), block, 0, st, b, v, o);
        hipLaunchKernelGGL(k_let_info, dim3(1), dim3(64), 0, st, b, batch, t.info);
    });
}

}  // namespace bh
