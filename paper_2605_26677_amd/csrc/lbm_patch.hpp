// Geometry shared by the patch kernels (lbm_patch.hip, lbm_patch_adj.hip): the patch of a
// workgroup and the node of a thread.
#pragma once

#include "lbm_device.hpp"
#include "lbm_internal.hpp"
#include "lbm_kernel_util.hpp"

namespace lbm {

// Position of thread i of a patch of pw x ph nodes: the nodes of the patch first, row by row
// (ring 0), then the rings of nodes at distance 1, 2, ... around it (top row, bottom row, left
// and right columns), so that the nodes a level still needs are a prefix of the threads and
// whole wavefronts retire as the halo shrinks.
struct PatchPos {
    int x, y, ring;
};
__device__ __forceinline__ PatchPos patch_pos(int i, int pw, int ph) {
    PatchPos p;
    if (i < pw * ph) {
        p.y = i / pw;
        p.x = i - p.y * pw;
        p.ring = 0;
        return p;
    }
    int k = 1;
    while (i >= (pw + 2 * k) * (ph + 2 * k)) ++k;
    const int w = pw + 2 * k, h = ph + 2 * k - 2;
    const int j = i - (w - 2) * h;
    p.ring = k;
    if (j < 2 * w) {
        p.x = (j < w ? j : j - w) - k;
        p.y = j < w ? -k : ph - 1 + k;
    } else {
        const int c = j - 2 * w;
        p.x = c < h ? -k : pw - 1 + k;
        p.y = (c < h ? c : c - h) - k + 1;
    }
    return p;
}

// The patch of this workgroup: its size and first node.
__device__ __forceinline__ void patch_at(const PatchMap& m, int& pw, int& ph, int& px0, int& py0, int& x1, int& y1) {
    int g = blockIdx.x, rc = 0;
    while (rc + 1 < m.nrect && g >= m.rect[rc + 1].first) ++rc;
    const PatchRect& pr = m.rect[rc];
    g -= pr.first;
    if (rc == m.nrect - 1) g = remap_tile(g, m.nwg - pr.first);
    const int by = fdiv(g, pr.d_npx), bx = g - by * pr.npx;
    pw = m.pw;
    ph = m.ph;
    px0 = pr.x0 + bx * pw;
    py0 = pr.y0 + by * ph;
    x1 = pr.x1;
    y1 = pr.y1;
}

}  // namespace lbm
