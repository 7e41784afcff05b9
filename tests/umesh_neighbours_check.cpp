// Host entry point over the neighbour tables of the unstructured-mesh
// construction (paper_2008_11520_amd/csrc/umesh_build.h): counts the entries
// that disagree with the mesh's own gather lists, for the CPU test.
#include "umesh_build.h"

using namespace dnnmg;

extern "C" int un_check(int nc, int ne, const double *xy, const int *elems, int ndir, const int *dirs, int ncirc,
                        const double *circ, int ncurved, const int *curved, int K, int *checked)
{
    UMeshHost m;
    if (!build_umesh(nc, ne, xy, elems, ndir, dirs, ncirc, circ, ncurved, curved, K, m).empty()) return -1;
    const int n = m.n, nf = m.nf;
    int bad = 0, seen = 0;
    for (int e = 0; e < ne; ++e)
        for (int l = 0; l < nf; ++l) {
            const int a = l % (n + 1), b = l / (n + 1), f = m.pmap[(size_t)e * nf + l];
            const int k0 = m.node_ptr[f], cnt = m.node_ptr[f + 1] - k0;
            int t = 0;
            const int k = edge_of_node(n, a, b, t);
            ++seen;
            if (k == -1) {
                bad += cnt != 1 || m.mask[f];
            } else if (k >= 0) {
                const unsigned code = m.ecode[e] >> (8 * k);
                const int e2 = m.enb[4 * (size_t)e + k];
                bad += edge_node(n, k, t) != l;
                bad += ((code & kEdgeDirichlet) != 0u) != (m.mask[f] != 0);
                bad += e2 < 0 ? cnt != 1
                              : cnt != 2 || m.node_occ[k0] + m.node_occ[k0 + 1] != e * nf + l + e2 * nf + neighbour_node(n, code, t);
            } else {
                const int c = b == 0 ? (a == 0 ? 0 : 1) : (a == 0 ? 3 : 2);
                const int *o = &m.vocc[4 * (4 * (size_t)e + c)];
                bad += m.corners[4 * (size_t)e + c] != f;
                bad += ((m.ecode[e] >> (8 * c) & kCornerDirichlet) != 0u) != (m.mask[f] != 0);
                if (cnt > 4) bad += o[0] != kLongList;
                else
                    for (int i = 0; i < 4; ++i) bad += o[i] != (i < cnt ? m.node_occ[k0 + i] : -1);
            }
        }
    *checked = seen;
    return bad;
}
