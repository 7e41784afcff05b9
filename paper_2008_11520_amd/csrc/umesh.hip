// The fine DNN-MG step on unstructured quadrilateral meshes (explicit
// connectivity; fine nodes on curved edges moved onto the curve).
//
// Per step (the fine part of Alg. 2), all data addressed through the patch maps:
//   k_udefect  one thread per fine element: the element residual of the
//              defect (quad_residual: its own bilinear map and nodal P v, P p,
//              u_prev, formed once per patch node in LDS); every patch-local
//              node then adds its up to four elements' shares in the order
//              of their parity;
//   k_unode    one thread per fine node: the patches' contributions summed in
//              patch order (node_occ), zero at Dirichlet nodes (the stage
//              entry point);
//   k_uinput   the network input rows [P v, D, hx, hy, aspect, area], D
//              summed from the contributions as k_unode sums them;
//   (network)  the structured path's kernels on the rows;
//   k_urhs     the mean of the patches' outputs at the patch's nodes, masked;
//              the first patch that holds a node stores it and the corrected
//              velocity P v + d, the next u_prev; then, in FP64, the patch's
//              share of b^L = R (1/dt) M (P v + d) at its corners: on a patch
//              with straight edges (the bilinear image of the reference
//              square) from exact moments of det J, as on structured meshes;
//              on one with a curved edge from its hat-weighted mass rows
//              (formed at create from the fine elements' 2 x 2 Gauss points);
//              R = P^T;
//   k_ugather  one thread per coarse node: the shares summed in patch order.
// Sums over shared nodes are gathers in a fixed order: no atomics, bitwise
// deterministic.  A node inside a patch edge has at most two patches: the other
// one's entry is found through the patch's neighbour table (enb, ecode), one
// dependent load where the node's gather list takes three; a sum of two terms
// from +0 does not depend on their order.  Corners take their gather lists.
// P v at a fine node is the bilinear interpolation, in the reference coordinates
// of the first patch that holds the node, of that patch's corner values.
#include "device.h"
#include "element.h"
#include "internal.h"
#include "umesh_build.h"

namespace dnnmg {

// Coarse hats of corners v0 (0,0), v1 (1,0), v2 (1,1), v3 (0,1) at the
// patch-local node l = b (n+1) + a.
template <typename T>
__device__ inline void corner_hats(int n, int l, T (&N)[4])
{
    const int a = l % (n + 1), b = l / (n + 1);
    const T s = (T)a / (T)n, t = (T)b / (T)n;
    N[0] = (1 - s) * (1 - t);
    N[1] = s * (1 - t);
    N[2] = s * t;
    N[3] = (1 - s) * t;
}

// ------------------------------------------------------------------ defect
// Bound by latency (gathers through the patch map) and vector issue.  The nodal
// values are formed once per (patch, node) and shared through LDS; formed by
// each element for its four corners they were loaded and interpolated up to
// four times (70 840 patches, K = 2: 29.0 -> 23.1 us, about 460 of 760 instructions a wave in
// quad_residual).
template <int K>
__global__ __launch_bounds__(kThreads) void k_udefect(UArgs u)
{
    // NE threads per patch: thread j takes nodes j, j + NE, ... and element j
    constexpr int n = 1 << K, nf = (n + 1) * (n + 1), NE = n * n, PPB = kThreads / NE, NN = PPB * nf;
    constexpr int IT = (nf + NE - 1) / NE;
    __shared__ float2 s_R[4][kThreads], s_x[NN], s_v[NN], s_w[NN], s_cv[4 * PPB];
    __shared__ float s_p[NN], s_cp[4 * PPB];
    static_assert(4 * PPB <= kThreads, "one patch corner per thread");
    const int tid = threadIdx.x, pb = tid / NE, j = tid % NE, e0 = blockIdx.x * PPB, np = min(PPB, u.P - e0);
    const bool valid = pb < np;
    const size_t base = (size_t)(e0 + min(pb, np - 1)) * nf;
    const int first = *u.first_flag;
    const float idt = first ? 0.0f : u.inv_dt;
    const float2 *rel = reinterpret_cast<const float2 *>(u.rel) + base;
    const float2 *up = reinterpret_cast<const float2 *>(u.uprev);
    int f[IT];
    float2 x[IT], w[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) f[i] = u.pmap[base + min(j + i * NE, nf - 1)];
#pragma unroll
    for (int i = 0; i < IT; ++i) x[i] = rel[min(j + i * NE, nf - 1)];
    if (tid < 4 * np) {
        const int c = u.corners[4 * (size_t)e0 + tid];
        s_cv[tid] = reinterpret_cast<const float2 *>(u.v)[c];
        s_cp[tid] = u.p ? u.p[c] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) w[i] = up[f[i]];
    __syncthreads();
    const float2 *cv = s_cv + 4 * pb;
    const float *cp = s_cp + 4 * pb;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int l = j + i * NE, t = pb * nf + l;
        if (l >= nf || !valid) continue;
        float N[4];
        corner_hats(n, l, N);
        float2 v;
        v.x = N[0] * cv[0].x + N[1] * cv[1].x + N[2] * cv[2].x + N[3] * cv[3].x;
        v.y = N[0] * cv[0].y + N[1] * cv[1].y + N[2] * cv[2].y + N[3] * cv[3].y;
        s_p[t] = N[0] * cp[0] + N[1] * cp[1] + N[2] * cp[2] + N[3] * cp[3];
        s_v[t] = v;
        s_x[t] = x[i];
        if (first) w[i] = make_float2(0.f, 0.f);
        s_w[t] = make_float2(w[i].x * idt, w[i].y * idt);
    }
    __syncthreads();
    const int a = j % n, b = j / n;
    const int l00 = pb * nf + b * (n + 1) + a, ls[4] = {l00, l00 + 1, l00 + n + 1, l00 + n + 2};
    if (valid) {
        float R[8];
        float ex[4], ey[4], vx[4], vy[4], pn[4], wx[4], wy[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float2 r = s_x[ls[k]], v = s_v[ls[k]], q = s_w[ls[k]];
            ex[k] = r.x; ey[k] = r.y;
            vx[k] = v.x; vy[k] = v.y;
            wx[k] = q.x; wy[k] = q.y;
            pn[k] = s_p[ls[k]];
        }
        quad_residual<HwRcp>(ex, ey, vx, vy, pn, wx, wy, u.nu, idt, R);
#pragma unroll
        for (int k = 0; k < 4; ++k) s_R[k][tid] = make_float2(R[2 * k], R[2 * k + 1]);
    }
    __syncthreads();
    // every node adds its (up to four) elements' shares in the order of the
    // elements' parity (a & 1) + 2 (b & 1)
    float2 *dl = reinterpret_cast<float2 *>(u.dloc) + base;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int l = j + i * NE, na = l % (n + 1), nb = l / (n + 1);
        if (l >= nf || !valid) continue;
        float2 s = make_float2(0.f, 0.f);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            // the element of parity c among (na - 1, na) x (nb - 1, nb), and the node's corner in it
            const int ca = (na ^ c) & 1, cb = (nb ^ (c >> 1)) & 1, ea = na - ca, eb = nb - cb;
            if ((unsigned)ea >= (unsigned)n || (unsigned)eb >= (unsigned)n) continue;
            const float2 q = s_R[ca + 2 * cb][pb * NE + eb * n + ea];
            s.x += q.x;
            s.y += q.y;
        }
        dl[l] = s;
    }
}

__global__ __launch_bounds__(kThreads) void k_unode(UArgs u, float *D)
{
    const int f = blockIdx.x * kThreads + threadIdx.x;
    if (f >= u.Fn) return;
    const float2 *dl = reinterpret_cast<const float2 *>(u.dloc);
    float2 s = make_float2(0.f, 0.f);
    for (int k = u.node_ptr[f]; k < u.node_ptr[f + 1]; ++k) {
        const float2 q = dl[u.node_occ[k]];
        s.x += q.x;
        s.y += q.y;
    }
    if (u.mask[f]) s = make_float2(0.f, 0.f);
    reinterpret_cast<float2 *>(D)[f] = s;
}

// D == nullptr: the element contributions only (the step: the network input
// sums them per node itself); else also the defect at the fine nodes.
template <int K>
static void launch_udefect_k(const UArgs &u, float *D, hipStream_t s)
{
    constexpr int n = 1 << K, PPB = kThreads / (n * n);
    hipLaunchKernelGGL(k_udefect<K>, dim3((u.P + PPB - 1) / PPB), dim3(kThreads), 0, s, u);
    if (D) hipLaunchKernelGGL(k_unode, dim3((u.Fn + kThreads - 1) / kThreads), dim3(kThreads), 0, s, u, D);
}

hipError_t launch_udefect(const UArgs &u, float *D, hipStream_t s)
{
    switch (u.K) {
    case 1: launch_udefect_k<1>(u, D, s); break;
    case 2: launch_udefect_k<2>(u, D, s); break;
    case 3: launch_udefect_k<3>(u, D, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ------------------------------------------------------- network input rows
// A workgroup takes upatches<K>() patches: P v and D at every (patch, node) (pairs as
// one store) and the patches' features.  D comes from the patches' element
// contributions directly, summed over the node's patches as k_unode sums them
// (the same value bit for bit), zero at Dirichlet nodes.  Bound by latency: the
// entries of all of a thread's nodes are requested before any is used (70 840
// patches, K = 2: 27.4 -> 15.0 us).
template <typename XT>
__device__ inline void store_pair(XT *o, float a, float b)
{
    if constexpr (sizeof(XT) == 4) {
        *reinterpret_cast<float2 *>(o) = make_float2(a, b);
    } else {
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        b2 v;
        v[0] = (__bf16)a;
        v[1] = (__bf16)b;
        *reinterpret_cast<b2 *>(o) = v;
    }
}

// Patches per workgroup of the per-node kernels, kThreads / upatches threads each
// (thread j of a patch takes nodes j, j + that, ...), and the workgroup's staging
// of its patches: neighbours and edge codes, corner velocities.
template <int K> constexpr int upatches() { return K == 3 ? 8 : 32; }
template <int K> struct UStage {
    int nb[4 * upatches<K>()];
    float2 cv[4 * upatches<K>()];
    unsigned code[upatches<K>()];
};
// Node l of patch e0 + p, which no corner is: the entry (patch nf + node) of the
// other patch that holds it, or -1; masked: on a Dirichlet edge.
template <int K>
__device__ __forceinline__ int uother(const UStage<K> &s, int p, int l, bool &masked)
{
    constexpr int n = 1 << K, nf = (n + 1) * (n + 1);
    int t = 0;
    const int k = edge_of_node(n, l % (n + 1), l / (n + 1), t);
    masked = false;
    if (k < 0) return -1;
    const unsigned code = s.code[p] >> (8 * k);
    masked = (code & kEdgeDirichlet) != 0u;
    const int e2 = s.nb[4 * p + k];
    return e2 < 0 ? -1 : e2 * nf + neighbour_node(n, code, t);
}
// Patch-local node of corner k.
template <int K> __device__ inline int ucorner(int k)
{
    constexpr int n = 1 << K;
    return (k >> 1) * n * (n + 1) + ((k ^ (k >> 1)) & 1) * n;
}

// The sum of q over the gather list of coarse node c in patch order, from the
// list's first entries o (UMeshHost::vocc) and their values v, and its length.
__device__ __forceinline__ float2 ulist_sum(const UArgs &u, int4 o, const float2 (&v)[4], int c, const float2 *q, int &cnt)
{
    float2 s = make_float2(0.f, 0.f);
    if (o.x == kLongList) {
        const int k0 = u.node_ptr[c], k1 = u.node_ptr[c + 1];
        for (int k = k0; k < k1; ++k) {
            const float2 t = q[u.node_occ[k]];
            s.x += t.x;
            s.y += t.y;
        }
        cnt = k1 - k0;
        return s;
    }
    const int i[4] = {o.x, o.y, o.z, o.w};
    cnt = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (i[k] >= 0) { s.x += v[k].x; s.y += v[k].y; ++cnt; }
    return s;
}

// What both per-node kernels request at once: the own entries of q (the patches'
// contributions or outputs, per (patch, node)) at the thread's nodes, then,
// through the staged neighbour tables, the other patch's entry at each node
// inside an edge, and (threads < 4 upatches) the entries of one patch corner.
// Two dependent loads in all, the corner velocities included (stored to s.cv; the
// caller synchronises before it reads them).
template <int K> struct UNodes {
    static constexpr int n = 1 << K, nf = (n + 1) * (n + 1), PB = upatches<K>(), TP = kThreads / PB, IT = (nf + TP - 1) / TP;
    float2 q1[IT], q2[IT], vq[4];
    int o[IT], c;          // the other patch's entry, or -1; the corner's coarse node
    int4 vo;
    unsigned zero;         // bit i: node i on a Dirichlet edge; bit 31: the corner
};
template <int K>
__device__ __forceinline__ void unodes_load(const UArgs &u, int e0, int np, const float2 *q, UStage<K> &s, UNodes<K> &r)
{
    typedef UNodes<K> N;
    const int tid = threadIdx.x, p = tid / N::TP, j = tid % N::TP;
    const float2 *own = q + (size_t)(e0 + min(p, np - 1)) * N::nf;
#pragma unroll
    for (int i = 0; i < N::IT; ++i) r.q1[i] = own[min(j + i * N::TP, N::nf - 1)];
    static_assert(4 * N::PB + N::PB <= kThreads, "a corner and an edge, or an edge code, per thread");
    r.c = 0;
    r.vo = make_int4(-1, -1, -1, -1);
    if (tid < 4 * np) {
        r.c = u.corners[4 * (size_t)e0 + tid];
        r.vo = reinterpret_cast<const int4 *>(u.vocc)[4 * (size_t)e0 + tid];
        s.nb[tid] = u.enb[4 * (size_t)e0 + tid];
    } else if (tid >= kThreads - N::PB && tid - (kThreads - N::PB) < np) {
        s.code[tid - (kThreads - N::PB)] = u.ecode[(size_t)e0 + tid - (kThreads - N::PB)];
    }
    __syncthreads();
    r.zero = 0u;
#pragma unroll
    for (int i = 0; i < N::IT; ++i) {
        bool z = false;
        r.o[i] = p < np ? uother<K>(s, p, min(j + i * N::TP, N::nf - 1), z) : -1;
        if (z) r.zero |= 1u << i;
        r.q2[i] = q[max(r.o[i], 0)];
    }
    if (tid < 4 * np) {
        const int i[4] = {r.vo.x, r.vo.y, r.vo.z, r.vo.w};
        s.cv[tid] = reinterpret_cast<const float2 *>(u.v)[r.c];
#pragma unroll
        for (int k = 0; k < 4; ++k) r.vq[k] = q[max(i[k], 0)];
        if ((s.code[tid >> 2] >> (8 * (tid & 3))) & kCornerDirichlet) r.zero |= 1u << 31;
    }
}

template <int K, typename XT>
__global__ __launch_bounds__(kThreads) void k_uinput(UArgs u)
{
    typedef UNodes<K> N;
    constexpr int n = N::n, nf = N::nf, PB = N::PB;
    __shared__ UStage<K> st;
    const int tid = threadIdx.x, e0 = blockIdx.x * PB, np = min(PB, u.P - e0);
    const float2 *dl = reinterpret_cast<const float2 *>(u.dloc);
    XT *const X = reinterpret_cast<XT *>(u.X) + (size_t)e0 * u.nin;
    N r;
    unodes_load<K>(u, e0, np, dl, st, r);
    float4 ft = make_float4(0.f, 0.f, 0.f, 0.f);
    const int pf = tid - (kThreads - PB);
    if (pf >= 0 && pf < np) ft = reinterpret_cast<const float4 *>(u.feat)[(size_t)e0 + pf];
    __syncthreads();
    auto put = [&](int p, int l, float2 d) {
        const float2 *cv = st.cv + 4 * p;
        XT *x = X + (size_t)p * u.nin;
        float H[4];
        corner_hats(n, l, H);
        store_pair(x + 2 * l, H[0] * cv[0].x + H[1] * cv[1].x + H[2] * cv[2].x + H[3] * cv[3].x,
                   H[0] * cv[0].y + H[1] * cv[1].y + H[2] * cv[2].y + H[3] * cv[3].y);
        store_pair(x + 2 * nf + 2 * l, d.x, d.y);
    };
    const int p = tid / N::TP, j = tid % N::TP;
    if (p < np) {
#pragma unroll
        for (int i = 0; i < N::IT; ++i) {
            const int l = j + i * N::TP, a = l % (n + 1), b = l / (n + 1);
            if (l >= nf || ((a == 0 || a == n) && (b == 0 || b == n))) continue;
            // (a node inside the patch is this patch's alone: its value as it is)
            float2 d = r.q1[i];
            if (a == 0 || a == n || b == 0 || b == n) {
                d = make_float2(0.f, 0.f);
                d.x += r.q1[i].x; d.y += r.q1[i].y;
                if (r.o[i] >= 0) { d.x += r.q2[i].x; d.y += r.q2[i].y; }
            }
            if ((r.zero >> i) & 1u) d = make_float2(0.f, 0.f);
            put(p, l, d);
        }
    }
    if (tid < 4 * np) {
        int cnt;
        float2 d = ulist_sum(u, r.vo, r.vq, r.c, dl, cnt);
        if (r.zero >> 31) d = make_float2(0.f, 0.f);
        put(tid >> 2, ucorner<K>(tid & 3), d);
    }
    if (pf >= 0 && pf < np) {
        XT *x = X + (size_t)pf * u.nin + 4 * nf;
        store_pair(x, ft.x, ft.y);
        store_pair(x + 2, ft.z, ft.w);
    }
}

hipError_t launch_uinput(const UArgs &u, hipStream_t s)
{
    const int pb = u.K == 3 ? upatches<3>() : upatches<1>();
    dim3 g((u.P + pb - 1) / pb), b(kThreads);
#define DNNMG_UINPUT(KK)                                                                  \
    case KK:                                                                              \
        if (u.xfmt == 1) hipLaunchKernelGGL((k_uinput<KK, __bf16>), g, b, 0, s, u);       \
        else hipLaunchKernelGGL((k_uinput<KK, float>), g, b, 0, s, u);                    \
        break;
    switch (u.K) {
        DNNMG_UINPUT(1)
        DNNMG_UINPUT(2)
        DNNMG_UINPUT(3)
    default: return hipErrorInvalidValue;
    }
#undef DNNMG_UINPUT
    return hipGetLastError();
}

// P v (and P p) at fine node f from its first patch.
template <typename T>
__device__ inline void uprolong_node(const UArgs &u, int nf, int n, int f, T &vx, T &vy, bool want_p, T &pp)
{
    const int occ = u.node_occ[u.node_ptr[f]];
    const int e = occ / nf, l = occ - e * nf;
    const int *cn = u.corners + 4 * (size_t)e;
    T N[4];
    corner_hats(n, l, N);
    const float2 *v2 = reinterpret_cast<const float2 *>(u.v);
    vx = 0;
    vy = 0;
    T q = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float2 c = v2[cn[k]];
        vx += N[k] * (T)c.x;
        vy += N[k] * (T)c.y;
        if (want_p) q += N[k] * (T)u.p[cn[k]];
    }
    pp = q;
}

__global__ __launch_bounds__(kThreads) void k_uprolong(UArgs u)
{
    const int f = blockIdx.x * kThreads + threadIdx.x;
    if (f >= u.Fn) return;
    const int n = 1 << u.K, nf = (n + 1) * (n + 1);
    float vx, vy, q = 0.0f;
    uprolong_node<float>(u, nf, n, f, vx, vy, u.p && u.pp_out, q);
    if (u.pv_out) reinterpret_cast<float2 *>(u.pv_out)[f] = make_float2(vx, vy);
    if (u.p && u.pp_out) u.pp_out[f] = q;
}

hipError_t launch_uprolong(const UArgs &u, hipStream_t s)
{
    hipLaunchKernelGGL(k_uprolong, dim3((u.Fn + kThreads - 1) / kThreads), dim3(kThreads), 0, s, u);
    return hipGetLastError();
}

// ------------------------- averaging, state, correction, FP64 rhs shares
// A workgroup takes upatches<K>() patches.  STEP: the averaged correction at all of
// their nodes from the patches' outputs (every patch that holds a node forms
// the same mean; the first one in patch order stores it and the corrected
// velocity), else the given correction dbar.  It stays in LDS for the patch's
// share of R (1/dt) M_f u at each corner, u = P v + d, one item per (patch,
// component, corner column) as in the structured rhs.  Straight edges: at
// structured corner (cx, cy)
//   d0 S0 + d1 S1 + d2 S2,  S_k = sum_b A[my_k][cy][b] sum_a A[mx_k][cx][a] d(a, b)
// ((mx, my) = (0, 0), (1, 0), (0, 1)), and the coarse term of P v from the moment
// tables M.  A curved edge: the hat-weighted mass rows formed at create,
//   sum_k M4[c][k] v_k + sum_l W[c][l] d_l.
// Bound by latency: all map entries, outputs and neighbours' outputs of a thread
// are requested before any is used.  70 840 patches, K = 2: 18.1 us, where a thread
// per fine node through the gather lists and a thread per patch for the shares
// took 21.6 + 11.4 us and wrote and read the correction between them.
template <int K, bool STEP>
__global__ __launch_bounds__(kThreads) void k_urhs(UArgs u, const float *dbar)
{
    typedef UNodes<K> N;
    constexpr int n = N::n, nf = N::nf, PB = N::PB, IT = N::IT;
    constexpr int NA = 4 * (n + 1), NM = 48;
    static_assert(NA + NM <= kThreads && 4 * PB <= kThreads, "one table entry, one rhs item per thread");
    __shared__ UStage<K> st;
    __shared__ double s_A[NA], s_M[NM];
    __shared__ float2 s_d[PB * nf];
    const int tid = threadIdx.x, e0 = blockIdx.x * PB, np = min(PB, u.P - e0);
    const int pn = tid / N::TP, jn = tid % N::TP;
    const int *pm = u.pmap + (size_t)(e0 + min(pn, np - 1)) * nf;
    const double tab = tid < NA ? u.tab.A[tid] : u.tab.M[min(tid - NA, NM - 1)];
    int f[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) f[i] = pm[min(jn + i * N::TP, nf - 1)];
    // the fourth item of this thread's patch: its determinant or its curved rows
    const int e = e0 + min(tid >> 2, np - 1);
    const int ci = u.cidx[e];
    const double2 g01 = reinterpret_cast<const double2 *>(u.dgeo)[2 * (size_t)e];
    const double g2 = u.dgeo[4 * (size_t)e + 2];
    if constexpr (STEP) {
        const float2 *dp = reinterpret_cast<const float2 *>(u.dpatch);
        N r;
        unodes_load<K>(u, e0, np, dp, st, r);
        if (tid < NA) s_A[tid] = tab;
        else if (tid < NA + NM) s_M[tid - NA] = tab;
        __syncthreads();
        bool nonfin = false;
        // the averaged correction d at node l of patch e0 + p; `first`: this
        // patch is the node's first and stores it at fine node fn
        auto put = [&](int p, int l, float2 d, bool first, int fn) {
            s_d[p * nf + l] = d;
            if (!first) return;
            const float2 *cv = st.cv + 4 * p;
            float H[4];
            corner_hats(n, l, H);
            float vx = 0.0f, vy = 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                vx += H[k] * cv[k].x;
                vy += H[k] * cv[k].y;
            }
            reinterpret_cast<float2 *>(u.uprev)[fn] = make_float2(vx + d.x, vy + d.y);
            if (u.dbar_out) reinterpret_cast<float2 *>(u.dbar_out)[fn] = d;
            nonfin |= !(__builtin_isfinite(d.x) && __builtin_isfinite(d.y));
        };
        if (pn < np) {
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const int l = jn + i * N::TP, a = l % (n + 1), b = l / (n + 1);
                if (l >= nf || ((a == 0 || a == n) && (b == 0 || b == n))) continue;
                float2 s = make_float2(0.f, 0.f);
                s.x += r.q1[i].x; s.y += r.q1[i].y;
                if (r.o[i] >= 0) { s.x += r.q2[i].x; s.y += r.q2[i].y; }
                const float inv = r.o[i] >= 0 ? 0.5f : 1.0f;
                const float2 d = ((r.zero >> i) & 1u) ? make_float2(0.f, 0.f) : make_float2(s.x * inv, s.y * inv);
                put(pn, l, d, r.o[i] < 0 || r.o[i] > (e0 + pn) * nf + l, f[i]);
            }
        }
        if (tid < 4 * np) {
            const int p = tid >> 2, l = ucorner<K>(tid & 3);
            int cnt;
            const float2 s = ulist_sum(u, r.vo, r.vq, r.c, dp, cnt);
            const float inv = 1.0f / (float)cnt;
            const float2 d = (r.zero >> 31) ? make_float2(0.f, 0.f) : make_float2(s.x * inv, s.y * inv);
            const int occ0 = r.vo.x == kLongList ? u.node_occ[u.node_ptr[r.c]] : r.vo.x;
            put(p, l, d, occ0 == (e0 + p) * nf + l, r.c);
        }
        // coarse nodes that no patch holds: no output to average, the correction is zero
        for (int t = blockIdx.x * kThreads + tid; t < u.nlone; t += gridDim.x * kThreads) {
            const int c = u.lone[t];
            reinterpret_cast<float2 *>(u.uprev)[c] = reinterpret_cast<const float2 *>(u.v)[c];
            if (u.dbar_out) reinterpret_cast<float2 *>(u.dbar_out)[c] = make_float2(0.f, 0.f);
        }
        if (nonfin && u.nonfinite) atomicOr(u.nonfinite, 1);
        if (blockIdx.x == 0 && tid == 0) *u.first_flag = 0;   // the step's defect has read it (stream order)
    } else {
        float2 w[IT];
#pragma unroll
        for (int i = 0; i < IT; ++i) w[i] = reinterpret_cast<const float2 *>(dbar)[f[i]];
        if (tid < 4 * np) st.cv[tid] = reinterpret_cast<const float2 *>(u.v)[u.corners[4 * (size_t)e0 + tid]];
        if (tid < NA) s_A[tid] = tab;
        else if (tid < NA + NM) s_M[tid - NA] = tab;
        if (pn < np) {
#pragma unroll
            for (int i = 0; i < IT; ++i)
                if (jn + i * N::TP < nf) s_d[pn * nf + jn + i * N::TP] = w[i];
        }
    }
    __syncthreads();
    if (tid >= 4 * np) return;
    const int cx = tid & 1, comp = (tid >> 1) & 1, p = tid >> 2;
    const float *d1 = reinterpret_cast<const float *>(s_d + p * nf) + comp;
    const float *v1 = reinterpret_cast<const float *>(st.cv + 4 * p) + comp;
    double out[2];     // structured corners (cx, 0) and (cx, 1)
    if (ci < 0) {
        const double g0 = g01.x, g1 = g01.y;
        double S[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
#pragma unroll
        for (int b = 0; b <= n; ++b) {
            double s0 = 0.0, s1 = 0.0;
#pragma unroll
            for (int a = 0; a <= n; ++a) {
                const double w = (double)d1[2 * (b * (n + 1) + a)];
                s0 += s_A[(0 * 2 + cx) * (n + 1) + a] * w;
                s1 += s_A[(1 * 2 + cx) * (n + 1) + a] * w;
            }
#pragma unroll
            for (int cy = 0; cy < 2; ++cy) {
                const double y0 = s_A[(0 * 2 + cy) * (n + 1) + b], y1 = s_A[(1 * 2 + cy) * (n + 1) + b];
                S[cy][0] += y0 * s0;
                S[cy][1] += y0 * s1;
                S[cy][2] += y1 * s0;
            }
        }
#pragma unroll
        for (int cy = 0; cy < 2; ++cy) {
            const int cs = cx + 2 * cy;
            double acc = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int ks = k ^ (k >> 1);
                const double m = g0 * s_M[(0 * 4 + cs) * 4 + ks] + g1 * s_M[(1 * 4 + cs) * 4 + ks] +
                                 g2 * s_M[(2 * 4 + cs) * 4 + ks];
                acc += m * (double)v1[2 * k];
            }
            out[cy] = acc + g0 * S[cy][0] + g1 * S[cy][1] + g2 * S[cy][2];
        }
    } else {
        // a curved edge: the stored rows of corners v0, v3 (cx = 0) or v1, v2
#pragma unroll
        for (int cy = 0; cy < 2; ++cy) {
            const int c = cy ? 3 - cx : cx;
            const double *W = u.W + ((size_t)ci * 4 + c) * nf, *M = u.M4 + 16 * (size_t)ci + 4 * c;
            double acc = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) acc += M[k] * (double)v1[2 * k];
            for (int l = 0; l < nf; ++l) acc += W[l] * (double)d1[2 * l];
            out[cy] = acc;
        }
    }
    double *o = u.part + 8 * (size_t)e + comp;
    o[2 * cx] = u.inv_dt64 * out[0];
    o[2 * (3 - cx)] = u.inv_dt64 * out[1];
}

// dbar == nullptr: the step.
hipError_t launch_urhs(const UArgs &u, const float *dbar, hipStream_t s)
{
    const int pb = u.K == 3 ? upatches<3>() : upatches<1>();
    const dim3 g((u.P + pb - 1) / pb), b(kThreads);
    switch (u.K) {
#define DNNMG_URHS(KK)                                                                                \
    case KK:                                                                                          \
        if (dbar) hipLaunchKernelGGL((k_urhs<KK, false>), g, b, 0, s, u, dbar);                       \
        else hipLaunchKernelGGL((k_urhs<KK, true>), g, b, 0, s, u, dbar);                             \
        break;
        DNNMG_URHS(1)
        DNNMG_URHS(2)
        DNNMG_URHS(3)
#undef DNNMG_URHS
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

__global__ __launch_bounds__(kThreads) void k_ugather(UArgs u)
{
    const int c = blockIdx.x * kThreads + threadIdx.x;
    if (c >= u.Nc) return;
    const double2 *pt = reinterpret_cast<const double2 *>(u.part);
    double bx = 0.0, by = 0.0;
    for (int k = u.cnode_ptr[c]; k < u.cnode_ptr[c + 1]; ++k) {
        const double2 q = pt[u.cnode_occ[k]];
        bx += q.x;
        by += q.y;
    }
    reinterpret_cast<double2 *>(u.bL)[c] = make_double2(bx, by);
    if (u.nonfinite && !(__builtin_isfinite(bx) && __builtin_isfinite(by))) atomicOr(u.nonfinite, 2);
}

hipError_t launch_ugather(const UArgs &u, hipStream_t s)
{
    hipLaunchKernelGGL(k_ugather, dim3((u.Nc + kThreads - 1) / kThreads), dim3(kThreads), 0, s, u);
    return hipGetLastError();
}

}  // namespace dnnmg
