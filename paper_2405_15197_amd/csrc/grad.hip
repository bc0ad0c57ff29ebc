// Adjoint of the triangulation at fixed topology.
//
// Loss terms over the triangle mesh (Area, the volume enclosed about a fixed
// point p0, and the sum of squared vertex norms) and their gradient with
// respect to the mesh vertices; then, per node, the gradient of the loss
// with respect to the node centres and nodal-sphere radii, propagated back
// through the node's mesh vertices while the discrete structure (labels,
// arcs, segment counts, triangles) stays that of the forward pass:
//
//   hole centre (Eq. 13)  rho * b / |b|, b the mean of the contour vertices;
//   interior point (Eq. 12)  o + a sin t_i + b cos t_i, t_i = t1 + (t2 - t1) i / N;
//   arc ends  t1, t2 are the conic parameters of the arc's end vertices;
//   conic (o, a, b)  the tangency circle or the Eq. 7 ellipse of struts p, q;
//   vertex  the tie P_p = P_q = P_r, |w|^2 - rho^2 = P_p^2 (Sec. 4.3.1),
//           differentiated implicitly;
//   strut table  g_m, h_m, e_m from the two node centres and radii.
//
// Everything is taken in reverse.
#include "geom.h"

namespace lm {
namespace {

using namespace geo;

constexpr int kBlock = 256;

// ---------------------------------------------------------------------------
// loss terms and their gradient with respect to the mesh vertices

__device__ inline float3 f3(const float *p) { return make_float3(p[0], p[1], p[2]); }
__device__ inline float3 sub3(float3 a, float3 b) { return make_float3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ inline float3 crs3(float3 a, float3 b)
{
    return make_float3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ inline void add3(float *p, float3 v, float s)
{
    atomicAdd(p, v.x * s);
    atomicAdd(p + 1, v.y * s);
    atomicAdd(p + 2, v.z * s);
}

// Triangle terms: area 1/2 |N| with N = (b - a) x (c - a), dA/da =
// 1/2 n x (c - b) (cyclic); volume (a' . (b' x c')) / 6 about p0,
// dV/da = (b' x c') / 6.
// Per node (one wave): the gradient of the loss with respect to the node's
// own mesh vertices, gathered over the triangles that touch them (its hole
// fans and the bands of its incident struts) in LDS and written once; the
// loss terms count each band at its lower end node and each fan at its
// node.
//
// A band lists the triangles of the edges of one end loop, then those of the
// other, each in loop order; an edge triangle's apex is on the other loop.
// So the wave adds without LDS atomics, in steps of distinct addresses with a
// barrier after each (of no cost in a block of one wave, and what orders a
// lane's reads after the others' writes):
// the edges of the node's own loop add their first ends, then their second
// ends, and the other loop's edges, whose apexes on this one come in runs of
// neighbouring lanes, add each run's sum.  (With an atomic per corner and
// coordinate the kernel was bound by them, some 60 cycles of the compute
// unit's LDS per instruction.)  The bands' bookkeeping is read for all struts
// at once, a lane per strut.  Octet 32^3, k = 16: 1.45 -> 0.62 ms.
//
// LDS vertices at a time; a node with more of them passes over its triangles
// again, up to kLossMost vertices, beyond that it adds through global atomics.
// Room for 512 lets 25 waves onto a compute unit, for 1,024 twelve, which
// spares nodes of 513 to 1,024 vertices the second pass: see launch_loss.
constexpr int kLossMost = 2048;
constexpr int kLossSmall = 512, kLossLarge = 1024;

struct LParams {
    Inputs in;
    Work w;
    const int32_t *tri;
    const float *xyz;
    int64_t cap_mesh, cap_tri;  // sizes of tri / xyz (and dldx) in rows
    float3 p0;
    float w_area, w_vol, w_sq;
    float *dldx;
    double *terms;
};

// The mesh of the last pass must be complete and fit the buffers given here
// (tri, xyz and dldx): otherwise nothing is read, and zeros are written.
__device__ inline bool mesh_fits(const LParams &P)
{
    const Work &W = P.w;
    const int64_t N = P.in.n_nodes, Np1 = N + 1;
    const int64_t m_all = W.node_off[(int64_t)NC_MESH * Np1 + N];
    const int64_t t_all = W.band_off[P.in.n_struts] + W.node_off[(int64_t)NC_FAN * Np1 + N];
    return !(W.flags[0] & (DF_CAPACITY | DF_RECCAP)) && m_all <= P.cap_mesh && t_all <= P.cap_tri;
}

// dldx beyond the mesh's vertices (which their nodes write), or all of it
__global__ void k_loss_rest(LParams P)
{
    const int64_t end = 3 * P.cap_mesh, Np1 = P.in.n_nodes + 1;
    const int64_t i0 = mesh_fits(P) ? 3 * P.w.node_off[(int64_t)NC_MESH * Np1 + P.in.n_nodes] : 0;
    for (int64_t i = i0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < end; i += (int64_t)gridDim.x * blockDim.x)
        P.dldx[i] = 0.f;
}

template <int LDS>
__global__ void __launch_bounds__(64) k_loss_node(LParams P)
{
    __shared__ float gx[LDS], gy[LDS], gz[LDS];
    const Work &W = P.w;
    const int64_t N = P.in.n_nodes, S = P.in.n_struts;
    const int64_t n = blockIdx.x;
    const int lane = threadIdx.x;
    if (n >= N) return;
    const int64_t Np1 = N + 1;
    double *nt = W.loss_node + 3 * n;  // this node's share of the loss terms
    const int64_t r0 = W.row[n], r1 = W.row[n + 1];
    const int64_t m0 = W.node_off[(int64_t)NC_MESH * Np1 + n], m1 = W.node_off[(int64_t)NC_MESH * Np1 + n + 1];
    const int64_t f0 = W.band_off[S] + W.node_off[(int64_t)NC_FAN * Np1 + n];
    const int64_t f1 = W.band_off[S] + W.node_off[(int64_t)NC_FAN * Np1 + n + 1];
    if (!mesh_fits(P)) {
        if (lane == 0) {
            atomicOr(&W.flags[0], DF_CAPACITY);
            nt[0] = nt[1] = nt[2] = 0.0;
        }
        return;
    }
    const int M = (int)(m1 - m0);
    if (M == 0) {
        if (lane == 0) nt[0] = nt[1] = nt[2] = 0.0;
        return;
    }
    // strut `lane`: its band, the samples of the own loop, which end this is
    const int v = (int)(r1 - r0);  // at most kVmaxBig = 64: the node has a mesh
    int64_t my_b0 = 0;
    int my_nb = 0, my_own = 0, my_lower = 0;
    if (lane < v) {
        const int2 he = W.he[r0 + lane];
        my_own = W.he_len[r0 + lane];
        my_lower = (int64_t)he.x > n;
        my_b0 = W.band_off[he.y];
        my_nb = (int)(W.band_off[he.y + 1] - my_b0);
    }
    double area = 0.0, vol = 0.0, sq = 0.0;
    const bool lds = M <= kLossMost;
    int c0 = 0;  // vertices [c0, c0 + LDS) of the node are in LDS
    // a triangle and its normal; its terms when counted (area twice, volume
    // six times what they are: scaled once per node)
    struct Tri {
        int32_t i0, i1, i2;
        float3 a, b, c, n;
        float wa;
    };
    const bool grad = P.w_area != 0.f || P.w_vol != 0.f;
    const float wv = P.w_vol / 6.f;
    // turn: its corners in the order 2, 0, 1
    auto tri_at = [&](int64_t t, bool count, bool turn) {
        Tri T;
        const int32_t j0 = P.tri[3 * t], j1 = P.tri[3 * t + 1], j2 = P.tri[3 * t + 2];
        T.i0 = turn ? j2 : j0;
        T.i1 = turn ? j0 : j1;
        T.i2 = turn ? j1 : j2;
        T.a = sub3(f3(P.xyz + 3 * (int64_t)T.i0), P.p0);
        T.b = sub3(f3(P.xyz + 3 * (int64_t)T.i1), P.p0);
        T.c = sub3(f3(P.xyz + 3 * (int64_t)T.i2), P.p0);
        // the normal from the first end of the edge, of the edge and of a side:
        // of the two sides from the apex it would be a small difference
        const float3 q0 = turn ? T.b : T.a, q1 = turn ? T.c : T.b, q2 = turn ? T.a : T.c;
        T.n = crs3(sub3(q1, q0), sub3(q2, q0));
        const float nl = sqrtf(T.n.x * T.n.x + T.n.y * T.n.y + T.n.z * T.n.z);
        if (count) {
            const float3 x = crs3(q1, q2);
            area += (double)nl;
            vol += (double)q0.x * x.x + (double)q0.y * x.y + (double)q0.z * x.z;
        }
        T.wa = (P.w_area != 0.f && nl > 0.f) ? 0.5f * P.w_area / nl : 0.f;
        return T;
    };
    // the gradient on the corner before the edge b -> c
    auto corner = [&](const Tri &T, float3 b, float3 c) {
        const float3 ga = crs3(T.n, sub3(c, b)), x = crs3(b, c);
        return make_float3(T.wa * ga.x + wv * x.x, T.wa * ga.y + wv * x.y, T.wa * ga.z + wv * x.z);
    };
    // place of a vertex in LDS, -1: not the node's, or of another pass
    auto place = [&](int32_t vi) {
        const uint32_t i = (uint32_t)vi - (uint32_t)(m0 + c0);
        return i < (uint32_t)(M - c0 < LDS ? M - c0 : LDS) ? (int)i : -1;
    };
    // adds of one step go to distinct places
    auto add = [&](int i, float3 d) {
        gx[i] += d.x;
        gy[i] += d.y;
        gz[i] += d.z;
    };
    auto add_any = [&](int32_t vi, float3 d) {
        if (vi < m0 || vi >= m1) return;
        if (!lds) {
            add3(P.dldx + 3 * (int64_t)vi, d, 1.f);
        } else if (const int i = place(vi); i >= 0) {
            atomicAdd(&gx[i], d.x);
            atomicAdd(&gy[i], d.y);
            atomicAdd(&gz[i], d.z);
        }
    };
    if (!lds) {
        for (int64_t i = 3 * m0 + lane; i < 3 * m1; i += 64) P.dldx[i] = 0.f;
        __threadfence();
    }
    for (c0 = 0; c0 < M; c0 += lds ? LDS : M) {
        const bool first = c0 == 0;
        const int mc = M - c0 < LDS ? M - c0 : LDS;
        if (lds)
            for (int i = lane; i < mc; i += 64) gx[i] = gy[i] = gz[i] = 0.f;
        __syncthreads();
        // hole fans of the node
        for (int64_t t = f0 + lane; t < f1; t += 64) {
            const Tri T = tri_at(t, first, false);
            if (grad) {
                add_any(T.i0, corner(T, T.b, T.c));
                add_any(T.i1, corner(T, T.c, T.a));
                add_any(T.i2, corner(T, T.a, T.b));
            }
        }
        __syncthreads();
        // bands of the incident struts (terms at the lower end)
        for (int h = 0; h < v; ++h) {
            const int64_t b0 = ((int64_t)__builtin_amdgcn_readlane((int)(my_b0 >> 32), h) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((int)my_b0, h);
            const int nb = __builtin_amdgcn_readlane(my_nb, h), own = __builtin_amdgcn_readlane(my_own, h);
            const bool lower = __builtin_amdgcn_readlane(my_lower, h) != 0;
            for (int base = 0; base < nb; base += 64) {
                const int l = base + lane;
                const bool act = l < nb;
                // the lower end's edges come first, run u, u'; then the
                // upper end's, u', u
                const bool edge = act && (lower ? l < own : l >= nb - own);
                const bool other = act && !edge;
                // an edge triangle adds at its edge's ends (corners 0 and 1),
                // the other loop's at its apex: turned, its corner 0
                Tri T;
                float3 g0 = make_float3(0.f, 0.f, 0.f), g1 = g0;
                T.i0 = T.i1 = -1;
                if (act) {
                    T = tri_at(b0 + l, lower && first, other);
                    g0 = corner(T, T.b, T.c);
                    g1 = corner(T, T.c, T.a);
                }
                if (!grad) continue;
                if (!lds) {
                    if (act) {
                        add_any(T.i0, g0);
                        if (edge) add_any(T.i1, g1);
                    }
                    continue;
                }
                const int p0 = edge ? place(lower ? T.i0 : T.i1) : -1, p1 = edge ? place(lower ? T.i1 : T.i0) : -1;
                if (p0 >= 0) add(p0, lower ? g0 : g1);
                __syncthreads();
                if (p1 >= 0) add(p1, lower ? g1 : g0);
                __syncthreads();
                // runs of equal apexes among the other loop's edges
                const int pa = other ? place(T.i0) : -1;
                const int pp = __shfl_up(pa, 1, 64);
                const bool head = lane == 0 || pa != pp;
                const unsigned long long hm = __ballot(head);
                const int lead = 63 - __clzll(hm & ((2ull << lane) - 1)), rank = lane - lead;
                float3 x = g0;
                for (int d = 1; __ballot(pa >= 0 && rank >= d) != 0; d <<= 1) {
                    const float3 y = make_float3(__shfl_up(x.x, d, 64), __shfl_up(x.y, d, 64), __shfl_up(x.z, d, 64));
                    if (rank >= d) {
                        x.x += y.x;
                        x.y += y.y;
                        x.z += y.z;
                    }
                }
                // the run's last lane has its sum; the loop closes, so the
                // first run and the last one may be of one vertex
                const bool tail = pa >= 0 && (lane == 63 || ((hm >> lane) >> 1 & 1));
                const unsigned long long om = __ballot(pa >= 0);
                const int lead0 = om ? __builtin_ctzll(om) : 0;
                if (tail && lead != lead0) add(pa, x);
                __syncthreads();
                if (tail && lead == lead0) add(pa, x);
                __syncthreads();
            }
        }
        __syncthreads();
        // sum of squared norms over the node's vertices
        const int done = lds ? mc : M;
        for (int i = lane; i < done; i += 64) {
            const float3 x = f3(P.xyz + 3 * (m0 + c0 + i));
            sq += (double)x.x * x.x + (double)x.y * x.y + (double)x.z * x.z;
            float *d = P.dldx + 3 * (m0 + c0 + i);
            if (lds) {
                d[0] = gx[i] + 2.f * P.w_sq * x.x;
                d[1] = gy[i] + 2.f * P.w_sq * x.y;
                d[2] = gz[i] + 2.f * P.w_sq * x.z;
            } else {
                atomicAdd(d, 2.f * P.w_sq * x.x);
                atomicAdd(d + 1, 2.f * P.w_sq * x.y);
                atomicAdd(d + 2, 2.f * P.w_sq * x.z);
            }
        }
        __syncthreads();
    }
    for (int o = 32; o > 0; o >>= 1) {
        area += __shfl_xor(area, o, 64);
        vol += __shfl_xor(vol, o, 64);
        sq += __shfl_xor(sq, o, 64);
    }
    if (lane == 0) {  // the node's terms; summed in a fixed order by k_loss_reduce
        nt[0] = 0.5 * area;
        nt[1] = vol / 6.0;
        nt[2] = sq;
    }
}

// per-node terms -> terms, in an order that does not depend on scheduling:
// block b sums the nodes of its contiguous slice (thread t takes every
// kBlock-th node of the slice in turn, then a fixed tree) into partial b;
// one block then adds the kLossParts partials by the same fixed tree.
constexpr int kLossParts = 256;

__device__ inline void block_tree3(double a, double b, double c, double *out)
{
    __shared__ double s[3][kBlock];
    const int t = threadIdx.x;
    s[0][t] = a;
    s[1][t] = b;
    s[2][t] = c;
    __syncthreads();
    for (int h = kBlock / 2; h > 0; h >>= 1) {
        if (t < h) {
            s[0][t] += s[0][t + h];
            s[1][t] += s[1][t + h];
            s[2][t] += s[2][t + h];
        }
        __syncthreads();
    }
    if (t < 3) out[t] = s[t][0];
}

__global__ void __launch_bounds__(256) k_loss_partial(int64_t N, const double *node_terms, double *partial)
{
    const int64_t slice = (N + kLossParts - 1) / kLossParts;
    const int64_t n0 = (int64_t)blockIdx.x * slice, n1 = n0 + slice < N ? n0 + slice : N;
    double a = 0.0, b = 0.0, c = 0.0;
    for (int64_t n = n0 + threadIdx.x; n < n1; n += kBlock) {
        a += node_terms[3 * n];
        b += node_terms[3 * n + 1];
        c += node_terms[3 * n + 2];
    }
    block_tree3(a, b, c, partial + 3 * blockIdx.x);
}

__global__ void __launch_bounds__(256) k_loss_reduce(const double *partial, double *terms)
{
    const int t = threadIdx.x;
    double a = 0.0, b = 0.0, c = 0.0;
    for (int i = t; i < kLossParts; i += kBlock) {
        a += partial[3 * i];
        b += partial[3 * i + 1];
        c += partial[3 * i + 2];
    }
    block_tree3(a, b, c, terms);
}

__global__ void k_zero_d(double *p, int n)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0.0;
}

// ---------------------------------------------------------------------------
// per-node adjoint

struct BParams {
    Inputs in;
    Work w;
    const float *dldx;  // [M][3]
    float *grad_xyz;    // [N][3]
    float *grad_r;      // [N]
};

// The adjoint's per-node scratch in LDS, for nodes of up to VM struts, AC
// arcs and VC vertices.
template <int VM, int AC, int VC>
struct BwdLds {
    SL<float> S[VM + 1];
    uint4 v[VC];            // name, x, y, z
    float vert[VC][9];      // adjoint parts left by the vertex's three arc ends; then
                            // the weights of its three labels, x, y, z, -1
    float arc[AC][9];       // circular arcs: part of their contour's barycentre, number of
                            // segments; then circles: adjoint of o, a, b; ellipses: of
                            // g_p, h_p, g_q, h_q
    float hole[AC][4];      // per contour: barycentre sum, segments; then mu
    float gh[VM][4];        // per strut: adjoint of g, h
    float conic[VM][9];     // per strut: sums of its circles' o, a, b
    uint32_t ent[2 * AC];   // loop entries: arc | start vertex << 8 | its label's place << 16 | kEnt*
    int base[VM + 1];       // first loop entry of each strut, and their number
};
constexpr uint32_t kEntCircle = 1u << 20, kEntSideQ = 1u << 21, kEntVertex = 1u << 22;

template <int CTRL, int ROWS = 0xf>
__device__ inline float dpp_add(float x)
{
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROWS, 0xf, true));
}
// sum of x over the wave, in every lane (row_shr 1, 2, 4, 8, row_bcast 15, 31)
__device__ inline float wave_sum(float x)
{
    x = dpp_add<0x111>(x);
    x = dpp_add<0x112>(x);
    x = dpp_add<0x114>(x);
    x = dpp_add<0x118>(x);
    x = dpp_add<0x142, 0xa>(x);
    x = dpp_add<0x143, 0xc>(x);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

template <int CTRL, int ROWS = 0xf>
__device__ inline double dpp_add(double x)
{
    return x + __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xf, true),
                                __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xf, true));
}
__device__ inline double wave_sum(double x)
{
    x = dpp_add<0x111>(x);
    x = dpp_add<0x112>(x);
    x = dpp_add<0x114>(x);
    x = dpp_add<0x118>(x);
    x = dpp_add<0x142, 0xa>(x);
    x = dpp_add<0x143, 0xc>(x);
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63),
                            __builtin_amdgcn_readlane(__double2loint(x), 63));
}

// 1 / x and 1 / sqrt(x) to some 48 bits: the hardware's estimate of 24, one
// Newton step
__device__ inline double rcp64(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    return fma(fma(-x, r, 1.0), r, r);
}
__device__ inline double rsq64(double x)
{
    const double r = __builtin_amdgcn_rsq(x);
    return fma(fma(-x * r, r, 1.0), 0.5 * r, r);
}

template <typename A, typename B>
__device__ inline auto dotf(const A *a, const B *b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; }
template <typename A, typename B, typename C>
__device__ inline void crs(const A *a, const B *b, C *c)
{
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}

// The adjoint of node n's mesh vertices, by one wave.  Writes the node's own
// input adjoint to grad_node[n] and, for every incident strut, the part that
// belongs to the far node's inputs to grad_he at the strut's half-edge here;
// k_grad_gather adds them up per node in a fixed order (no atomics between
// nodes, so the gradient's bits do not depend on scheduling).
//
// Lanes go over arcs, contours, vertices, (strut, input) pairs and struts in
// turn, and what one of them adds to another is stored at a place of its own
// and gathered: the forward pass leaves every vertex with the ends of three
// arcs, one for each pair of its labels, and every strut's end loop with all
// arcs and vertices that carry its label.  (Adding through LDS atomics, some
// 50 instructions of 60 cycles of the compute unit's LDS each, the kernel
// kept that unit busy for 82 % of its time.)  The strut table is taken in
// reverse too, a lane per strut.  Octet 32^3, k = 16: 654 -> 401 us,
// 420 with the parts that are in FP64.
template <int VM, int AC, int VC>
__device__ void backward_node(const BParams &P, BwdLds<VM, AC, VC> &sm, const int64_t n)
{
    static_assert(VM <= 64 && AC <= 256 && VC <= 256, "a lane per strut; entries hold 8-bit arcs and vertices");
    constexpr int NA = (AC + 63) / 64, NV = (VC + 63) / 64;
    auto &S = sm.S;
    const Work &W = P.w;
    const int64_t N = P.in.n_nodes;
    const int lane = threadIdx.x;
    const int64_t rb = W.node_rec[n];
    // the forward pass or the loss skipped writes: no usable mesh (the
    // gather then writes zeros)
    if (W.flags[0] & (DF_CAPACITY | DF_RECCAP)) return;
    if (rb < 0) return;
    const uint32_t *R = W.rec + rb;
    const int V = (int)R[0], E = (int)R[1], NC = (int)R[2], ncirc = (int)R[3];
    const int wsum = (int)R[4], M = (int)R[5];
    const int nent = (int)((R[7] >> 8) & 0xffffu);
    const bool wide = (R[7] & kRecWide) != 0;
    const uint32_t *RV = R + kRecHead;
    const uint32_t *RA = RV + 4 * V;
    const uint32_t *RH = RA + kRecArcFields * E;
    const uint32_t *RT = R + rec_table_word(V, E, NC + wsum - V);
    const int64_t row = W.row[n];
    const int v = (int)(W.row[n + 1] - row);
    const int64_t moff = W.node_off[(int64_t)NC_MESH * (N + 1) + n];
    const float4 c4 = W.node4[n];
    const float rho = c4.w;
    const float *L = P.dldx + 3 * moff;
    // adjoint of this node's x, y, z and radius: this lane's share.  The
    // radius's terms all but cancel: added up in FP64.
    float own[3] = {0.f, 0.f, 0.f};
    double own_r = 0.0;

    // ---- strut table, vertices, arcs ---------------------------------------
    if (lane < v) {
        const int2 he = W.he[row + lane];
        const float4 f4 = W.node4[he.x];
        bool bad;
        SL<float> s = strut_entry(v3(c4.x, c4.y, c4.z), rho, v3(f4.x, f4.y, f4.z), f4.w, (int)((int64_t)he.x > n), bad);
        s.far = he.x;
        S[lane + 1] = s;
    }
    for (int i = lane; i < V; i += 64) sm.v[i] = *(const uint4 *)(RV + 4 * i);
    auto tab = [&](int i) { return wide ? (int)((const uint16_t *)RT)[i] : (int)((const uint8_t *)RT)[i]; };
    for (int i = lane; i <= v; i += 64) sm.base[i] = tab(i);
    float o[NA][3], a[NA][3], b[NA][3], t1[NA], dt[NA];
    uint32_t w11[NA], w12[NA], w13[NA];
    int mb[NA];
#pragma unroll
    for (int t = 0; t < NA; ++t) {
        const int j = lane + 64 * t;
        w11[t] = w12[t] = 0;
        w13[t] = 0xffff0001u;  // one segment, no contour
        mb[t] = 0;
        t1[t] = dt[t] = 0.f;
        for (int d = 0; d < 3; ++d) o[t][d] = a[t][d] = b[t][d] = 0.f;
        if (j >= E) continue;
        const uint4 *q = (const uint4 *)(RA + kRecArcFields * j);
        const uint4 q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
        auto f = [](uint32_t x) { return __uint_as_float(x); };
        o[t][0] = f(q0.x); o[t][1] = f(q0.y); o[t][2] = f(q0.z);
        a[t][0] = f(q0.w); a[t][1] = f(q1.x); a[t][2] = f(q1.y);
        b[t][0] = f(q1.z); b[t][1] = f(q1.w); b[t][2] = f(q2.x);
        t1[t] = f(q2.y); dt[t] = f(q2.z);
        w11[t] = q2.w; w12[t] = q3.x; w13[t] = q3.y;
        mb[t] = (int)q3.z;
    }
    // absolute positions are c + w: every mesh vertex of the node moves with c
#pragma unroll 4
    for (int i = lane; i < M; i += 64)
        for (int d = 0; d < 3; ++d) own[d] += L[3 * i + d];
    __syncthreads();

    // what the gather over the end loops reads of each entry
    for (int e = lane; e < nent; e += 64) {
        const uint32_t ea = (uint32_t)tab(v + 1 + e);
        const int j = (int)(ea & (wide ? 0x7fffu : 0x7fu));
        const bool along = (ea & (wide ? 0x8000u : 0x80u)) != 0;
        const uint32_t pq = RA[kRecArcFields * j + 11], ends = RA[kRecArcFields * j + 12];
        int m = 1;
        while (sm.base[m] <= e) ++m;  // entries of strut m: base[m - 1] .. base[m] - 1
        const uint32_t vi = along ? ends & 0xffffu : ends >> 16, name = sm.v[vi].x;
        const uint32_t place = (name >> 24) == (uint32_t)m ? 0u : (((name >> 16) & 0xffu) == (uint32_t)m ? 1u : 2u);
        sm.ent[e] = (uint32_t)j | (vi << 8) | (place << 16) | (j < ncirc ? kEntCircle : 0u) |
                    (((pq >> 8) & 0xffu) == (uint32_t)m ? kEntSideQ : 0u) | (((pq >> 16) & 1u) ? 0u : kEntVertex);
    }

    // ---- interior points ----------------------------------------------------
    // x_i = o + a sin t_i + b cos t_i, t_i = t1 + f dt, f = i / nseg.  For the
    // circular arcs also what the contour's mu will add: it is the same at
    // all of their points.
    float acc[NA][9], lt1[NA], lt2[NA], sn1[NA], cs1[NA], snf[NA], csf[NA];
#pragma unroll
    for (int t = 0; t < NA; ++t) {
        const int j = lane + 64 * t;
        for (int f = 0; f < 9; ++f) acc[t][f] = 0.f;
        lt1[t] = lt2[t] = sn1[t] = cs1[t] = snf[t] = csf[t] = 0.f;
        if (j >= E) continue;
        const int nseg = (int)(w13[t] & 0xffffu);
        const bool fwd = (w11[t] >> 17) & 1u;
        const float *Li = L + 3 * (mb[t] + (fwd ? 0 : nseg - 2));
        const int step = fwd ? 3 : -3;
        for (int ii = 1; ii < nseg; ++ii, Li += step) {
            const float lam[3] = {Li[0], Li[1], Li[2]};
            const float f = (float)ii / (float)nseg;
            float sn, cs;
            sincos_f32(t1[t] + dt[t] * f, &sn, &cs);
            float g = 0.f;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                acc[t][d] += lam[d];
                acc[t][3 + d] += lam[d] * sn;
                acc[t][6 + d] += lam[d] * cs;
                g += lam[d] * (a[t][d] * cs - b[t][d] * sn);
            }
            lt1[t] += (1.f - f) * g;
            lt2[t] += f * g;
            sn1[t] += sn;
            cs1[t] += cs;
            snf[t] += f * sn;
            csf[t] += f * cs;
        }
        if (j < ncirc) {
            const uint4 vs = sm.v[w12[t] & 0xffffu], ve = sm.v[w12[t] >> 16];
            const float es[3] = {__uint_as_float(vs.y), __uint_as_float(vs.z), __uint_as_float(vs.w)};
            const float ee[3] = {__uint_as_float(ve.y), __uint_as_float(ve.z), __uint_as_float(ve.w)};
            for (int d = 0; d < 3; ++d)
                sm.arc[j][d] = 0.5f * (es[d] + ee[d]) + ((float)(nseg - 1) * o[t][d] + a[t][d] * sn1[t] + b[t][d] * cs1[t]);
            sm.arc[j][3] = (float)nseg;
        }
    }
    __syncthreads();

    // ---- hole centres (Eq. 13) ----------------------------------------------
    // sums over the arcs of each contour: four lanes per contour
    for (int c0 = 0; c0 < NC; c0 += 16) {
        const int ci = lane >> 2, d = lane & 3, nc = NC - c0 < 16 ? NC - c0 : 16;
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < NA; ++t) {
            const int rel = (int)(w13[t] >> 16) - c0;  // 0xffff: no contour
            unsigned long long mine = 0;
            for (int i = 0; i < nc; ++i) {
                const unsigned long long m = __ballot(rel == i);
                if (ci == i) mine = m;
            }
            while (mine) {
                sum += sm.arc[64 * t + __ffsll(mine) - 1][d];
                mine &= mine - 1;
            }
        }
        if (ci < nc) sm.hole[c0 + ci][d] = sum;
    }
    __syncthreads();
    float lse[3] = {0.f, 0.f, 0.f};  // adjoint of the sum of the struts' e
    bool any_se = false;
    for (int c = lane; c < NC; c += 64) {
        const float *lp = L + 3 * (wsum + c);
        const float lh[3] = {lp[0], lp[1], lp[2]};
        const float hc[3] = {__uint_as_float(RH[3 * c]), __uint_as_float(RH[3 * c + 1]), __uint_as_float(RH[3 * c + 2])};
        const float sum[3] = {sm.hole[c][0], sm.hole[c][1], sm.hole[c][2]}, cnt = sm.hole[c][3];
        const float sl = sqrtf(dotf(sum, sum));
        // One strut: the hole is its whole circle, the barycentre rho sigma e,
        // and the direction is e's whatever sigma is; through the barycentre
        // rounding grows by 1 / sigma (radii alike to 1e-3: 1 % of the
        // gradient).
        const bool use_b = v > 1 && sl >= 1e-3f * rho * cnt;
        // dir = sgn b / |b|, or -sgn se / |se|: the sign is that of the
        // forward pass's centre
        float base[3], len = sl;
        for (int d = 0; d < 3; ++d) base[d] = sum[d];
        if (!use_b) {
            float se[3] = {0.f, 0.f, 0.f};
            for (int m = 1; m <= v; ++m) {
                se[0] += S[m].ex;
                se[1] += S[m].ey;
                se[2] += S[m].ez;
            }
            len = sqrtf(dotf(se, se));
            for (int d = 0; d < 3; ++d) base[d] = se[d];
        }
        const float sgn = dotf(hc, base) < 0.f ? -1.f : 1.f;
        float dir[3], mu[3];
        for (int d = 0; d < 3; ++d) dir[d] = sgn * base[d] / len;
        const float dl = dotf(dir, lh);
        own_r += dl;  // apex rho * dir
        for (int d = 0; d < 3; ++d) mu[d] = sgn * rho * (lh[d] - dir[d] * dl) / len;
        for (int d = 0; d < 3; ++d) {
            // the sum's length is cnt |b|, so this is 1 / cnt per vertex
            sm.hole[c][d] = use_b ? mu[d] : 0.f;
            if (!use_b) lse[d] += mu[d];
        }
        any_se |= !use_b;
    }
    if (__ballot(any_se))
        for (int d = 0; d < 3; ++d) lse[d] = wave_sum(lse[d]);
    __syncthreads();

    // ---- arc ends: t1, t2 are the parameters of the end vertices ------------
#pragma unroll
    for (int t = 0; t < NA; ++t) {
        const int j = lane + 64 * t;
        if (j >= E) continue;
        const int p = (int)(w11[t] & 0xffu), q = (int)((w11[t] >> 8) & 0xffu);
        const int vs = (int)(w12[t] & 0xffffu), ve = (int)(w12[t] >> 16);
        float mu[3] = {0.f, 0.f, 0.f};
        if (j < ncirc) {
            // mu at every interior point
            const float *h = sm.hole[w13[t] >> 16];
            const float cnt = (float)((w13[t] & 0xffffu) - 1u);
            float g = 0.f, gf = 0.f;
            for (int d = 0; d < 3; ++d) {
                mu[d] = h[d];
                acc[t][d] += cnt * mu[d];
                acc[t][3 + d] += mu[d] * sn1[t];
                acc[t][6 + d] += mu[d] * cs1[t];
                g += mu[d] * (a[t][d] * cs1[t] - b[t][d] * sn1[t]);
                gf += mu[d] * (a[t][d] * csf[t] - b[t][d] * snf[t]);
            }
            lt1[t] += g - gf;
            lt2[t] += gf;
        }
        if ((w11[t] >> 16) & 1u) {
            // whole conic: the start vertex is its point at t = 0, o + b
            for (int d = 0; d < 3; ++d) {
                const float l = L[3 * vs + d] + mu[d];
                acc[t][d] += l;
                acc[t][6 + d] += l;
            }
        } else {
            const float iaa = 1.f / dotf(a[t], a[t]), ibb = 1.f / dotf(b[t], b[t]);
#pragma unroll
            for (int end = 0; end < 2; ++end) {
                const float Lt = end ? lt2[t] : lt1[t];
                const int vi = end ? ve : vs;
                const uint4 w = sm.v[vi];
                const float r[3] = {__uint_as_float(w.y) - o[t][0], __uint_as_float(w.z) - o[t][1],
                                    __uint_as_float(w.w) - o[t][2]};
                const float u = dotf(r, a[t]) * iaa, vv = dotf(r, b[t]) * ibb;
                const float k = Lt / (u * u + vv * vv);
                const float lu = k * vv * iaa, lv = -k * u * ibb;
                // the place of the arc's pair of labels among the vertex's
                const uint32_t np = w.x >> 24, nq = (w.x >> 16) & 0xffu;
                const int place = (uint32_t)q == nq ? 0 : ((uint32_t)p == np ? 1 : 2);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const float lw = lu * a[t][d] + lv * b[t][d];
                    sm.vert[vi][3 * place + d] = lw + 0.5f * mu[d];
                    acc[t][d] -= lw;
                    // u = (r . a) / (a . a): du/da = (r - 2 u a) / aa
                    acc[t][3 + d] += lu * (r[d] - 2.f * u * a[t][d]);
                    acc[t][6 + d] += lv * (r[d] - 2.f * vv * b[t][d]);
                }
            }
        }
        if (j < ncirc) {
            for (int f = 0; f < 9; ++f) sm.arc[j][f] = acc[t][f];
            continue;
        }
        // ---- ellipse (p, q), Eq. 7, in reverse mode: the steps of the
        // conic's construction (plane p = q, in-plane axis u1, the completed
        // square) are recomputed, then their adjoints taken in reverse order.
        // Inputs: g_p, h_p, g_q, h_q and rho (kappa_p and sigma_p follow from
        // g_p, h_p and rho, so 1 - |in-plane g_p|^2 = (g_p . n)^2 - (h_p / rho)^2).
        // In FP64 from the FP32 record and table: what is left of a node's
        // radius gradient are small differences of these terms (cubic 9^3, k =
        // 10: error 2.9e-7 of its norm, with FP32 here and in own_r 3.3e-7; octet
        // 32^3: kernel 400 -> 416 us).
        // u1 is the record's own, a / |a|: computed again it turns by a rounding
        // over |gam|, and with it the frame that a, b and their adjoints are in
        // (two struts 2.2e-4 from in line: gradient off by 1.4e-3 of the sum of
        // all |lambda| instead of 2e-6).
        const SL<float> &Sp = S[p], &Sq = S[q];
        const double gp[3] = {Sp.gx, Sp.gy, Sp.gz}, hp = Sp.h, ir = rcp64((double)rho);
        const double nv[3] = {gp[0] - Sq.gx, gp[1] - Sq.gy, gp[2] - Sq.gz};
        const double inn = rsq64(dotf(nv, nv));
        double nh[3], gam[3], u1[3], tv[3] = {0.0, 0.0, 0.0};
        for (int d = 0; d < 3; ++d) nh[d] = nv[d] * inn;
        const double d0 = (hp - Sq.h) * inn, gpn = dotf(gp, nh), hr = hp * ir;
        const double om = gpn * gpn - hr * hr;
        for (int d = 0; d < 3; ++d) u1[d] = a[t][d];
        const double a2 = dotf(u1, u1);
        if (!(om > 0.0) || !(a2 > 0.0)) {  // not an ellipse: the forward pass kept no arc of it
            for (int f = 0; f < 8; ++f) sm.arc[j][f] = 0.f;
            continue;
        }
        const double iom = rcp64(om), ia = rsq64(a2);
        for (int d = 0; d < 3; ++d) {
            u1[d] *= ia;
            gam[d] = gp[d] - nh[d] * gpn;
        }
        const double gl2 = dotf(gam, gam), igl = gl2 > 0.0 ? rsq64(gl2) : 0.0, gl = gl2 * igl;
        const bool axis_from_g = gl2 > 1e-8 * dotf(gp, gp);
        double il = igl;  // 1 / length of the vector that u1 is normalised from
        if (!axis_from_g) {
            double x[3];
            tv[fabs(nh[0]) < 0.9 ? 0 : 1] = 1.0;
            crs(nh, tv, x);
            il = rsq64(dotf(x, x));
        }
        const double k0 = d0 * gpn - hp, ko = k0 * iom, al0 = gl * ko;
        const double R2 = (double)rho * rho - d0 * d0 + k0 * ko;
        const double iR = R2 > 0.0 ? rsq64(R2) : 0.0, Rr = R2 * iR, isom = rsq64(om), A = Rr * isom;
        double cv[3];
        crs(u1, nh, cv);
        // o = d0 nh + al0 u1, a = A u1, b = R (u1 x nh)
        const float *Lo = acc[t], *La = acc[t] + 3, *Lb = acc[t] + 6;
        double L_nh[3], L_u1[3], L_c[3], tmp[3];
        for (int d = 0; d < 3; ++d) {
            L_nh[d] = Lo[d] * d0;
            L_u1[d] = Lo[d] * al0 + La[d] * A;
            L_c[d] = Lb[d] * Rr;
        }
        double L_d0 = dotf(Lo, nh);
        const double L_al0 = dotf(Lo, u1), L_A = dotf(La, u1), L_R = dotf(Lb, cv) + L_A * isom;
        crs(nh, L_c, tmp);
        for (int d = 0; d < 3; ++d) L_u1[d] += tmp[d];
        crs(L_c, u1, tmp);
        for (int d = 0; d < 3; ++d) L_nh[d] += tmp[d];
        // A = R / sqrt(om), R = sqrt(max(R2, 0))
        double L_om = -0.5 * L_A * A * iom;
        const double L_R2 = 0.5 * L_R * iR;
        // R2 = rho^2 - d0^2 + k0^2 / om, al0 = gl k0 / om, k0 = d0 gpn - hp
        double L_rho = 2.0 * rho * L_R2;
        L_d0 -= 2.0 * d0 * L_R2;
        const double L_gl = ko * L_al0, L_k0 = 2.0 * ko * L_R2 + gl * iom * L_al0;
        L_om -= ko * ko * L_R2 + al0 * iom * L_al0;
        L_d0 += gpn * L_k0;
        double L_gpn = d0 * L_k0, L_hp = -L_k0;
        // u1: gam / |gam| (the re-projection and renormalisation have zero
        // derivative: u1 stays a unit vector in the plane), else the unit
        // vector along nh x t
        double L_gam[3];
        const double uu = dotf(u1, L_u1);
        for (int d = 0; d < 3; ++d) L_gam[d] = gam[d] * (L_gl * igl);
        for (int d = 0; d < 3; ++d) L_u1[d] = (L_u1[d] - u1[d] * uu) * il;
        if (axis_from_g) {
            for (int d = 0; d < 3; ++d) L_gam[d] += L_u1[d];
        } else {
            crs(tv, L_u1, tmp);
            for (int d = 0; d < 3; ++d) L_nh[d] += tmp[d];
        }
        // gam = g_p - nh gpn
        double L_gp[3];
        L_gpn -= dotf(L_gam, nh);
        for (int d = 0; d < 3; ++d) {
            L_gp[d] = L_gam[d];
            L_nh[d] -= gpn * L_gam[d];
        }
        // om = gpn^2 - (h_p / rho)^2
        L_gpn += 2.0 * gpn * L_om;
        L_hp -= 2.0 * hr * ir * L_om;
        L_rho += 2.0 * hr * hr * ir * L_om;
        // gpn = g_p . nh
        for (int d = 0; d < 3; ++d) {
            L_gp[d] += nh[d] * L_gpn;
            L_nh[d] += gp[d] * L_gpn;
        }
        // d0 = (h_p - h_q) / |n|, nh = n / |n|, n = g_p - g_q
        const double L_dn = L_d0 * inn, L_nn = -d0 * L_dn - dotf(nh, L_nh) * inn;
        for (int d = 0; d < 3; ++d) {
            const double L_n = L_nh[d] * inn + nh[d] * L_nn;
            sm.arc[j][d] = (float)(L_gp[d] + L_n);
            sm.arc[j][4 + d] = (float)-L_n;
        }
        sm.arc[j][3] = (float)(L_hp + L_dn);
        sm.arc[j][7] = (float)-L_dn;
        own_r += L_rho;
    }
    __syncthreads();

    // ---- vertices: implicit function theorem on the tie equations ------------
    // F1 = (g_p - g_q) . w - (h_p - h_q), F2 = (g_p - g_r) . w - (h_p - h_r),
    // F3 = g_p . w - h_p - s, F4 = |w|^2 - rho^2 - s^2 (label 0: g = 0, h = 0).
    // J^T mu = (lam_w, 0) gives mu3 = -2 s mu4 and
    // [n1 | n2 | 2 (w - s g_p)] (mu1, mu2, mu4) = lam_w.
    // In FP64: in FP32 the solve's own rounding, grown by the tie's condition, is
    // what the least well conditioned nodes of a lattice leave in its gradient
    // (cubic 9^3, k = 10, radius gradient, the worst of 60: error 11.4e-7 of its
    // norm, 4.3e-7 so; octet 32^3: kernel +4 us).
#pragma unroll
    for (int t = 0; t < NV; ++t) {
        const int i = lane + 64 * t;
        if (i >= V) continue;
        const uint4 vw = sm.v[i];
        const int p = (int)(vw.x >> 24), q = (int)((vw.x >> 16) & 0xffu), r = (int)((vw.x >> 8) & 0xffu);
        if (r == 0xff) continue;  // start point of a whole conic (handled with its arc)
        const double w[3] = {__uint_as_float(vw.y), __uint_as_float(vw.z), __uint_as_float(vw.w)};
        double gp[3] = {0.0, 0.0, 0.0}, hp = 0.0;
        if (p) {
            gp[0] = S[p].gx; gp[1] = S[p].gy; gp[2] = S[p].gz;
            hp = S[p].h;
        }
        const double gq[3] = {S[q].gx, S[q].gy, S[q].gz}, gr[3] = {S[r].gx, S[r].gy, S[r].gz};
        const double s = dotf(gp, w) - hp;
        double n1[3], n2[3], n3[3], lw[3];
        for (int d = 0; d < 3; ++d) {
            n1[d] = gp[d] - gq[d];
            n2[d] = gp[d] - gr[d];
            n3[d] = 2.0 * (w[d] - s * gp[d]);
            lw[d] = (double)L[3 * i + d] + sm.vert[i][d] + sm.vert[i][3 + d] + sm.vert[i][6 + d];
        }
        // Cramer on columns n1, n2, n3
        double x23[3], x31[3], x12[3];
        crs(n2, n3, x23);
        crs(n3, n1, x31);
        crs(n1, n2, x12);
        const double idt = rcp64(dotf(n1, x23));
        const double mu1 = dotf(lw, x23) * idt;
        const double mu2 = dotf(lw, x31) * idt;
        const double mu4 = dotf(lw, x12) * idt;
        const double mu3 = -2.0 * s * mu4;
        // dL/dtheta = -mu^T dF/dtheta: label m's g gets weight * w, its h -weight
        sm.vert[i][0] = (float)-(mu1 + mu2 + mu3);
        sm.vert[i][1] = (float)mu1;
        sm.vert[i][2] = (float)mu2;
        for (int d = 0; d < 3; ++d) sm.vert[i][3 + d] = (float)w[d];
        sm.vert[i][6] = -1.f;
        own_r += 2.0 * rho * mu4;
    }
    __syncthreads();

    // ---- sums over each strut's end loop: its arcs and their start vertices
    for (int x = lane; x < 4 * v; x += 64) {
        const int m = x >> 2, d = x & 3, dc = d < 3 ? d : 0;
        float gh = 0.f, so = 0.f, sa = 0.f, sb = 0.f;
        const int e1 = sm.base[m + 1];
#pragma unroll 2
        for (int e = sm.base[m]; e < e1; ++e) {
            const uint32_t en = sm.ent[e];
            const float *A = sm.arc[en & 0xffu], *X = sm.vert[(en >> 8) & 0xffu];
            if (en & kEntCircle) {
                so += A[dc];
                sa += A[3 + dc];
                sb += A[6 + dc];
            } else {
                gh += A[(en & kEntSideQ ? 4 : 0) + d];
            }
            if (en & kEntVertex) gh += X[(en >> 16) & 3u] * X[3 + d];
        }
        sm.gh[m][d] = gh;
        if (d < 3) {
            sm.conic[m][d] = so;
            sm.conic[m][3 + d] = sa;
            sm.conic[m][6 + d] = sb;
        }
    }
    __syncthreads();

    // ---- strut table: g, h, e, sigma, kappa, frame from the two nodes' inputs
    // Tangency circle (0, q): o = rho sigma e, a = rho kappa q^, b = rho kappa r^.
    if (lane < v) {
        const SL<float> s = S[lane + 1];
        const float *gh = sm.gh[lane], *Lo = sm.conic[lane], *La = Lo + 3, *Lb = Lo + 6;
        const float e[3] = {s.ex, s.ey, s.ez}, g[3] = {s.gx, s.gy, s.gz}, es[3] = {s.sx, s.sy, s.sz};
        const float qf[3] = {s.qx, s.qy, s.qz}, rf[3] = {s.rx, s.ry, s.rz};
        const float4 f4 = W.node4[s.far];
        const float dv[3] = {f4.x - c4.x, f4.y - c4.y, f4.z - c4.z};
        const float iL = 1.f / sqrtf(dotf(dv, dv)), ik = 1.f / s.kap;
        const float lo_e = dotf(Lo, e), lab = dotf(La, qf) + dotf(Lb, rf);
        const float lh = gh[3];
        // h = rho sigma / kappa, g = e / kappa, kappa = sqrt(1 - sigma^2)
        const float l_kap = rho * lab - (dotf(gh, g) + lh * s.h) * ik;
        const float l_sig = rho * lo_e + (lh * rho - l_kap * s.sig) * ik;
        own_r += s.sig * lo_e + s.kap * lab + lh * s.sig * ik + l_sig * iL;
        // frame: r = es x axis / |es x axis|, q = es x r
        const float ax = fabsf(es[0]), ay = fabsf(es[1]), az = fabsf(es[2]);
        const int ja = ay < ax ? (az < ay ? 2 : 1) : (az < ax ? 2 : 0);
        const float axis[3] = {ja == 0 ? 1.f : 0.f, ja == 1 ? 1.f : 0.f, ja == 2 ? 1.f : 0.f};
        float c[3], l_q[3], l_r[3], l_es[3], tmp[3];
        crs(es, axis, c);
        const float ic = 1.f / sqrtf(dotf(c, c)), rk = rho * s.kap;
        for (int d = 0; d < 3; ++d) l_q[d] = rk * La[d];
        crs(rf, l_q, l_es);
        crs(l_q, es, tmp);
        for (int d = 0; d < 3; ++d) l_r[d] = rk * Lb[d] + tmp[d];
        const float rr = dotf(rf, l_r);
        for (int d = 0; d < 3; ++d) l_r[d] = (l_r[d] - rf[d] * rr) * ic;
        crs(axis, l_r, tmp);
        // e and es = +-e along d = far - node, sigma = (rho - r_far) / |d|
        float l_e[3];
        for (int d = 0; d < 3; ++d)
            l_e[d] = gh[d] * ik + rho * s.sig * Lo[d] + lse[d] + (s.lower ? l_es[d] + tmp[d] : -(l_es[d] + tmp[d]));
        const float el = dotf(e, l_e) + s.sig * l_sig;
        float *out = W.grad_he + 4 * (row + lane);
        for (int d = 0; d < 3; ++d) {
            const float l = (l_e[d] - e[d] * el) * iL;
            out[d] = l;
            own[d] -= l;
        }
        out[3] = -l_sig * iL;
    }
    for (int d = 0; d < 3; ++d) own[d] = wave_sum(own[d]);
    own_r = wave_sum(own_r);
    if (lane == 0) *(float4 *)(W.grad_node + 4 * n) = make_float4(own[0], own[1], own[2], (float)own_r);
}

// nodes of up to kVmax struts, one block (wave) each
__global__ void __launch_bounds__(64) k_backward(BParams P)
{
    __shared__ BwdLds<kVmax, kAcap, kVcap> sm;
    const int64_t n = blockIdx.x;
    if (n >= P.in.n_nodes) return;
    if (P.w.row[n + 1] - P.w.row[n] > kVmax) return;  // k_backward_big
    backward_node(P, sm, n);
}

// nodes of the multi-wave class (queue class 3), one wave each with the
// larger capacities, a fixed grid looping over the class
__global__ void __launch_bounds__(64) k_backward_big(BParams P)
{
    __shared__ BwdLds<kVmaxBig, kAcapBig, kVcapBig> sm;
    const int64_t cnt = P.w.cls_info[3], base = P.w.cls_info[4 + 3];
    for (int64_t i = blockIdx.x; i < cnt; i += gridDim.x) {
        backward_node(P, sm, P.w.queue[base + i]);
        __syncthreads();
    }
}

// gradient of node n = its own part + the parts its neighbours wrote for
// it at the other half-edge of each incident strut, in adjacency order
__global__ void k_grad_gather(BParams P)
{
    const Work &W = P.w;
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= P.in.n_nodes) return;
    float g[4] = {0.f, 0.f, 0.f, 0.f};
    if (W.flags[0] & (DF_CAPACITY | DF_RECCAP)) {
        P.grad_xyz[3 * n] = P.grad_xyz[3 * n + 1] = P.grad_xyz[3 * n + 2] = 0.f;
        P.grad_r[n] = 0.f;
        return;
    }
    if (W.node_rec[n] >= 0)
        for (int d = 0; d < 4; ++d) g[d] = W.grad_node[4 * n + d];
    // four half-edges' loads of one kind at once: a chain of three per half-edge
    // is what takes the time (octet 32^3: 40 -> 29 us)
    constexpr int K = 4;
    const int64_t end = W.row[n + 1];
    for (int64_t h = W.row[n]; h < end; h += K) {
        int2 he[K];
        int64_t rec[K], tw[K];
        float4 d[K];
#pragma unroll
        for (int i = 0; i < K; ++i) he[i] = W.he[h + i < end ? h + i : h];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            rec[i] = W.node_rec[he[i].x];
            const int64_t h0 = W.strut_he[2 * (int64_t)he[i].y], h1 = W.strut_he[2 * (int64_t)he[i].y + 1];
            tw[i] = h0 == h + i ? h1 : h0;
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const float *q = W.grad_he + 4 * tw[i];
            d[i] = make_float4(q[0], q[1], q[2], q[3]);
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            if (h + i >= end || rec[i] < 0) continue;
            g[0] += d[i].x;
            g[1] += d[i].y;
            g[2] += d[i].z;
            g[3] += d[i].w;
        }
    }
    P.grad_xyz[3 * n] = g[0];
    P.grad_xyz[3 * n + 1] = g[1];
    P.grad_xyz[3 * n + 2] = g[2];
    P.grad_r[n] = g[3];
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }
constexpr int64_t kBigGridBwd = 1024;  // blocks of k_backward_big

}  // namespace

hipError_t launch_loss(const Inputs &in, const Work &w, const FillOut &o, float3 p0, float w_area, float w_vol,
                       float w_sq, int k, float *dldx, double *terms, hipStream_t st)
{
    if (in.n_nodes == 0) {
        k_zero_d<<<1, 64, 0, st>>>(terms, 3);
        return hipGetLastError();
    }
    LParams P;
    P.in = in;
    P.w = w;
    P.tri = o.tri;
    P.xyz = o.mesh_xyz;
    P.cap_mesh = o.cap_mesh;
    P.cap_tri = o.cap_tri;
    P.p0 = p0;
    P.w_area = w_area;
    P.w_vol = w_vol;
    P.w_sq = w_sq;
    P.dldx = dldx;
    P.terms = terms;
    // (before the nodes: they set the flag that it reads)
    if (o.cap_mesh > 0) {
        const unsigned g = grid_for(3 * o.cap_mesh);
        k_loss_rest<<<g < 2048 ? g : 2048, kBlock, 0, st>>>(P);
    }
    // Which room: a node of v struts has about v (k + 5) / 2 vertices.  The
    // larger where the mean node needs it (us, 512 / 1,024: cubic 20^3 at k =
    // 200, 580 vertices, 288 / 218; BCC 16^3 at 200, 740, 387 / 302; octet 14^3 at
    // 128, 740, 437 / 425; but at k = 64, 390, 147 / 230, and at 200, 1,150, 939 /
    // 1,004), and where all blocks fit the chip at once anyway, so that the last
    // node's second pass is what the others wait for (9-NN 14^3, the mean below
    // 512 but up to 589, 877, 1,164 at k = 64, 96, 128: 120 / 77, 171 / 101, 278 /
    // 194; at k = 16 and 32 no difference).
    const double mean = (double)in.n_struts / (double)in.n_nodes * (k + 5);
    const bool large = (mean > kLossSmall && mean <= kLossLarge) || in.n_nodes <= 256 * 12;
    if (large) k_loss_node<kLossLarge><<<(unsigned)in.n_nodes, 64, 0, st>>>(P);
    else k_loss_node<kLossSmall><<<(unsigned)in.n_nodes, 64, 0, st>>>(P);
    double *partial = w.loss_node + 3 * (in.n_nodes + 1);  // kLossParts x 3 after the node terms
    k_loss_partial<<<kLossParts, kBlock, 0, st>>>(in.n_nodes, w.loss_node, partial);
    k_loss_reduce<<<1, kBlock, 0, st>>>(partial, terms);
    return hipGetLastError();
}

hipError_t launch_backward(const Inputs &in, const Work &w, const float *dldx, float *grad_xyz, float *grad_r,
                           hipStream_t st)
{
    const int64_t N = in.n_nodes;
    if (N == 0) return hipSuccess;
    BParams P;
    P.in = in;
    P.w = w;
    P.dldx = dldx;
    P.grad_xyz = grad_xyz;
    P.grad_r = grad_r;
    k_backward<<<(unsigned)N, 64, 0, st>>>(P);
    k_backward_big<<<(unsigned)(N < kBigGridBwd ? N : kBigGridBwd), 64, 0, st>>>(P);
    k_grad_gather<<<grid_for(N), kBlock, 0, st>>>(P);
    return hipGetLastError();
}

}  // namespace lm
