// Lattice preparation (validation, node adjacency, valence queues) and the
// sizes of a mesh (band counts, prefix sums of every count, totals).
#include "common.h"

namespace lm {
namespace {

constexpr int kBlock = 256;
constexpr int kSortReg = 16;  // rows up to this length are sorted in registers

__global__ void k_pack(Inputs in, float4 *node4, int32_t *deg, int32_t *flags)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) flags[1] = 0;  // what is found below
    if (i >= in.n_nodes) return;
    node4[i] = make_float4(in.x[i], in.y[i], in.z[i], in.r[i]);
    deg[i] = 0;
}

// Runs of equal keys among neighbouring lanes of a wave (struts listed cell
// by cell share endpoints with their neighbours): the first lane of a run
// does one atomic for the whole run.  Keys of lanes without work must differ
// from every node id (negative, unique per lane).
struct Run {
    int leader, rank, len;
};
__device__ inline Run wave_run(int32_t key)
{
    const int lane = threadIdx.x & 63;
    const int32_t prev = __shfl_up(key, 1, 64);
    const bool head = lane == 0 || key != prev;
    const unsigned long long hm = __ballot(head);
    const unsigned long long upto = (2ull << lane) - 1;  // lanes 0..lane (all for lane 63)
    const int leader = 63 - __clzll(hm & upto);
    const unsigned long long above = hm & ~upto;
    const int next = above ? __ffsll(above) - 1 : 64;
    return Run{leader, lane - leader, next - leader};
}

// the two endpoint keys of strut s for the run aggregation (negative: none)
__device__ inline void strut_keys(const Inputs &in, int64_t s, int32_t &ka, int32_t &kb, bool &bad)
{
    const int lane = threadIdx.x & 63;
    ka = -1 - lane;
    kb = -1 - lane;
    bad = false;
    if (s >= in.n_struts) return;
    const int32_t a = in.sa[s], b = in.sb[s];
    if (a < 0 || b < 0 || (int64_t)a >= in.n_nodes || (int64_t)b >= in.n_nodes) {
        bad = true;
        return;
    }
    ka = a;
    if (b != a) kb = b;
}

// Degree histogram; out-of-range endpoints raise DF_BADLAT.
__global__ void k_degree(Inputs in, int32_t *deg, int32_t *flags)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int32_t ka, kb;
    bool bad;
    strut_keys(in, s, ka, kb, bad);
    if (bad) atomicOr(&flags[1], DF_BADLAT);
    const Run ra = wave_run(ka), rb = wave_run(kb);
    if (ka >= 0 && ra.rank == 0) atomicAdd(&deg[ka], ra.len);
    if (kb >= 0 && rb.rank == 0) atomicAdd(&deg[kb], rb.len);
}

__global__ void k_scatter(Inputs in, const int64_t *row, int32_t *cursor, int2 *he)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int32_t ka, kb;
    bool bad;
    strut_keys(in, s, ka, kb, bad);
    const Run ra = wave_run(ka), rb = wave_run(kb);
    int32_t ba = 0, bb = 0;
    if (ka >= 0 && ra.rank == 0) ba = atomicAdd(&cursor[ka], ra.len);
    if (kb >= 0 && rb.rank == 0) bb = atomicAdd(&cursor[kb], rb.len);
    ba = __shfl(ba, ra.leader, 64);
    bb = __shfl(bb, rb.leader, 64);
    // the order inside a row is arbitrary here; k_sort_rows fixes it
    if (ka >= 0) he[row[ka] + ba + ra.rank] = make_int2(kb >= 0 ? kb : ka, (int32_t)s);
    if (kb >= 0) he[row[kb] + bb + rb.rank] = make_int2(ka, (int32_t)s);
}

// Half-edge i of strut s at node n, in the strut's two
__device__ inline void put_half_edge(int64_t *strut_he, const int32_t *sa, const int32_t *sb, int32_t s, int64_t n,
                                     int64_t i)
{
    const int32_t a = sa[s], c = sb[s];
    const int64_t s2 = 2 * (int64_t)s;
    if (a == c) {
        strut_he[s2] = i;
        strut_he[s2 + 1] = i;
    } else {
        strut_he[s2 + (n == (a < c ? a : c) ? 0 : 1)] = i;
    }
}

// Incident struts of each node in increasing strut id (canonical labels
// 1..v), then the half-edge index of every strut at its lower and higher
// node id.  A lane per node; rows that its registers cannot hold but a wave
// can are sorted by the wave, one after the other, each lane counting what
// goes before its element.  (In memory, by one lane, the few such rows of
// k-NN 19^3 took most of the kernel: 35 -> 12 us.)
__global__ void k_sort_rows(int64_t n_nodes, const int64_t *row, int2 *he, int64_t *strut_he, const int32_t *sa,
                            const int32_t *sb)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    int64_t b = 0, e = 0;
    if (n < n_nodes) {
        b = row[n];
        e = row[n + 1];
    }
    for (unsigned long long m = __ballot(e - b > kSortReg && e - b <= 64); m; m &= m - 1) {
        const int r = __ffsll(m) - 1;
        const int64_t rb = __shfl(b, r, 64);
        const int v = __builtin_amdgcn_readlane((int)(e - b), r);
        int2 x = make_int2(0, 0x7fffffff);
        if (lane < v) x = he[rb + lane];
        int rank = 0;
        for (int i = 0; i < v; ++i) rank += __builtin_amdgcn_readlane(x.y, i) < x.y;
        if (lane < v) {
            he[rb + rank] = x;
            put_half_edge(strut_he, sa, sb, x.y, n - lane + r, rb + rank);
        }
    }
    if (n >= n_nodes || (e - b > kSortReg && e - b <= 64)) return;
    if (e - b <= kSortReg) {
        // in registers: bitonic network over kSortReg slots, empty slots last
        const int v = (int)(e - b);
        int2 x[kSortReg];
#pragma unroll
        for (int i = 0; i < kSortReg; ++i) x[i] = i < v ? he[b + i] : make_int2(0, 0x7fffffff);
#pragma unroll
        for (int k = 2; k <= kSortReg; k <<= 1) {
#pragma unroll
            for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
                for (int i = 0; i < kSortReg; ++i) {
                    const int l = i ^ j;
                    if (l > i) {
                        const bool up = (i & k) == 0;
                        const bool sw = up ? x[i].y > x[l].y : x[i].y < x[l].y;
                        const int2 lo = sw ? x[l] : x[i], hi = sw ? x[i] : x[l];
                        x[i] = lo;
                        x[l] = hi;
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kSortReg; ++i)
            if (i < v) he[b + i] = x[i];
        // half-edge ids per strut end, all endpoint loads issued at once
        int32_t lo[kSortReg];
#pragma unroll
        for (int i = 0; i < kSortReg; ++i) {
            lo[i] = 0;
            if (i < v) {
                const int32_t a = sa[x[i].y], c = sb[x[i].y];
                lo[i] = a == c ? -1 : (a < c ? a : c);
            }
        }
#pragma unroll
        for (int i = 0; i < kSortReg; ++i) {
            if (i < v) {
                const int64_t s2 = 2 * (int64_t)x[i].y;
                if (lo[i] < 0) {
                    strut_he[s2] = b + i;
                    strut_he[s2 + 1] = b + i;
                } else {
                    strut_he[s2 + (n == lo[i] ? 0 : 1)] = b + i;
                }
            }
        }
        return;
    } else {
        for (int64_t i = b + 1; i < e; ++i) {
            int2 x = he[i];
            int64_t j = i - 1;
            while (j >= b && he[j].y > x.y) {
                he[j + 1] = he[j];
                --j;
            }
            he[j + 1] = x;
        }
    }
    for (int64_t i = b; i < e; ++i) put_half_edge(strut_he, sa, sb, he[i].y, n, i);
}

// ---------------------------------------------------------------------------
// Prefix sums, int32 -> int64, in tiles of kTile elements: one launch leaves
// every tile's sum of every column, one writes the prefix sums.  In the second
// each block sums up the tiles before its own where a wave can (at most kFew
// tiles, one per lane); above that a launch between the two scans the tiles'
// sums.  Small lattices are bound by their launches (one costs 2 to 5 us,
// whatever it does), so whatever is counted over the same elements shares
// them: BCC 64^3, k = 16: preparation and sizes 23 launches -> 10; cubic 6^3:
// 21 -> 8, step 152 -> 114 us.

constexpr int kScanItems = 8;
constexpr int kTile = kBlock * kScanItems;
constexpr int kFew = 64;

inline __host__ __device__ int64_t tiles_of(int64_t n)
{
    const int64_t nb = (n + kTile - 1) / kTile;
    return nb < 1 ? 1 : nb;
}

__device__ inline int64_t wave_incl_scan(int64_t x)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int64_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Exclusive scan of one value per thread across the block; returns the
// exclusive prefix and writes the block total to *total.
__device__ inline int64_t block_excl_scan(int64_t x, int64_t *total)
{
    __shared__ int64_t wsum[kBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int64_t inc = wave_incl_scan(x);
    if (lane == 63) wsum[wid] = inc;
    __syncthreads();
    int64_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        if (w < wid) base += wsum[w];
        tot += wsum[w];
    }
    __syncthreads();
    *total = tot;
    return base + inc - x;
}

// sums over the block of up to kBlock / 64 waves' worth of several values;
// thread 0 gets them
template <int NV>
__device__ inline void block_sums(int64_t (&x)[NV])
{
    __shared__ int64_t s_x[kBlock / 64][NV];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) x[v] += __shfl_xor(x[v], d, 64);
        if (lane == 0) s_x[wid][v] = x[v];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            x[v] = 0;
            for (int w = 0; w < kBlock / 64; ++w) x[v] += s_x[w][v];
        }
    }
}

// Column sums of nb tiles, p[0 .. nb): their total, and the sum of those
// before tile b.  At most kFew: summed here by the calling wave; otherwise
// scanned already, with the total at p[nb].
__device__ inline int64_t tiles_before(const int64_t *p, int64_t nb, int64_t b, int64_t *total)
{
    if (nb > kFew) {
        *total = p[nb];
        return p[b];
    }
    const int lane = threadIdx.x & 63;
    const int64_t x = lane < nb ? p[lane] : 0, inc = wave_incl_scan(x);
    *total = __shfl(inc, 63, 64);
    return __shfl(inc - x, (int)b, 64);
}

// the tiles' sums of each column scanned in place, the total after them; one
// block per column, columns `stride` apart
__global__ void __launch_bounds__(kBlock) k_scan_tile_sums(int64_t *part, int64_t nb, int64_t stride)
{
    int64_t *p = part + blockIdx.x * stride;
    int64_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kBlock) {
        const int64_t i = b0 + threadIdx.x;
        const int64_t x = i < nb ? p[i] : 0;
        int64_t tot;
        const int64_t ex = block_excl_scan(x, &tot);
        if (i < nb) p[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) p[nb] = carry;
}

// Adjacency rows and valence queues: columns degree, then one per class.
constexpr int kRowCols = 1 + kClasses;
__global__ void __launch_bounds__(kBlock) k_rows_reduce(int64_t N, const int32_t *deg, int64_t *part, int64_t stride)
{
    const int64_t base = (int64_t)blockIdx.x * kTile;
    int64_t x[kRowCols] = {};
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t n = base + (int64_t)j * kBlock + threadIdx.x;
        if (n >= N) continue;
        const int d = deg[n], c = valence_class(d);
        x[0] += d;
#pragma unroll
        for (int k = 0; k < kClasses; ++k) x[1 + k] += k == c;
    }
    block_sums(x);
    if (threadIdx.x == 0)
        for (int c = 0; c < kRowCols; ++c) part[c * stride + blockIdx.x] = x[c];
}

// row offsets, the queue (nodes class by class, in node order) and the class
// sizes and starts; deg is cleared for k_scatter
__global__ void __launch_bounds__(kBlock) k_rows_tiles(int64_t N, int32_t *deg, const int64_t *part, int64_t nb,
                                                       int64_t stride, int64_t *row, int32_t *queue,
                                                       int64_t *cls_info)
{
    static_assert(kClasses * 16 <= 64 && kTile < 65536, "class counts of a tile are 16-bit fields of one word");
    const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kScanItems;
    int32_t d[kScanItems];
    int64_t acc = 0;
    uint64_t cls = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t n = base + j;
        d[j] = n < N ? deg[n] : 0;
        acc += d[j];
        if (n < N) cls += 1ull << (16 * valence_class(d[j]));
    }
    // this tile's sums, and those of all (the same, of one tile: no sums are
    // left by a launch before, then)
    int64_t tile, tile_cls;
    int64_t ex = block_excl_scan(acc, &tile);
    uint64_t exc = (uint64_t)block_excl_scan((int64_t)cls, &tile_cls);
    int64_t total = tile, start[kClasses], at = 0;
    if (nb > 1) ex += tiles_before(part, nb, blockIdx.x, &total);
    if (blockIdx.x == 0 && threadIdx.x == 0) row[N] = total;
#pragma unroll
    for (int k = 0; k < kClasses; ++k) {
        total = (tile_cls >> (16 * k)) & 0xffff;
        start[k] = at;
        if (nb > 1) start[k] += tiles_before(part + (1 + k) * stride, nb, blockIdx.x, &total);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            cls_info[k] = total;
            cls_info[kClasses + k] = at;
        }
        at += total;
    }
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t n = base + j;
        if (n >= N) break;
        row[n] = ex;
        deg[n] = 0;
        ex += d[j];
        const int c = valence_class(d[j]);
        int64_t s = start[0];
#pragma unroll
        for (int k = 1; k < kClasses; ++k) s = c == k ? start[k] : s;
        queue[s + (int64_t)((exc >> (16 * c)) & 0xffff)] = (int32_t)n;
        exc += 1ull << (16 * c);
    }
}

// Sizes: the node counts' columns over nodes, the band counts over struts.
// Tiles of nodes come first in the grid, then tiles of struts.
struct SizesParams {
    Inputs in;
    Work w;
    FillOut o;
    int check;          // o's capacities are checked
    OffsetsOut out;
    int64_t nbn, nbs;   // tiles of nodes, of struts
    int64_t stride;     // of the node columns in scan_tmp; the bands' sums follow them
};

__global__ void __launch_bounds__(kBlock) k_sizes_reduce(SizesParams P)
{
    const Work &W = P.w;
    const int64_t N = P.in.n_nodes, S = P.in.n_struts;
    const int32_t *status = W.node_cnt + (int64_t)NC_STATUS * N;
    int64_t x[kNodeScanCols + 1] = {};
    if (blockIdx.x < P.nbn) {
        const int64_t base = (int64_t)blockIdx.x * kTile;
#pragma unroll
        for (int j = 0; j < kScanItems; ++j) {
            const int64_t n = base + (int64_t)j * kBlock + threadIdx.x;
            if (n >= N) continue;
#pragma unroll
            for (int c = 0; c < kNodeScanCols; ++c) x[c] += W.node_cnt[c * N + n];
            x[kNodeScanCols] += status[n] != 0;
        }
        block_sums(x);
        if (threadIdx.x == 0) {
            for (int c = 0; c < kNodeScanCols; ++c) W.scan_tmp[c * P.stride + blockIdx.x] = x[c];
            if (x[kNodeScanCols]) atomicAdd((unsigned long long *)&W.totals[8], (unsigned long long)x[kNodeScanCols]);
        }
        return;
    }
    // all struts' loads of one kind at once: a chain of them per strut is what
    // takes the time (k-NN 19^3 16 -> 12 us)
    const int64_t b = blockIdx.x - P.nbn, base = b * kTile;
    int32_t u[kScanItems], v[kScanItems], c[kScanItems];
    int64_t h0[kScanItems], h1[kScanItems];
    bool ok[kScanItems];
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t s = base + (int64_t)j * kBlock + threadIdx.x;
        u[j] = v[j] = -1;
        h0[j] = h1[j] = 0;
        if (s >= S) continue;
        u[j] = P.in.sa[s];
        v[j] = P.in.sb[s];
        h0[j] = W.strut_he[2 * s];
        h1[j] = W.strut_he[2 * s + 1];
    }
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        ok[j] = u[j] != v[j] && (uint64_t)(int64_t)u[j] < (uint64_t)N && (uint64_t)(int64_t)v[j] < (uint64_t)N;
        if (ok[j]) {
            u[j] = status[u[j]];
            v[j] = status[v[j]];
            c[j] = W.he_len[h0[j]];
            h1[j] = W.he_len[h1[j]];
        }
    }
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t s = base + (int64_t)j * kBlock + threadIdx.x;
        if (s >= S) continue;
        ok[j] = ok[j] && u[j] == 0 && v[j] == 0;
        c[j] = ok[j] ? c[j] + (int32_t)h1[j] : 0;
        x[1] += !ok[j];
        x[0] += c[j];
        W.band_cnt[s] = c[j];
    }
    block_sums(x);
    if (threadIdx.x == 0) {
        W.scan_tmp[kNodeScanCols * P.stride + b] = x[0];
        if (x[1]) atomicAdd((unsigned long long *)&W.totals[9], (unsigned long long)x[1]);
    }
}

// grid y: the node columns, then the bands, then (one block) the totals
__global__ void __launch_bounds__(kBlock) k_sizes_tiles(SizesParams P)
{
    const Work &W = P.w;
    const int64_t N = P.in.n_nodes, S = P.in.n_struts;
    const int col = blockIdx.y;
    const int64_t *part = W.scan_tmp + (int64_t)col * P.stride;
    if (col <= kNodeScanCols) {
        const bool nodes = col < kNodeScanCols;
        const int64_t n = nodes ? N : S, nb = nodes ? P.nbn : P.nbs;
        if (blockIdx.x >= nb) return;
        const int32_t *src = nodes ? W.node_cnt + col * N : W.band_cnt;
        int64_t *dst = nodes ? W.node_off + col * (N + 1) : W.band_off;
        int64_t *dst2 = nodes ? P.out.node_off : P.out.strut_off;
        if (nodes && dst2) dst2 += col * (N + 1);
        // Through LDS, so that neighbouring lanes load and store neighbouring
        // elements while each thread sums eight in a row (BCC 64^3: 56 -> 21
        // us).  A tile's sum fits 32 bits: the most are band triangles, one per
        // segment of at most kAcapBig arcs at either end of each strut.
        static_assert(2ull * kAcapBig * kMaxK * kTile < 1ull << 32, "a tile's sum in 32 bits");
        __shared__ uint32_t s_v[kTile + kTile / kScanItems];
        auto slot = [](int i) { return i + i / kScanItems; };
        const int64_t base = (int64_t)blockIdx.x * kTile;
        int64_t total;
        const int64_t before = tiles_before(part, nb, blockIdx.x, &total);
#pragma unroll
        for (int j = 0; j < kScanItems; ++j) {
            const int i = j * kBlock + (int)threadIdx.x;
            s_v[slot(i)] = base + i < n ? (uint32_t)src[base + i] : 0u;
        }
        __syncthreads();
        uint32_t v[kScanItems];
        uint32_t acc = 0;
#pragma unroll
        for (int j = 0; j < kScanItems; ++j) {
            v[j] = s_v[slot((int)threadIdx.x * kScanItems + j)];
            acc += v[j];
        }
        int64_t tot;
        uint32_t ex = (uint32_t)block_excl_scan((int64_t)acc, &tot);
#pragma unroll
        for (int j = 0; j < kScanItems; ++j) {
            s_v[slot((int)threadIdx.x * kScanItems + j)] = ex;
            ex += v[j];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kScanItems; ++j) {
            const int i = j * kBlock + (int)threadIdx.x;
            if (base + i < n) {
                const int64_t x = before + s_v[slot(i)];
                dst[base + i] = x;
                if (dst2) dst2[base + i] = x;
            }
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            dst[n] = total;
            if (dst2) dst2[n] = total;
        }
        if (col == 0 && P.out.status) {
            // int32 status column -> uint8 (values fit in 8 bits)
#pragma unroll
            for (int j = 0; j < kScanItems; ++j) {
                const int64_t i = (int64_t)blockIdx.x * kTile + (int64_t)j * kBlock + threadIdx.x;
                if (i < N) P.out.status[i] = (uint8_t)W.node_cnt[(int64_t)NC_STATUS * N + i];
            }
        }
        return;
    }
    // totals and capacity checks, by one wave
    if (blockIdx.x != 0 || threadIdx.x >= 64) return;
    const int lane = threadIdx.x;
    int64_t tot[kNodeScanCols + 1];
#pragma unroll
    for (int c = 0; c <= kNodeScanCols; ++c)
        tiles_before(W.scan_tmp + c * P.stride, c < kNodeScanCols ? P.nbn : P.nbs, 0, &tot[c]);
    // record words: the fullest region times the region count
    unsigned long long top = 0;
    for (int g = lane; g < kRecRegions; g += 64) top = W.rec_top[g] > top ? W.rec_top[g] : top;
    int64_t handed = lane < 2 * kSub ? *sched_ctr(W.sched, SCHED_HAND + lane / kSub, lane % kSub) : 0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const unsigned long long y = __shfl_xor(top, d, 64);
        top = y > top ? y : top;
        handed += __shfl_xor(handed, d, 64);
    }
    if (lane != 0) return;
    const int64_t nv = tot[NC_VERT], na = tot[NC_ARC], nm = tot[NC_MESH], nf = tot[NC_FAN], nb = tot[kNodeScanCols];
    W.totals[0] = nv;
    W.totals[1] = na;
    W.totals[2] = tot[NC_HOLE];
    W.totals[3] = nm;
    W.totals[4] = nb + nf;
    W.totals[5] = nb;
    W.totals[6] = nf;
    W.totals[7] = (int64_t)top * kRecRegions * 4;
    W.totals[10] = handed;
    if (nm > 0x7fffffffLL) atomicOr(W.flags, DF_RECCAP);
    if (P.check) {
        const FillOut &o = P.o;
        bool bad = nm > o.cap_mesh || nb + nf > o.cap_tri;
        if (o.vert_name && nv > o.cap_vert) bad = true;
        if (o.arc_f32 && na > o.cap_arc) bad = true;
        if (bad) atomicOr(W.flags, DF_CAPACITY);
    }
}

// offsets and status of the last count, where they were not written with it
__global__ void __launch_bounds__(kBlock) k_copy_offsets(int64_t N, int64_t S, Work W, OffsetsOut out)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x, n5 = kNodeScanCols * (N + 1);
    if (out.node_off && i < n5) out.node_off[i] = W.node_off[i];
    if (out.strut_off && i <= S) out.strut_off[i] = W.band_off[i];
    if (out.status && i < N) out.status[i] = (uint8_t)W.node_cnt[(int64_t)NC_STATUS * N + i];
}

// up to five runs of 32-bit words cleared in one launch
__global__ void __launch_bounds__(kBlock) k_clear(ClearRuns r)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
#pragma unroll
    for (int j = 0; j < ClearRuns::kMax; ++j)
        for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < r.n[j]; i += stride) r.p[j][i] = 0u;
}

// Node radius from per-strut end radii (Sec. 4.1: a strut is tangent to the
// nodal spheres of its ends, so the end radii at a node agree): the mean of
// the end radii of the node's struts in adjacency (strut id) order; a node
// whose end radii spread by more than rel_tol times that mean is counted.
__global__ void k_end_radii(int64_t N, const int64_t *row, const int2 *he, const int32_t *sa, const float *end_r,
                            float rel_tol, float *radius, int32_t *mismatch)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    const int64_t h0 = row[n], h1 = row[n + 1];
    float sum = 0.f, lo = 3.0e38f, hi = -3.0e38f;
    for (int64_t h = h0; h < h1; ++h) {
        const int64_t st = he[h].y;
        const float r = end_r[2 * st + (sa[st] == (int32_t)n ? 0 : 1)];
        sum += r;
        lo = fminf(lo, r);
        hi = fmaxf(hi, r);
    }
    // equal end radii give exactly that radius
    const float mean = h1 > h0 ? (hi == lo ? lo : sum / (float)(h1 - h0)) : 0.f;
    radius[n] = mean;
    if (h1 > h0 && hi - lo > rel_tol * fabsf(mean)) atomicAdd(mismatch, 1);
}

// d mean / d end radius = 1 / (struts at the node)
__global__ void k_end_grad(int64_t S, const int64_t *row, const int32_t *sa, const int32_t *sb, const float *grad_r,
                           float *grad_end)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * S) return;
    const int64_t st = i >> 1;
    const int32_t n = (i & 1) ? sb[st] : sa[st];
    const int64_t deg = row[n + 1] - row[n];
    grad_end[i] = deg > 0 ? grad_r[n] / (float)deg : 0.f;
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

hipError_t launch_end_radii(const Inputs &in, const Work &w, const float *end_r, float rel_tol, float *radius,
                            int32_t *mismatch, hipStream_t st)
{
    if (in.n_nodes > 0)
        k_end_radii<<<grid_for(in.n_nodes, kBlock), kBlock, 0, st>>>(in.n_nodes, w.row, w.he, in.sa, end_r, rel_tol,
                                                                      radius, mismatch);
    return hipGetLastError();
}

hipError_t launch_end_grad(const Inputs &in, const Work &w, const float *grad_r, float *grad_end, hipStream_t st)
{
    if (in.n_struts > 0)
        k_end_grad<<<grid_for(2 * in.n_struts, kBlock), kBlock, 0, st>>>(in.n_struts, w.row, in.sa, in.sb, grad_r,
                                                                         grad_end);
    return hipGetLastError();
}

// columns of tile sums, each with room for its total: five over the nodes
// (adjacency, then sizes), and the bands'
int64_t scan_tmp_needed(int64_t n_nodes, int64_t n_struts, bool sizes)
{
    static_assert(kRowCols <= kNodeScanCols, "the adjacency's columns fit the sizes'");
    const int64_t nodes = kNodeScanCols * (tiles_of(n_nodes) + 1), struts = tiles_of(n_struts) + 1;
    return sizes ? nodes + struts : (nodes > struts ? nodes : struts);
}

hipError_t launch_clear(const ClearRuns &r, hipStream_t st)
{
    int64_t most = 1;
    for (int j = 0; j < ClearRuns::kMax; ++j) most = r.n[j] > most ? r.n[j] : most;
    const int64_t blocks = (most + kBlock - 1) / kBlock;
    k_clear<<<(unsigned)(blocks < 1024 ? blocks : 1024), kBlock, 0, st>>>(r);
    return hipGetLastError();
}

hipError_t launch_sizes(const Inputs &in, const Work &w, const FillOut *o, const OffsetsOut &out, hipStream_t st)
{
    SizesParams P;
    P.in = in;
    P.w = w;
    P.o = o ? *o : FillOut{};
    P.check = o ? 1 : 0;
    P.out = out;
    P.nbn = tiles_of(in.n_nodes);
    P.nbs = tiles_of(in.n_struts);
    P.stride = P.nbn + 1;
    if (scan_tmp_needed(in.n_nodes, in.n_struts, true) > w.scan_tmp_len) return hipErrorInvalidValue;
    k_sizes_reduce<<<(unsigned)(P.nbn + P.nbs), kBlock, 0, st>>>(P);
    if (P.nbn > kFew) k_scan_tile_sums<<<kNodeScanCols, kBlock, 0, st>>>(w.scan_tmp, P.nbn, P.stride);
    if (P.nbs > kFew)
        k_scan_tile_sums<<<1, kBlock, 0, st>>>(w.scan_tmp + kNodeScanCols * P.stride, P.nbs, 0);
    k_sizes_tiles<<<dim3((unsigned)(P.nbn > P.nbs ? P.nbn : P.nbs), kNodeScanCols + 2), kBlock, 0, st>>>(P);
    return hipGetLastError();
}

hipError_t launch_copy_offsets(const Inputs &in, const Work &w, const OffsetsOut &out, hipStream_t st)
{
    if (!out.node_off && !out.strut_off && !out.status) return hipSuccess;
    const int64_t n5 = kNodeScanCols * (in.n_nodes + 1), n = n5 > in.n_struts + 1 ? n5 : in.n_struts + 1;
    k_copy_offsets<<<grid_for(n, kBlock), kBlock, 0, st>>>(in.n_nodes, in.n_struts, w, out);
    return hipGetLastError();
}

hipError_t launch_prepare(const Inputs &in, const Work &w, hipStream_t st)
{
    const int64_t N = in.n_nodes, S = in.n_struts, nb = tiles_of(N), stride = nb + 1;
    if (kRowCols * stride > w.scan_tmp_len) return hipErrorInvalidValue;
    // (at least one block: it clears the flags)
    k_pack<<<grid_for(N > 0 ? N : 1, kBlock), kBlock, 0, st>>>(in, w.node4, w.deg, w.flags);
    if (S > 0) k_degree<<<grid_for(S, kBlock), kBlock, 0, st>>>(in, w.deg, w.flags);
    if (nb > 1) k_rows_reduce<<<(unsigned)nb, kBlock, 0, st>>>(N, w.deg, w.scan_tmp, stride);
    if (nb > kFew) k_scan_tile_sums<<<kRowCols, kBlock, 0, st>>>(w.scan_tmp, nb, stride);
    k_rows_tiles<<<(unsigned)nb, kBlock, 0, st>>>(N, w.deg, w.scan_tmp, nb, stride, w.row, w.queue, w.cls_info);
    if (S > 0) k_scatter<<<grid_for(S, kBlock), kBlock, 0, st>>>(in, w.row, w.deg, w.he);
    if (N > 0) k_sort_rows<<<grid_for(N, kBlock), kBlock, 0, st>>>(N, w.row, w.he, w.strut_he, in.sa, in.sb);
    return hipGetLastError();
}

}  // namespace lm
