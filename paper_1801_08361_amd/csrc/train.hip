// Split training: a split structure learned from posed frames of one scene,
// whose leaves are then adapted online to others (Sec. 4.2.2, Table 2: a
// forest pre-trained on one scene and adapted to the rest).
//
// Every node of every tree, level by level from the root, takes from n_cand
// candidate splits (drawn like random splits, from the generator keyed by
// (seed, TRAIN) at counter (tree, node, candidate)) the one that leaves the
// training samples reaching it with the smallest summed squared deviation of
// their world points (integer mm) from their child's mean; ties go to the
// lower candidate. A sample is every stride-th pixel in u and v, from
// stride / 2, of every training frame with a valid depth, with its world
// point as adaptation stores it. The per-child sums (count, coordinate sums,
// sum of squared norms) are exact 64-bit integers, so any grouping of the
// samples gives the same sums; the cost of a child with n samples is
// S2 - |S|^2 / n in FP64, in that order, summed left then right.
//
// Layout: per tree, one 32-byte record per sample (packed word, divisor of its
// probe offsets, position, world point), kept grouped by the node that the
// sample has reached: a level ends by splitting every node's range stably
// into its children's. So no sample is ever counted or placed by a contended
// atomic, a node's samples are read in order, and nothing of a level passes
// through the host. Per level:
//   k_tr_units    the nodes' ranges cut into units of 256 or 512 samples
//   k_tr_eval     one wavefront per unit, one lane per candidate: the
//                 candidate's response for each sample, the right child's
//                 sums in registers (the left's are the unit's less those); a
//                 node of one unit picks its split there, larger nodes store
//                 partial sums
//   k_tr_pick     one workgroup per node of several units: the partials'
//                 sums (exact), the costs and the split
//   k_tr_route    the side of every sample of a unit, and the unit's count of
//                 left ones
//   k_tr_scan     prefix sums of those counts over all units
//   k_tr_move     every record to its child's range
//   k_tr_nodes    the children's ranges and the prefix sums of their units
#include <hip/hip_runtime.h>

#include <string.h>

#include <algorithm>
#include <vector>

#include "common.h"

namespace rl {

int frame_from(const Forest *f, const uint16_t *depth, const uint8_t *rgb, const reloc_intrinsics *K, Frame &fr);
bool pose_is_se3(const double T[16]);
int forest_empty_leaves(Forest *f, hipStream_t s);

namespace {

// How a level's nodes are cut into evaluation units: samples per unit and
// wavefronts that share one, by the samples a node has on average. The
// wavefronts of a unit take neighbouring samples, whose probes share cache
// lines, so the fewer units a CU holds the more of its probes its L1 serves:
// on 960 000 samples of 50 640 x 480 frames in 5 trees the root's level took
// 2.7 ms with a wavefront per unit, 0.98 with 8 and 0.95 with 16, the level
// of 117 samples a node 2.8, 2.15 and 2.10, and that of 58 2.8, 2.20 and 2.56
// (a unit's candidates are drawn by every wavefront); units of 1024 and 2048
// samples took 0.98 and 1.10 ms at the root.
struct UnitShape {
    int samples, waves;
};

constexpr int SMALL_UNIT = 256;   // the smallest, for bounds on their number

static UnitShape unit_shape(int32_t S, int level)
{
    const int32_t mean = S >> level;
    return mean >= 100 ? UnitShape{512, 16} : mean >= 16 ? UnitShape{512, 8} : UnitShape{SMALL_UNIT, 1};
}

constexpr int NSUMS = 5;        // per candidate and child: n, Sx, Sy, Sz, S2
constexpr int SCAN_ITEMS = 8, SCAN_BLOCK = 256 * SCAN_ITEMS;

struct TrainPose {
    float R[9], t[3];
};

// one sample as the levels read it
struct __align__(32) Rec {
    uint64_t own;        // packed word of its pixel
    uint32_t magic;      // pixel_den of its depth: the multiplier
    uint32_t uv;         // u | v << 13 | the divisor's shift << 26
    int32_t frame;
    int32_t x, y, z;     // world point (mm)
};
static_assert(sizeof(Rec) == 32, "one scalar load of eight words");

__device__ __forceinline__ int rec_u(const Rec &r) { return (int)(r.uv & 0x1FFFu); }
__device__ __forceinline__ int rec_v(const Rec &r) { return (int)((r.uv >> 13) & 0x1FFFu); }
__device__ __forceinline__ PixelDen rec_den(const Rec &r) { return PixelDen{r.magic, r.uv >> 26}; }

struct Unit {
    int32_t node;        // tree * n_level + node within the level
    int32_t start, len;  // range of the records
    int32_t slot;        // partial-sum slot, or -1: the unit is its node's only one
};

// a posed frame and where its planes begin (bytes)
struct TrainFrame {
    Frame fr;
    TrainPose pose;
    int64_t poff;
};

// A frame as its probes read it: a plane of 16-bit depths (65535 - z, 0 outside
// the valid range) and three of 8-bit colours (255 - r, g, b): 5 bytes a pixel,
// and 64 or 128 neighbours of a row in a cache line, where the traversal's
// 8-byte words would hold 16. Planes have a multiple of 8 pixels, so that the
// next frame's begin where its depths' 8-byte stores may.
__host__ __device__ __forceinline__ int plane_pixels(int P) { return (P + 7) & ~7; }
__host__ __device__ __forceinline__ int plane_bytes(int P) { return 5 * plane_pixels(P); }

struct TrainArgs {
    const TrainFrame *frames;     // [n_frames]
    const uint8_t *planes;
    int32_t n_frames;
    int32_t unit;                 // samples per unit at this level
    int32_t S;                    // samples
    int32_t T, L;
    int32_t level_first;          // heap index of the level's first node
    int32_t n_level;              // nodes in the level
    int32_t n_cand;
    int32_t stride;
    uint64_t seed;
    int32_t O, thr_d, thr_c;
    const Rec *rec;               // [T][S], grouped by node
    Rec *next;                    // [T][S], the next level's
    int2 *range;                  // [T][n_level] start, count
    int2 *next_range;             // [T][2 n_level]
    uint64_t *first;              // [T][n_level] prefix of (slots << 32 | units), less the block's
    uint64_t *first_sum;          // per SCAN_BLOCK nodes; the total follows
    Unit *units;
    int32_t *several;             // number of nodes of several units, then those nodes
    uint64_t *side;               // [units][unit / 64] samples that go right
    uint32_t *left;               // [units] samples that go left, then their prefix, less the block's
    uint64_t *left_sum;           // per SCAN_BLOCK units
    long long *partial;           // [slots][NSUMS][64] right child
    long long *total;             // [slots][NSUMS] both children
    uint64_t *nodes;              // the forest's split nodes [T][L - 1]
    DeepNode *deep;
};

// Uniform reads of what earlier kernels wrote go through the scalar cache:
// its address space says that nothing in this kernel writes there.
template <typename X>
__device__ __forceinline__ X scalar_read(const X *p)
{
    struct Words {
        uint32_t w[sizeof(X) / 4];
    } v;
#pragma unroll
    for (size_t i = 0; i < sizeof(X) / 4; ++i)
        v.w[i] = ((const __attribute__((address_space(4))) uint32_t *)(uintptr_t)p)[i];
    return __builtin_bit_cast(X, v);
}

// units of a node of n samples (an empty node has one, which picks its split)
// and the partial-sum slots they need
__device__ __forceinline__ uint64_t node_units(const TrainArgs &A, int n)
{
    const uint32_t u = n <= A.unit ? 1u : (uint32_t)((n + A.unit - 1) / A.unit);
    return ((uint64_t)(u > 1u ? u : 0u) << 32) | u;
}

// all frames' planes, blockIdx.y over the frames, 4 pixels a thread
__global__ void __launch_bounds__(256) k_tr_pack(TrainArgs A, uint8_t *__restrict__ planes)
{
    for (int fi = blockIdx.y; fi < A.n_frames; fi += gridDim.y) {
        const Frame fr = scalar_read(&A.frames[fi].fr);
        uint8_t *base = planes + scalar_read(&A.frames[fi].poff);
        const int P = fr.W * fr.H, n = plane_pixels(P);
        for (int p = 4 * (blockIdx.x * 256 + threadIdx.x); p < P; p += 4 * 256 * gridDim.x) {
            uint64_t z = 0;
            uint32_t c[3] = {0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t w = p + e < P ? pack_pixel(fr, p + e) : 0ull;
                z |= (w & 0xFFFFull) << (16 * e);
#pragma unroll
                for (int a = 0; a < 3; ++a) c[a] |= ((uint32_t)(w >> (16 + 16 * a)) & 0xFFu) << (8 * e);
            }
            *(uint64_t *)(base + 2 * p) = z;
#pragma unroll
            for (int a = 0; a < 3; ++a) *(uint32_t *)(base + (2 + a) * n + p) = c[a];
        }
    }
}

// one thread per point of the frames' sampling grids, blockIdx.y over the
// frames; a workgroup's samples take one place in the list, in raster order
__global__ void __launch_bounds__(256) k_tr_samples(TrainArgs A, Rec *__restrict__ rec, int32_t *__restrict__ count)
{
    __shared__ int wave_n[4], block_at;
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    for (int fi = blockIdx.y; fi < A.n_frames; fi += gridDim.y) {
        const Frame fr = scalar_read(&A.frames[fi].fr);
        const TrainPose pose = scalar_read(&A.frames[fi].pose);
        const int st = A.stride, gw = (fr.W - st / 2 + st - 1) / st, gh = (fr.H - st / 2 + st - 1) / st;
        for (int g0 = blockIdx.x * 256; g0 < gw * gh; g0 += gridDim.x * 256) {
            const int g = g0 + (int)threadIdx.x;
            const bool in = g < gw * gh;
            const int u = in ? st / 2 + (g % gw) * st : 0, v = in ? st / 2 + (g / gw) * st : 0;
            const uint32_t d = fr.depth[v * fr.W + u];
            const bool ok = in && valid_depth(fr, d);
            const uint64_t m = __ballot(ok);
            __syncthreads();   // the previous place has been read
            if (lane == 0) wave_n[wave] = __popcll(m);
            __syncthreads();
            if (threadIdx.x == 0) block_at = atomicAdd(count, wave_n[0] + wave_n[1] + wave_n[2] + wave_n[3]);
            __syncthreads();
            int at = block_at + __popcll(m & ((1ull << lane) - 1ull));
            for (int w = 0; w < wave; ++w) at += wave_n[w];
            if (ok) {
                float c[3];
                cam_point(fr, u, v, d, c);
                const float w0 = ((pose.R[0] * c[0] + pose.R[1] * c[1]) + pose.R[2] * c[2]) + pose.t[0];
                const float w1 = ((pose.R[3] * c[0] + pose.R[4] * c[1]) + pose.R[5] * c[2]) + pose.t[1];
                const float w2 = ((pose.R[6] * c[0] + pose.R[7] * c[1]) + pose.R[8] * c[2]) + pose.t[2];
                const PixelDen pd = pixel_den(fr, (int32_t)d);
                Rec r;
                r.own = pack_pixel(fr, v * fr.W + u);
                r.magic = pd.magic;
                r.uv = (uint32_t)u | ((uint32_t)v << 13) | (pd.shift << 26);
                r.frame = fi;
                r.x = (int32_t)rintf(w0 * 1000.0f);
                r.y = (int32_t)rintf(w1 * 1000.0f);
                r.z = (int32_t)rintf(w2 * 1000.0f);
                rec[at] = r;
            }
        }
    }
}

// the records into every tree's range, and the roots
__global__ void __launch_bounds__(256) k_tr_roots(TrainArgs A, const Rec *__restrict__ drawn, Rec *__restrict__ rec)
{
    const int t = blockIdx.y;
    if (blockIdx.x == 0 && threadIdx.x == 0) A.range[t] = make_int2(t * A.S, A.S);
    for (int i = blockIdx.x * 256 + threadIdx.x; i < A.S; i += gridDim.x * 256) rec[(int64_t)t * A.S + i] = drawn[i];
}

// exclusive scan over the workgroup of one value a thread; the total to *sum
__device__ __forceinline__ uint64_t block_scan(uint64_t v, uint64_t *sum)
{
    __shared__ uint64_t ws[4];
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    uint64_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    __syncthreads();
    if (lane == 63) ws[wave] = x;
    __syncthreads();
    uint64_t off = 0;
    for (int w = 0; w < wave; ++w) off += ws[w];
    *sum = ((ws[0] + ws[1]) + ws[2]) + ws[3];
    return off + x - v;
}

// exclusive scan of the n block sums in place; the total to sum[n]. One
// workgroup; the number of sums is that of *n_items items where it is given.
__global__ void __launch_bounds__(256) k_tr_sums(uint64_t *__restrict__ sum, int n, const uint64_t *__restrict__ n_items)
{
    if (n_items) n = ((int)(uint32_t)*n_items + SCAN_BLOCK - 1) / SCAN_BLOCK;
    uint64_t carry = 0;
    for (int b = 0; b < n; b += 256) {
        const int i = b + (int)threadIdx.x;
        const uint64_t v = i < n ? sum[i] : 0ull;
        uint64_t total;
        const uint64_t x = block_scan(v, &total);
        if (i < n) sum[i] = carry + x;
        carry += total;
    }
    if (threadIdx.x == 0) sum[n] = carry;
}

// number of units of the level (the total of the nodes' prefix sums)
__device__ __forceinline__ int level_units(const TrainArgs &A)
{
    const int nodes = A.T * A.n_level;
    return (int)(uint32_t)scalar_read(A.first_sum + (nodes + SCAN_BLOCK - 1) / SCAN_BLOCK);
}

__device__ __forceinline__ uint64_t node_first(const TrainArgs &A, int node)
{
    return A.first[node] + A.first_sum[node / SCAN_BLOCK];
}

// left ones among the samples of the units before unit u (u up to their count)
__device__ __forceinline__ uint32_t left_before(const TrainArgs &A, int u, int n_units)
{
    const int nb = (n_units + SCAN_BLOCK - 1) / SCAN_BLOCK;
    return u < n_units ? A.left[u] + (uint32_t)A.left_sum[u / SCAN_BLOCK] : (uint32_t)A.left_sum[nb];
}

// The level's nodes: their ranges (from their parents' split below the root)
// and the prefix sums of their units, SCAN_BLOCK nodes a workgroup.
__global__ void __launch_bounds__(256) k_tr_nodes(TrainArgs A)
{
    const int nodes = A.T * A.n_level;
    const int b0 = blockIdx.x * SCAN_BLOCK + (int)threadIdx.x * SCAN_ITEMS;
    uint64_t v[SCAN_ITEMS], s = 0;
#pragma unroll
    for (int e = 0; e < SCAN_ITEMS; ++e) {
        const int i = b0 + e;
        v[e] = s;
        if (i < nodes) s += node_units(A, A.range[i].y);
    }
    uint64_t total;
    const uint64_t off = block_scan(s, &total);
#pragma unroll
    for (int e = 0; e < SCAN_ITEMS; ++e)
        if (b0 + e < nodes) A.first[b0 + e] = off + v[e];
    if (threadIdx.x == 0) A.first_sum[blockIdx.x] = total;
    if (threadIdx.x == 0 && blockIdx.x == 0) A.several[0] = 0;
}

// a wavefront per node writes its units
__global__ void __launch_bounds__(256) k_tr_units(TrainArgs A)
{
    const int node = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (node >= A.T * A.n_level) return;
    const int2 r = A.range[node];
    const uint64_t f = node_first(A, node);
    const int n = (int)(uint32_t)node_units(A, r.y);
    for (int k = __lane_id(); k < n; k += 64) {
        const int at = k * A.unit;
        A.units[(uint32_t)f + k] = Unit{node, r.x + at, min(A.unit, r.y - at), n > 1 ? (int32_t)(f >> 32) + k : -1};
    }
    if (n > 1 && __lane_id() == 0) A.several[1 + atomicAdd(A.several, 1)] = node;
}

// the cost of one candidate's sums (as the oracle defines it)
__device__ __forceinline__ double split_cost(const long long l[NSUMS], const long long r[NSUMS])
{
    double c = 0.0;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const long long *q = side ? r : l;
        if (q[0] == 0) continue;
        const double sx = (double)q[1], sy = (double)q[2], sz = (double)q[3];
        c = c + ((double)q[4] - ((sx * sx + sy * sy) + sz * sz) / (double)q[0]);
    }
    return c;
}

// lane k's candidate, or the first of equal lowest costs over the lanes: the
// lane of the chosen candidate
__device__ __forceinline__ int wave_argmin(double c, int k)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const double co = __shfl_xor(c, o, 64);
        const int ko = __shfl_xor(k, o, 64);
        if (co < c || (co == c && ko < k)) {
            c = co;
            k = ko;
        }
    }
    return k;
}

__device__ __forceinline__ void write_split(const TrainArgs &A, int t, int j, uint64_t w)
{
    const int64_t at = (int64_t)t * (A.L - 1) + A.level_first + j;
    A.nodes[at] = w;
    A.deep[at] = deep_node(w);
}

__device__ __forceinline__ uint64_t candidate(const TrainArgs &A, int t, int j, int k)
{
    return split_from_draw(philox((uint64_t)t, (uint64_t)(A.level_first + j), (uint64_t)k, 0, A.seed, TAG_TRAIN), A.O,
                           A.thr_d, A.thr_c);
}

// lane k's candidate from the sums of both children and of the right one
__device__ __forceinline__ void pick_split(const TrainArgs &A, int t, int j, int k, const long long tot[NSUMS],
                                           const long long right[NSUMS], uint64_t w)
{
    long long l[NSUMS];
#pragma unroll
    for (int e = 0; e < NSUMS; ++e) l[e] = tot[e] - right[e];
    const double c = k < A.n_cand ? split_cost(l, right) : INFINITY;
    if (k == wave_argmin(c, k)) write_split(A, t, j, w);
}

// A split prepared for the planes of one frame: its offsets scaled by the
// focal lengths as div_mag2 takes them, its plane's first byte, log2 of its
// bytes a pixel and its bits.
struct PlaneNode {
    uint32_t ax, ay, sxy;
    uint32_t base, lg, bits, wout, sh;
};

__device__ __forceinline__ PlaneNode plane_node(uint64_t w, const Frame &fr)
{
    const ProbeNode n = probe_node(w, fr);
    const int kind = (int)(w & 3u);
    PlaneNode q;
    q.ax = n.ax;
    q.ay = n.ay;
    q.sxy = n.sxy;
    q.base = kind ? (uint32_t)((1 + kind) * plane_pixels(fr.W * fr.H)) : 0u;
    q.lg = kind ? 0u : 1u;
    q.bits = kind ? 8u : 16u;
    q.wout = kind ? 8u : 0u;
    q.sh = n.sh;
    return q;
}

// probe_response from a frame's planes: the clamped probe position, the word
// that holds its field, and the field's place in it
struct PlaneProbe {
    uint32_t at;       // byte of the field
    bool out;          // the position was clamped
};

__device__ __forceinline__ PlaneProbe plane_probe(int W, int H, const Rec &r, const PlaneNode &n)
{
    const PixelDen pd = rec_den(r);
    const uint32_t ox = div_mag2(n.ax, pd), oy = div_mag2(n.ay, pd);
    const i16x2 uv = __builtin_bit_cast(i16x2, (uint32_t)rec_u(r) | ((uint32_t)rec_v(r) << 16));
    const i16x2 q = __builtin_bit_cast(i16x2, ox | (oy << 16)) * __builtin_bit_cast(i16x2, n.sxy) + uv;
    const i16x2 zero = {0, 0};
    const i16x2 hi = __builtin_bit_cast(i16x2, (uint32_t)(W - 1) | ((uint32_t)(H - 1) << 16));
    const i16x2 c = __builtin_elementwise_min(__builtin_elementwise_max(q, zero), hi);
    const u16x2_t row = __builtin_bit_cast(u16x2_t, 1u | ((uint32_t)W << 16));
    PlaneProbe p;
    p.at = (__builtin_amdgcn_udot2(__builtin_bit_cast(u16x2_t, c), row, 0u, false) << n.lg) + n.base;
    p.out = __builtin_bit_cast(uint32_t, q) != __builtin_bit_cast(uint32_t, c);
    return p;
}

__device__ __forceinline__ int32_t plane_response(const PlaneProbe &p, uint32_t word, uint64_t own, const PlaneNode &n)
{
    const uint32_t probed = __builtin_amdgcn_ubfe(word, p.at << 3, p.out ? n.wout : n.bits);
    return (int32_t)((uint32_t)(own >> n.sh) & 0xFFFFu) - (int32_t)probed;
}

// One unit on kWaves wavefronts, lane k its node's candidate k. A sample is
// the same for all lanes, so its record comes by one scalar load and its
// totals are scalar sums; per lane there remain the probe (64 candidates
// gather 64 different lines) and the right child's sums. EVAL_BATCH samples'
// probes are in flight together; the wavefronts of a unit take neighbouring
// batches, whose probes share lines. kSame: all frames have one size and one
// pair of focal lengths, which then scale the candidates once a unit.
// The gathers bound this kernel: it serves 0.53 lanes a cycle and CU at the
// root, 0.23 at nodes of 58 samples, whose lines come from far more of the
// frames (four samples in flight instead of two took 1.18 ms at the root, one
// 0.98: more lines compete for the L1).
constexpr int EVAL_BATCH = 2;

template <bool kSame, int kWaves>
__global__ void __launch_bounds__(64 * kWaves) k_tr_eval(TrainArgs A)
{
    __shared__ long long part[kWaves > 1 ? kWaves : 1][NSUMS][64], part_tot[kWaves][NSUMS];
    const int n_units = level_units(A), k = __lane_id();
    const int wave = kWaves > 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    const Frame f0 = scalar_read(&A.frames[0].fr);
    for (int ui = (int)blockIdx.x; ui < n_units; ui += (int)gridDim.x) {
        const Unit U = scalar_read(A.units + ui);
        const int t = U.node / A.n_level, j = U.node % A.n_level;
        const uint64_t w = candidate(A, t, j, k < A.n_cand ? k : 0);
        PlaneNode node = plane_node(w, f0);
        int32_t kind, dx, dy, thr;
        unpack_node(w, kind, dx, dy, thr);
        long long tot[NSUMS] = {0, 0, 0, 0, 0}, right[NSUMS] = {0, 0, 0, 0, 0};
        int32_t nr = 0;
        const Rec *rec = A.rec + U.start;
        for (int o = EVAL_BATCH * wave; o < U.len; o += EVAL_BATCH * kWaves) {
            Rec r[EVAL_BATCH];
            PlaneProbe pr[EVAL_BATCH];
            uint32_t word[EVAL_BATCH];
#pragma unroll
            for (int b = 0; b < EVAL_BATCH; ++b) r[b] = scalar_read(rec + min(o + b, U.len - 1));
#pragma unroll
            for (int b = 0; b < EVAL_BATCH; ++b) {
                const int fi = r[b].frame;
                int W = f0.W, H = f0.H;
                const uint8_t *img = A.planes + (int64_t)fi * plane_bytes(W * H);
                if constexpr (!kSame) {
                    const Frame fr = scalar_read(&A.frames[fi].fr);
                    W = fr.W;
                    H = fr.H;
                    img = A.planes + scalar_read(&A.frames[fi].poff);
                    node.ax = (uint32_t)abs(dx * fr.Fx) << 1;
                    node.ay = (uint32_t)abs(dy * fr.Fy) << 1;
                    node.base = kind ? (uint32_t)((1 + kind) * plane_pixels(W * H)) : 0u;
                }
                const __amdgpu_buffer_rsrc_t rs =
                    __builtin_amdgcn_make_buffer_rsrc((void *)img, (short)0, plane_bytes(W * H), 0x00020000);
                pr[b] = plane_probe(W, H, r[b], node);
                word[b] = __builtin_bit_cast(uint32_t,
                                             __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(pr[b].at & ~3u), 0, 0));
            }
#pragma unroll
            for (int b = 0; b < EVAL_BATCH; ++b) {
                if (o + b >= U.len) break;
                const long long x = r[b].x, y = r[b].y, z = r[b].z;
                const long long q2 = x * x + y * y + z * z;
                tot[1] += x;
                tot[2] += y;
                tot[3] += z;
                tot[4] += q2;
                if (plane_response(pr[b], word[b], r[b].own, node) >= thr) {
                    nr += 1;
                    right[1] += x;
                    right[2] += y;
                    right[3] += z;
                    right[4] += q2;
                }
            }
        }
        right[0] = nr;
        if constexpr (kWaves > 1) {
            __syncthreads();   // the previous unit's sums have been read
#pragma unroll
            for (int e = 0; e < NSUMS; ++e) part[wave][e][k] = right[e];
            if (k < NSUMS) part_tot[wave][k] = k == 1 ? tot[1] : k == 2 ? tot[2] : k == 3 ? tot[3] : tot[4];
            __syncthreads();
            if (wave) continue;
            for (int o = 1; o < kWaves; ++o)
#pragma unroll
                for (int e = 0; e < NSUMS; ++e) {
                    right[e] += part[o][e][k];
                    tot[e] += part_tot[o][e];
                }
        }
        tot[0] = U.len;
        if (U.slot < 0) {
            pick_split(A, t, j, k, tot, right, w);
        } else {
#pragma unroll
            for (int e = 0; e < NSUMS; ++e) A.partial[((int64_t)U.slot * NSUMS + e) * 64 + k] = right[e];
            if (k < NSUMS)
                A.total[(int64_t)U.slot * NSUMS + k] =
                    k == 0 ? tot[0] : k == 1 ? tot[1] : k == 2 ? tot[2] : k == 3 ? tot[3] : tot[4];
        }
    }
}

// nodes of several units: a workgroup per node, its wavefronts stride the slots
constexpr int PICK_WAVES = 16;

__global__ void __launch_bounds__(64 * PICK_WAVES) k_tr_pick(TrainArgs A)
{
    __shared__ long long part[PICK_WAVES][NSUMS][64], part_tot[PICK_WAVES][NSUMS];
    const int wave = threadIdx.x >> 6, k = __lane_id();
    const int n_several = A.several[0];
    for (int i = (int)blockIdx.x; i < n_several; i += (int)gridDim.x) {
        const int node = A.several[1 + i];
        const int first = (int)(node_first(A, node) >> 32), slots = (A.range[node].y + A.unit - 1) / A.unit;
        long long right[NSUMS] = {0, 0, 0, 0, 0}, tot = 0;   // lane e < NSUMS holds total e
        for (int sl = first + wave; sl < first + slots; sl += PICK_WAVES) {
#pragma unroll
            for (int e = 0; e < NSUMS; ++e) right[e] += A.partial[((int64_t)sl * NSUMS + e) * 64 + k];
            if (k < NSUMS) tot += A.total[(int64_t)sl * NSUMS + k];
        }
        __syncthreads();   // the previous node's sums have been read
#pragma unroll
        for (int e = 0; e < NSUMS; ++e) part[wave][e][k] = right[e];
        if (k < NSUMS) part_tot[wave][k] = tot;
        __syncthreads();
        if (wave == 0) {
            long long all[NSUMS];
#pragma unroll
            for (int e = 0; e < NSUMS; ++e) {
                all[e] = part_tot[0][e];
                for (int o = 1; o < PICK_WAVES; ++o) {
                    right[e] += part[o][e][k];
                    all[e] += part_tot[o][e];
                }
            }
            const int t = node / A.n_level, j = node % A.n_level;
            pick_split(A, t, j, k, all, right, candidate(A, t, j, k < A.n_cand ? k : 0));
        }
    }
}

// a wavefront per unit, a lane per sample: which samples go right
__global__ void __launch_bounds__(64) k_tr_route(TrainArgs A)
{
    const int n_units = level_units(A), l = __lane_id();
    for (int ui = (int)blockIdx.x; ui < n_units; ui += (int)gridDim.x) {
        const Unit U = scalar_read(A.units + ui);
        const int t = U.node / A.n_level, j = U.node % A.n_level;
        const uint64_t w = scalar_read(A.nodes + (int64_t)t * (A.L - 1) + A.level_first + j);
        int32_t kind, dx, dy, thr;
        unpack_node(w, kind, dx, dy, thr);
        uint32_t left = 0;
        for (int c = 0; 64 * c < U.len; ++c) {
            const int o = 64 * c + l;
            bool go = false;
            if (o < U.len) {
                const Rec r = A.rec[U.start + o];
                const TrainFrame &F = A.frames[r.frame];
                const PlaneNode n = plane_node(w, F.fr);
                const PlaneProbe p = plane_probe(F.fr.W, F.fr.H, r, n);
                go = plane_response(p, *(const uint32_t *)(A.planes + F.poff + (p.at & ~3u)), r.own, n) >= thr;
            }
            const uint64_t m = __ballot(go), in = __ballot(o < U.len);
            if (l == 0) A.side[(int64_t)ui * (A.unit / 64) + c] = m;
            left += (uint32_t)__popcll(in & ~m);
        }
        if (l == 0) A.left[ui] = left;
    }
}

// the units' left counts become their prefix sums, less the block's
__global__ void __launch_bounds__(256) k_tr_scan(TrainArgs A)
{
    const int n_units = level_units(A);
    const int b0 = blockIdx.x * SCAN_BLOCK + (int)threadIdx.x * SCAN_ITEMS;
    if (blockIdx.x * SCAN_BLOCK >= n_units) return;
    uint32_t v[SCAN_ITEMS], s = 0;
#pragma unroll
    for (int e = 0; e < SCAN_ITEMS; ++e) {
        v[e] = s;
        if (b0 + e < n_units) s += A.left[b0 + e];
    }
    uint64_t total;
    const uint32_t off = (uint32_t)block_scan(s, &total);
#pragma unroll
    for (int e = 0; e < SCAN_ITEMS; ++e)
        if (b0 + e < n_units) A.left[b0 + e] = off + v[e];
    if (threadIdx.x == 0) A.left_sum[blockIdx.x] = total;
}

// every record to its child's range (stable), and the children's ranges
__global__ void __launch_bounds__(64) k_tr_move(TrainArgs A)
{
    const int n_units = level_units(A), l = __lane_id();
    for (int ui = (int)blockIdx.x; ui < n_units; ui += (int)gridDim.x) {
        const Unit U = A.units[ui];
        const int2 R = A.range[U.node];
        const int u0 = (int)(uint32_t)node_first(A, U.node), nu = (int)(uint32_t)node_units(A, R.y);
        const uint32_t l0 = left_before(A, u0, n_units);
        const int node_left = (int)(left_before(A, u0 + nu, n_units) - l0);
        int left = (int)(left_before(A, ui, n_units) - l0);
        int right = node_left + (U.start - R.x) - left;
        for (int c = 0; 64 * c < U.len; ++c) {
            const int o = 64 * c + l;
            const uint64_t m = A.side[(int64_t)ui * (A.unit / 64) + c];
            const int nr = __popcll(m & ((1ull << l) - 1ull));
            if (o < U.len) A.next[R.x + ((m >> l) & 1 ? right + nr : left + l - nr)] = A.rec[U.start + o];
            const int all = __popcll(m);
            right += all;
            left += min(64, U.len - 64 * c) - all;
        }
        if (ui == u0 && l == 0) {
            A.next_range[2 * U.node] = make_int2(R.x, node_left);
            A.next_range[2 * U.node + 1] = make_int2(R.x + node_left, R.y - node_left);
        }
    }
}

// device scratch of one training call, freed in stream order
struct Scratch {
    std::vector<void *> ptrs;
    hipStream_t s;
    explicit Scratch(hipStream_t st) : s(st) {}
    template <typename X>
    bool get(X **p, size_t count)
    {
        *p = nullptr;
        if (device_malloc_async((void **)p, std::max<size_t>(count, 1) * sizeof(X), s) != hipSuccess) return false;
        ptrs.push_back((void *)*p);
        return true;
    }
    ~Scratch()
    {
        for (void *p : ptrs) (void)hipFreeAsync(p, s);
        (void)hipStreamSynchronize(s);
    }
};

void (*eval_kernel(bool same, int waves))(TrainArgs)
{
    switch (waves) {
    case 16: return same ? k_tr_eval<true, 16> : k_tr_eval<false, 16>;
    case 8: return same ? k_tr_eval<true, 8> : k_tr_eval<false, 8>;
    default: return same ? k_tr_eval<true, 1> : k_tr_eval<false, 1>;
    }
}

unsigned blocks_of(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace
}  // namespace rl

using namespace rl;

extern "C" int reloc_forest_train(reloc_forest *f, const reloc_train_frame *frames, int32_t n_frames, int32_t stride,
                                  int32_t n_candidates, void *stream)
{
    if (!f || !frames || n_frames < 1 || stride < 1 || n_candidates < 1 || n_candidates > 64) return RELOC_E_ARG;
    if (f->dropped) return RELOC_E_STATE;
    hipStream_t s = (hipStream_t)stream;
    std::vector<TrainFrame> tf(n_frames);
    int64_t bytes_all = 0, S_cap = 0;
    int P_max = 0, G_max = 0;
    bool same = true;
    for (int k = 0; k < n_frames; ++k) {
        Frame &fr = tf[k].fr;
        int rc = frame_from(f, frames[k].depth_dev, frames[k].rgb_dev, &frames[k].K, fr);
        if (rc) return rc;
        if (!pose_is_se3(frames[k].pose_c2w)) return RELOC_E_ARG;
        for (int r = 0; r < 3; ++r) {
            for (int c = 0; c < 3; ++c) tf[k].pose.R[r * 3 + c] = (float)frames[k].pose_c2w[r * 4 + c];
            tf[k].pose.t[r] = (float)frames[k].pose_c2w[r * 4 + 3];
        }
        tf[k].poff = bytes_all;
        const int gw = std::max(0, (fr.W - stride / 2 + stride - 1) / stride),
                  gh = std::max(0, (fr.H - stride / 2 + stride - 1) / stride);
        bytes_all += plane_bytes(fr.W * fr.H);
        P_max = std::max(P_max, fr.W * fr.H);
        S_cap += (int64_t)gw * gh;
        G_max = std::max(G_max, gw * gh);
        same = same && fr.W == tf[0].fr.W && fr.H == tf[0].fr.H && fr.Fx == tf[0].fr.Fx && fr.Fy == tf[0].fr.Fy;
    }
    if (S_cap > (int64_t)INT32_MAX / std::max(f->T, 1)) return RELOC_E_RANGE;
    Scratch sc(s);
    TrainFrame *d_frames;
    uint8_t *planes;
    Rec *drawn;
    int32_t *d_count;
    if (!sc.get(&d_frames, n_frames) || !sc.get(&planes, bytes_all) || !sc.get(&drawn, S_cap) || !sc.get(&d_count, 1))
        return RELOC_E_NOMEM;
    TrainArgs A;
    memset(&A, 0, sizeof(A));
    A.frames = d_frames;
    A.planes = planes;
    A.n_frames = n_frames;
    A.T = f->T;
    A.L = f->L;
    A.n_cand = n_candidates;
    A.stride = stride;
    A.seed = f->p.seed;
    A.O = f->p.offset_pxmm;
    A.thr_d = f->p.thr_depth_mm;
    A.thr_c = f->p.thr_rgb;
    A.nodes = f->nodes;
    A.deep = f->deep;
    RL_HIP(hipMemcpyAsync(d_frames, tf.data(), sizeof(TrainFrame) * n_frames, hipMemcpyHostToDevice, s));
    RL_HIP(hipMemsetAsync(d_count, 0, sizeof(int32_t), s));
    const unsigned fy = (unsigned)std::min(n_frames, 32768);
    RL_LAUNCH("k_tr_pack", k_tr_pack, dim3(std::min(blocks_of(P_max, 1024), 1024u), fy), dim3(256), 0, s, A, planes);
    if (G_max > 0)
        RL_LAUNCH("k_tr_samples", k_tr_samples, dim3(std::min(blocks_of(G_max, 256), 1024u), fy), dim3(256), 0, s, A,
                  drawn, d_count);
    int32_t S = 0;
    RL_HIP(hipMemcpyAsync(&S, d_count, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    RL_HIP(hipStreamSynchronize(s));
    A.S = S;
    const int64_t TS = (int64_t)f->T * S;
    const int64_t max_nodes = (int64_t)f->T << (f->D - 1);
    const int64_t max_units = max_nodes + TS / SMALL_UNIT + 1;
    // partial slots: only nodes of several units use them, fewer than 2 n / unit each
    const int64_t max_several = TS / SMALL_UNIT, max_slots = 2 * max_several + 2;
    int64_t side_words = 0;
    for (int l = 0; l < f->D; ++l) {
        const int64_t unit = unit_shape(S, l).samples;
        side_words = std::max(side_words, (((int64_t)f->T << l) + TS / unit) * (unit / 64));
    }
    Rec *rec[2];
    int2 *range[2];
    if (!sc.get(&rec[0], TS) || !sc.get(&rec[1], TS) || !sc.get(&range[0], max_nodes) ||
        !sc.get(&range[1], max_nodes) || !sc.get(&A.first, max_nodes) ||
        !sc.get(&A.first_sum, blocks_of(max_nodes, SCAN_BLOCK) + 1) || !sc.get(&A.units, max_units) ||
        !sc.get(&A.several, max_several + 2) || !sc.get(&A.side, side_words) || !sc.get(&A.left, max_units) ||
        !sc.get(&A.left_sum, blocks_of(max_units, SCAN_BLOCK) + 1) || !sc.get(&A.partial, max_slots * NSUMS * 64) ||
        !sc.get(&A.total, max_slots * NSUMS))
        return RELOC_E_NOMEM;
    A.range = range[0];
    RL_LAUNCH("k_tr_roots", k_tr_roots, dim3(std::min(std::max(blocks_of(S, 256), 1u), 1024u), (unsigned)f->T), dim3(256),
              0, s, A, (const Rec *)drawn, rec[0]);
    for (int l = 0; l < f->D; ++l) {
        A.level_first = (1 << l) - 1;
        A.n_level = 1 << l;
        A.rec = rec[l & 1];
        A.next = rec[(l + 1) & 1];
        A.range = range[l & 1];
        A.next_range = range[(l + 1) & 1];
        const UnitShape shape = unit_shape(S, l);
        A.unit = shape.samples;
        const int64_t nodes = (int64_t)f->T * A.n_level, units = nodes + TS / A.unit;
        const unsigned nb = blocks_of(nodes, SCAN_BLOCK), grid = (unsigned)std::min<int64_t>(units, 65536);
        RL_LAUNCH("k_tr_nodes", k_tr_nodes, dim3(nb), dim3(256), 0, s, A);
        RL_LAUNCH("k_tr_sums", k_tr_sums, dim3(1), dim3(256), 0, s, A.first_sum, (int)nb, (const uint64_t *)nullptr);
        RL_LAUNCH("k_tr_units", k_tr_units, dim3(blocks_of(nodes, 4)), dim3(256), 0, s, A);
        RL_LAUNCH("k_tr_eval", eval_kernel(same, shape.waves), dim3(grid), dim3(64 * shape.waves), 0, s, A);
        RL_LAUNCH("k_tr_pick", k_tr_pick, dim3((unsigned)std::min<int64_t>(std::min(nodes, max_several + 1), 2048)),
                  dim3(64 * PICK_WAVES), 0, s, A);
        if (l + 1 == f->D) break;
        RL_LAUNCH("k_tr_route", k_tr_route, dim3(grid), dim3(64), 0, s, A);
        RL_LAUNCH("k_tr_scan", k_tr_scan, dim3(blocks_of(units, SCAN_BLOCK)), dim3(256), 0, s, A);
        RL_LAUNCH("k_tr_sums", k_tr_sums, dim3(1), dim3(256), 0, s, A.left_sum, 0, (const uint64_t *)(A.first_sum + nb));
        RL_LAUNCH("k_tr_move", k_tr_move, dim3(grid), dim3(64), 0, s, A);
    }
    RL_HIP(hipGetLastError());
    return forest_empty_leaves(f, s);
}
