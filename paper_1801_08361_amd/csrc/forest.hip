// Forest state on the GPU: split-node generation, features and traversal,
// online reservoir adaptation and leaf-mode extraction.
//
// Reservoir adaptation keeps the sequential definition (per tree, pixels
// offered to their leaves in raster order; Algorithm R with draws keyed by
// (tree, leaf, k)) while running every pixel in parallel: a pixel's k is its
// leaf's counter plus its stable rank among the frame's pixels in the same
// leaf, and because a slot depends only on k, each slot keeps the sample with
// the largest k that maps to it. Ranks come from an ordered count of each
// chunk of pixels plus a per-leaf prefix over chunks; "largest k wins" is an
// atomicMax on a per-slot stamp: the first pixel of a frame that reaches a slot
// writes it, and of those that came later the one whose stamp remains.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include "common.h"

namespace rl {

// ---------------------------------------------------------------------------
// device memory
// ---------------------------------------------------------------------------

// A destroyed forest's tables are kept for the next forest of the same sizes:
// giving 21 allocations to the driver and taking them back costs more than a
// small room's frames (0.8 of 2.3 ms for 9 frames in a 267 MB forest), and
// quick rebuilding brings the driver into a state where giving back and taking
// 267 MB costs 5 ms, and the 3.5 GB of a full-size forest 60 to 90 ms.
//
// A kept block belongs to nobody: whoever returns one has waited for the
// device, so that any stream or thread can take it, and its contents are as
// undefined as new memory's. At most KEEP_BYTES are kept per process, the
// oldest going first, and beyond KEEP_SMALL no more than a KEEP_SHARE-th of
// what the device has free besides (asked once a second at most, since asking
// takes 15 us: 6 frames into a 450 MB forest 783 us with a question each, 770
// so). All of a device's go back to it before any allocation of this library
// there fails; those not taken within KEEP_TIME at the next allocation or
// destruction (calls that other threads' graph captures exclude in any case);
// and everything by reloc_trim.
namespace {
using Clock = std::chrono::steady_clock;
constexpr size_t KEEP_SMALL = 1ull << 30;
constexpr size_t KEEP_SHARE = 8;
constexpr std::chrono::seconds KEEP_TIME{10}, ROOM_TIME{1};

struct Block {
    void *p;
    size_t bytes;
    int device;
    Clock::time_point since;
};

struct Kept {
    std::mutex mu;
    std::vector<Block> blocks;   // oldest first
    size_t bytes = 0;
    size_t room = 0;             // what may be kept, as of room_since, on room_device
    int room_device = -1;
    Clock::time_point room_since;
};

// never destroyed: objects may outlive static ones
Kept &kept()
{
    alignas(Kept) static unsigned char place[sizeof(Kept)];
    static Kept *k = new (place) Kept();
    return *k;
}

size_t block_bytes(size_t bytes) { return ((bytes < 1 ? 1 : bytes) + 4095) & ~(size_t)4095; }

// the oldest (or newest) kept block that `which` accepts, no longer kept; p is
// null if there is none
template <typename Which>
Block kept_take(Which which, bool newest = false)
{
    Kept &k = kept();
    std::lock_guard<std::mutex> g(k.mu);
    const size_t n = k.blocks.size();
    for (size_t j = 0; j < n; ++j) {
        const size_t i = newest ? n - 1 - j : j;
        if (which(k.blocks[i], k.bytes)) {
            const Block b = k.blocks[i];
            k.bytes -= b.bytes;
            k.blocks.erase(k.blocks.begin() + (std::ptrdiff_t)i);
            return b;
        }
    }
    return Block{};
}

// keeps the block; the bytes kept with it, 0 if it is not
size_t kept_put(const Block &b)
{
    Kept &k = kept();
    std::lock_guard<std::mutex> g(k.mu);
    try {
        size_t i = k.blocks.size();
        while (i > 0 && k.blocks[i - 1].since > b.since) --i;
        k.blocks.insert(k.blocks.begin() + (std::ptrdiff_t)i, b);
    } catch (...) {
        return 0;
    }
    k.bytes += b.bytes;
    return k.bytes;
}

// gives those blocks back to their devices; whether there was one
template <typename Which>
bool kept_release(Which which)
{
    bool any = false;
    for (;;) {
        const Block b = kept_take(which);
        if (!b.p) return any;
        if (hipFree(b.p) != hipSuccess) {   // (refused while another thread captures a graph)
            (void)hipGetLastError();
            (void)kept_put(b);
            return any;
        }
        any = true;
    }
}

// An allocation, tried once more without the device's kept blocks if it fails.
// The error is the caller's alone: it is not left for the next launch's check.
template <typename Alloc>
hipError_t alloc_or_release(Alloc alloc)
{
    hipError_t e = alloc();
    if (e == hipSuccess) return e;
    int device = 0;
    if (e == hipErrorOutOfMemory && hipGetDevice(&device) == hipSuccess &&
        kept_release([&](const Block &b, size_t) { return b.device == device; }))
        e = alloc();
    (void)hipGetLastError();
    return e;
}

void kept_expire()
{
    const Clock::time_point now = Clock::now();
    kept_release([&](const Block &b, size_t) { return now - b.since > KEEP_TIME; });
}

// bytes that may be kept on the current device at the moment, `more` of them wanted
size_t kept_room(size_t more, int device)
{
    Kept &k = kept();
    const Clock::time_point now = Clock::now();
    {
        std::lock_guard<std::mutex> g(k.mu);
        if (k.bytes + more <= KEEP_SMALL) return KEEP_SMALL;
        if (k.room_device == device && now - k.room_since < ROOM_TIME) return k.room;
    }
    size_t free = 0, total = 0;
    if (hipMemGetInfo(&free, &total) != hipSuccess) return KEEP_SMALL;
    const size_t room = std::max(KEEP_SMALL, std::min(KEEP_BYTES, free / KEEP_SHARE));
    std::lock_guard<std::mutex> g(k.mu);
    k.room = room;
    k.room_device = device;
    k.room_since = now;
    return room;
}
}  // namespace

hipError_t block_take(void **p, size_t bytes)
{
    const size_t n = block_bytes(bytes);
    int device = 0;
    const hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    // (the newest one: more of it is in the caches still)
    *p = kept_take([&](const Block &b, size_t) { return b.bytes == n && b.device == device; }, true).p;
    return *p ? hipSuccess : device_malloc(p, n);
}

void block_return(void *p, size_t bytes, int device, size_t room)
{
    const size_t n = block_bytes(bytes);
    int current = -1;
    size_t all = 0;
    if (n <= room && hipGetDevice(&current) == hipSuccess && current == device)
        all = kept_put(Block{p, n, device, Clock::now()});
    if (!all)
        (void)hipFree(p);
    else if (all > room)
        kept_release([&](const Block &, size_t bytes_kept) { return bytes_kept > room; });
}

hipError_t device_malloc(void **p, size_t bytes)
{
    kept_expire();
    return alloc_or_release([&] { return hipMalloc(p, bytes); });
}

hipError_t device_malloc_async(void **p, size_t bytes, hipStream_t s)
{
    return alloc_or_release([&] { return hipMallocAsync(p, bytes, s); });
}

// ---------------------------------------------------------------------------
// parameters
// ---------------------------------------------------------------------------

static void params_default(reloc_params *p)
{
    memset(p, 0, sizeof(*p));
    p->n_trees = 5; p->depth = 10; p->reservoir_size = 256; p->max_modes = 10;
    p->seed = 180108361ull;
    p->depth_min_mm = 500; p->depth_max_mm = 5000;
    p->offset_pxmm = 130000; p->f_ref_px16 = 277 * 16;
    p->thr_depth_mm = 100; p->thr_rgb = 10;
    p->dens_radius_mm = 50; p->link_radius_mm = 100; p->min_cluster = 0; p->cov_reg_mm2 = 100;
    p->n_hypotheses = 256; p->batch_pixels = 64; p->max_tries = 64; p->refine = 1; p->rgb_tol = 15;
    p->rigid_ratio2 = 1.21f; p->min_pair2_m2 = 0.01f; p->min_area2_m4 = 1e-4f;
    p->resid_m = 0.05f; p->inlier_m = 0.1f;
}

static int params_check(const reloc_params *p)
{
    if (p->n_trees < 1 || p->n_trees > 16 || p->depth < 1 || p->depth > 16) return RELOC_E_ARG;
    if (p->reservoir_size < 1 || p->reservoir_size > MAX_R || p->max_modes < 1 || p->max_modes > MAX_M ||
        p->n_trees * p->max_modes > MAX_TM)
        return RELOC_E_ARG;
    if (p->n_hypotheses < 1 || p->n_hypotheses > MAX_HYP || p->batch_pixels < 1 || p->batch_pixels > MAX_B)
        return RELOC_E_ARG;
    if (p->max_tries < 1 || p->max_tries > 1024 || p->rgb_tol < 0 || p->depth_min_mm < 1 || p->depth_max_mm > 65534 ||
        p->depth_min_mm > p->depth_max_mm || p->f_ref_px16 < 1)
        return RELOC_E_ARG;
    if (p->offset_pxmm < 0 || p->thr_depth_mm < 0 || p->thr_rgb < 0 || p->dens_radius_mm < 0 ||
        p->link_radius_mm < 0 || p->dens_radius_mm > 20000 || p->link_radius_mm > 20000 || p->cov_reg_mm2 < 1)
        return RELOC_E_ARG;
    if (p->offset_pxmm > NODE_OFF_MAX || p->thr_depth_mm > NODE_THR_MAX || p->thr_rgb > NODE_THR_MAX)
        return RELOC_E_RANGE;
    // depth denominators d * F_ref must fit 32 bits
    if ((int64_t)p->depth_max_mm * p->f_ref_px16 > 2147483647LL) return RELOC_E_RANGE;
    return RELOC_OK;
}

static int32_t focal16(float f) { return (int32_t)floor((double)f * 16.0 + 0.5); }

// intrinsics valid, width and height at most 8191, the focal lengths F in
// 1/16 px below 2^24, and |offset| * F fits 32 bits (so features stay exact)
static int frame_of(const Forest *f, const uint16_t *depth, const uint8_t *rgb, const reloc_intrinsics *K,
                    Frame &fr)
{
    if (!depth || !rgb || !K) return RELOC_E_ARG;
    if (K->width < 1 || K->height < 1 || K->width > 8191 || K->height > 8191) return RELOC_E_ARG;
    if (!(K->fx > 0.0f) || !(K->fy > 0.0f) || !isfinite(K->cx) || !isfinite(K->cy) || !isfinite(K->fx) ||
        !isfinite(K->fy))
        return RELOC_E_ARG;
    fr.depth = (decltype(fr.depth))depth; fr.rgb = (decltype(fr.rgb))rgb; fr.W = K->width; fr.H = K->height;
    fr.fx = K->fx; fr.fy = K->fy; fr.cx = K->cx; fr.cy = K->cy;
    if (!(K->fx < 1048576.0f) || !(K->fy < 1048576.0f)) return RELOC_E_ARG;
    int64_t Fx = focal16(K->fx), Fy = focal16(K->fy);
    if ((int64_t)f->p.offset_pxmm * Fx > 2147483647LL || (int64_t)f->p.offset_pxmm * Fy > 2147483647LL)
        return RELOC_E_ARG;
    // and every probe offset, at most |offset| * F / (d_min * F_ref) pixels,
    // stays below 2^14
    const int64_t den14 = ((int64_t)f->p.depth_min_mm * f->p.f_ref_px16) << 14;
    if ((int64_t)f->p.offset_pxmm * Fx >= den14 || (int64_t)f->p.offset_pxmm * Fy >= den14) return RELOC_E_ARG;
    if (Fx >= (1 << 24) || Fy >= (1 << 24)) return RELOC_E_ARG;
    fr.Fx = (int32_t)Fx; fr.Fy = (int32_t)Fy;
    fr.dmin = f->p.depth_min_mm; fr.dmax = f->p.depth_max_mm; fr.Fref = f->p.f_ref_px16;
    return RELOC_OK;
}

static bool is_se3(const double T[16])
{
    if (T[12] != 0.0 || T[13] != 0.0 || T[14] != 0.0 || T[15] != 1.0) return false;
    for (int k = 0; k < 16; ++k)
        if (!isfinite(T[k])) return false;
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            double s = T[0 * 4 + a] * T[0 * 4 + b] + T[1 * 4 + a] * T[1 * 4 + b] + T[2 * 4 + a] * T[2 * 4 + b];
            if (fabs(s - (a == b ? 1.0 : 0.0)) > 1e-6) return false;
        }
    double d = T[0] * (T[5] * T[10] - T[6] * T[9]) - T[1] * (T[4] * T[10] - T[6] * T[8]) +
               T[2] * (T[4] * T[9] - T[5] * T[8]);
    return d > 0.0;
}

template <typename T>
static int dalloc(Forest *f, T **ptr, size_t count, hipStream_t s)
{
    size_t bytes = count * sizeof(T);
    if (bytes == 0) bytes = sizeof(T);
    // (no block while the stream records a graph, kept or new: hipMalloc refuses there)
    hipStreamCaptureStatus recording = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &recording) != hipSuccess) {   // (the null stream beside one that records)
        (void)hipGetLastError();
        recording = hipStreamCaptureStatusNone;
    }
    if (recording != hipStreamCaptureStatusNone || block_take((void **)ptr, bytes) != hipSuccess) {
        *ptr = nullptr;
        return RELOC_E_NOMEM;
    }
    f->bytes += bytes;
    return RELOC_OK;
}

// room: kept for the next forest as block_return keeps it (the device is idle)
template <typename T>
static void dfree(Forest *f, T **ptr, size_t count, size_t room = 0)
{
    if (*ptr) {
        const size_t bytes = std::max<size_t>(count * sizeof(T), sizeof(T));
        if (room)
            block_return(*ptr, bytes, f->device, room);
        else
            (void)hipFree(*ptr);
        f->bytes -= bytes;
        *ptr = nullptr;
    }
}

// ---------------------------------------------------------------------------
// kernels: node generation
// ---------------------------------------------------------------------------

__global__ void k_gen_nodes(uint64_t *nodes, DeepNode *deep, int T, int L, uint64_t seed, int32_t O, int32_t thr_d,
                            int32_t thr_c)
{
    int64_t n_split = (int64_t)T * (L - 1);
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_split + 8) return;
    uint64_t t, node;
    if (i < n_split) {
        t = (uint64_t)(i / (L - 1));
        node = (uint64_t)(i % (L - 1));
    } else {
        t = (uint64_t)T;
        node = (uint64_t)(i - n_split);
    }
    nodes[i] = split_from_draw(philox(t, node, 0, 0, seed, TAG_FOREST), O, thr_d, thr_c);
    if (i < n_split) deep[i] = deep_node(nodes[i]);
}

// ---------------------------------------------------------------------------
// kernels: features and traversal
// ---------------------------------------------------------------------------

// one thread per (pixel, tree): blockIdx.y is the tree, so the trees' node
// chains run side by side instead of one after another
__global__ void __launch_bounds__(256) k_pack(Frame fr, uint64_t *__restrict__ packed)
{
    const int p = 4 * (int)(blockIdx.x * blockDim.x + threadIdx.x), P = fr.W * fr.H;
    uint64_t w[4];
    if (p < P) pack_pixels4(fr, (uint64_t RL_GLOBAL *)packed, P, p, w);
}

// block (x) of 4 x 256 pixels and tree (y): each thread walks 4 pixels of
// the tree together (tid, tid + 256, ...)
constexpr int LEAF_PIX = 4;

__global__ void __launch_bounds__(256) k_leaves(const uint64_t *__restrict__ nodes, const DeepNode *__restrict__ deep,
                                                int T, int L, Frame fr, const uint64_t *__restrict__ packed,
                                                int32_t *__restrict__ leaves)
{
    __shared__ ProbeNode top[top_nodes(LEAF_PIX)];
    const int P = fr.W * fr.H;
    const int base = blockIdx.x * (LEAF_PIX * 256) + threadIdx.x;
    const int t = blockIdx.y;
    const uint64_t *tree = nodes + (int64_t)t * (L - 1);
    const int ntop = L - 1 < top_nodes(LEAF_PIX) ? L - 1 : top_nodes(LEAF_PIX);
    stage_top(top, tree, ntop, fr, (int)threadIdx.x, (int)blockDim.x);
    __syncthreads();
    if (base >= P || t >= T) return;
    int p[LEAF_PIX];
    uint64_t own[LEAF_PIX];
    bool ok[LEAF_PIX];
#pragma unroll
    for (int k = 0; k < LEAF_PIX; ++k) {
        const int q = base + k * 256;
        p[k] = q < P ? q : P - 1;
        own[k] = packed[p[k]];
        ok[k] = q < P && packed_valid(own[k]);
    }
    int32_t leaf[LEAF_PIX];
    traverse_packed_k<LEAF_PIX>(top, ntop, deep + (int64_t)t * (L - 1), L, fr, packed, p, own, ok, leaf);
#pragma unroll
    for (int k = 0; k < LEAF_PIX; ++k)
        if (base + k * 256 < P) leaves[(int64_t)t * P + base + k * 256] = leaf[k];
}

__global__ void k_features8(const uint64_t *__restrict__ extra, Frame fr, int32_t *__restrict__ feat)
{
    int P = fr.W * fr.H;
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    int u = p % fr.W, v = p / fr.W;
    uint32_t d = fr.depth[p];
    bool ok = valid_depth(fr, d);
    if (!ok) {
        for (int j = 0; j < 8; ++j) feat[(int64_t)p * 8 + j] = 0;
        return;
    }
    const PixelDen pd = pixel_den(fr, (int32_t)d);
    for (int j = 0; j < 8; ++j) {
        int32_t thr;
        feat[(int64_t)p * 8 + j] = node_response_d(fr, extra[j], u, v, (int32_t)d, pd, thr);
    }
}

// ---------------------------------------------------------------------------
// kernels: reservoir adaptation
// ---------------------------------------------------------------------------

// Per (chunk, tree): the stable rank of each valid pixel among the chunk's
// pixels in the same leaf, and the chunk's per-leaf counts into the dense
// [T][C][L] table (kept zero elsewhere). A wavefront finds the equal leaves of
// 64 consecutive pixels with one ballot per bit of the leaf index; then one
// wavefront takes the chunk's 16 E such rows in order through a table of
// counts in LDS (two 16-bit counts a word), each leaf once per row with all
// its pixels, so that what it finds there is the leaf's count in the rows
// before. A wavefront's LDS operations run in issue order, so the rows need no
// wait between them. (A bitonic sort of the chunk's keys took 33 us for a 640
// x 480 frame in 5 trees of depth 15 and 24 us for 320 x 240 in depth 10; this
// takes 13.6 and 4.5.)
constexpr int RANK_THREADS = 1024, RANK_BATCH = 16;

static inline size_t rank_smem(int L) { return (size_t)(L / 2 + 64) * 4; }

// Pixels of a chunk over RANK_THREADS: as many as leave about two chunks for
// three CUs (160 over all trees), 2 to 8. Larger chunks make the table of
// counts smaller, which the prefix reads whole (640 x 480: ranks and prefix take
// 13.6 + 11.2 us with 8, 14.6 + 13.3 with 4, 14 + 33 with 2); smaller ones keep
// small frames' chunks on all CUs (320 x 240: 4.5 us with 2, 6.9 with 4). The
// deepest tree's table of counts leaves no room for 8.
static inline int chunk_pixels(int64_t P, int T, int L)
{
    int e = L > 32768 ? 4 : 8;
    while (e > 2 && T * P < (int64_t)160 * RANK_THREADS * e) e >>= 1;
    return RANK_THREADS * e;
}

template <int E>
__global__ void __launch_bounds__(RANK_THREADS) k_chunk_rank(const int32_t *__restrict__ leaves, int P, int L, int D,
                                                             int C, uint16_t *__restrict__ rank,
                                                             uint16_t *__restrict__ cnt)
{
    constexpr int CHUNK = RANK_THREADS * E, ROWS = CHUNK / 64;
    extern __shared__ uint32_t leaf_cnt[];   // [L / 2], then a word a lane
    __shared__ uint32_t row[CHUNK];          // leaf | pixels << 16 of a row's leaders, then the count before
    const int c = blockIdx.x, t = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t base = (int64_t)t * P + (int64_t)c * CHUNK;
    const int left = P - c * CHUNK;
    int32_t leaf[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = 64 * (E * wave + e) + lane;
        leaf[e] = i < left ? leaves[base + i] : -1;
    }
    for (int i = tid; i < L / 2 + 64; i += RANK_THREADS) leaf_cnt[i] = 0u;
    uint32_t same[E][2];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const uint64_t valid = __ballot(leaf[e] >= 0);
        same[e][0] = (uint32_t)valid;
        same[e][1] = (uint32_t)(valid >> 32);
    }
    // four bits a step; those past the index's are zero in every valid lane
    for (int b0 = 0; b0 < D; b0 += 4)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t bit = (uint32_t)__builtin_amdgcn_sbfe(leaf[e], b0 + b, 1);   // all ones or zero
                const uint64_t with = __ballot(bit != 0u);
                same[e][0] &= ~((uint32_t)with ^ bit);
                same[e][1] &= ~((uint32_t)(with >> 32) ^ bit);
            }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const uint32_t lo = same[e][0], hi = same[e][1];
        const int first = lo ? __builtin_ctz(lo) : 32 + (hi ? __builtin_ctz(hi) : 0);
        row[64 * (E * wave + e) + lane] =
            leaf[e] >= 0 && first == lane ? (uint32_t)leaf[e] | ((uint32_t)(__popc(lo) + __popc(hi)) << 16) : 0u;
    }
    __syncthreads();
    if (wave == 0) {
        // lanes without a leader add nothing to a word of their own, so that no
        // row branches and a batch's additions are all in flight together
        for (int r0 = 0; r0 < ROWS; r0 += RANK_BATCH) {
            uint32_t v[RANK_BATCH], old[RANK_BATCH];
#pragma unroll
            for (int r = 0; r < RANK_BATCH; ++r) v[r] = row[64 * (r0 + r) + lane];
#pragma unroll
            for (int r = 0; r < RANK_BATCH; ++r)
                old[r] = atomicAdd(&leaf_cnt[v[r] ? (int)((v[r] & 0xFFFFu) >> 1) : L / 2 + lane],
                                   (v[r] >> 16) << (16u * (v[r] & 1u)));
#pragma unroll
            for (int r = 0; r < RANK_BATCH; ++r)
                row[64 * (r0 + r) + lane] = (old[r] >> (16u * (v[r] & 1u))) & 0xFFFFu;
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (leaf[e] < 0) continue;
        const int r = 64 * (E * wave + e);
        const uint64_t m = ((uint64_t)same[e][1] << 32) | same[e][0];
        const uint32_t k = row[r + __builtin_ctzll(m)] + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        rank[base + r + lane] = (uint16_t)k;
        const uint32_t all = (leaf_cnt[leaf[e] >> 1] >> (16 * (leaf[e] & 1))) & 0xFFFFu;
        if (k + 1u == all) cnt[((int64_t)t * C + c) * L + leaf[e]] = (uint16_t)all;
    }
}

// Per (tree, leaf): prefix of chunk counts in chunk order, reset of the
// table, counter update, and marking of the leaf for mode extraction (its flag;
// a list of flagged leaves kept here cost a same-address atomic per workgroup,
// 20 us a frame). A thread
// has two neighbouring leaves; the four wavefronts of a workgroup split the
// chunks of the same 128 leaves, add up their shares in LDS and then each
// writes its own (kept in registers up to SCAN_KEEP chunks, read again
// beyond).
constexpr int SCAN_KEEP = 24;

__global__ void __launch_bounds__(256) k_leaf_scan(int T, int L, int C, uint16_t *__restrict__ cnt,
                                                   uint32_t *__restrict__ pref, uint32_t *__restrict__ counter,
                                                   uint32_t *__restrict__ base, uint32_t *__restrict__ dirty,
                                                   unsigned long long *__restrict__ total)
{
    __shared__ uint2 share[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = 2 * ((int64_t)blockIdx.x * 64 + lane);
    const bool in = i < (int64_t)T * L;
    const int t = in ? (int)(i / L) : 0, leaf = in ? (int)(i % L) : 0;
    const int c0 = C * wave / 4, nc = C * (wave + 1) / 4 - c0;
    uint32_t *tab = (uint32_t *)(cnt + ((int64_t)t * C + c0) * L + leaf);   // row stride L / 2 words
    const int64_t step = L / 2;
    uint32_t v[SCAN_KEEP];
    uint2 sum = make_uint2(0u, 0u);
    if (in) {
        if (nc <= SCAN_KEEP) {
#pragma unroll
            for (int q = 0; q < SCAN_KEEP; ++q) v[q] = q < nc ? tab[q * step] : 0u;
#pragma unroll
            for (int q = 0; q < SCAN_KEEP; ++q) {
                sum.x += v[q] & 0xFFFFu;
                sum.y += v[q] >> 16;
            }
        } else {
            for (int q = 0; q < nc; ++q) {
                const uint32_t w = tab[q * step];
                sum.x += w & 0xFFFFu;
                sum.y += w >> 16;
            }
        }
    }
    share[wave][lane] = sum;
    __syncthreads();
    uint2 run = make_uint2(0u, 0u), all = make_uint2(0u, 0u);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w == wave) run = all;
        all.x += share[w][lane].x;
        all.y += share[w][lane].y;
    }
    uint2 *out = (uint2 *)(pref + ((int64_t)t * C + c0) * L + leaf);
    auto put = [&](int q, uint32_t w) {
        if (w) {
            out[q * step] = run;
            tab[q * step] = 0u;
            run.x += w & 0xFFFFu;
            run.y += w >> 16;
        }
    };
    if (in) {
        if (nc <= SCAN_KEEP) {
#pragma unroll
            for (int q = 0; q < SCAN_KEEP; ++q) put(q, v[q]);
        } else {
            for (int q = 0; q < nc; ++q) put(q, tab[q * step]);
        }
    }
    if (wave) return;
    unsigned long long first_tree = in && t == 0 ? (unsigned long long)all.x + all.y : 0ull;
    for (int o = 32; o >= 1; o >>= 1) first_tree += __shfl_xor(first_tree, o, 64);
    if (lane == 0 && first_tree) atomicAdd(total, first_tree);
    if (!in) return;
    const uint2 k0 = *(const uint2 *)(counter + i);
    *(uint2 *)(base + i) = k0;
    if (all.x | all.y) *(uint2 *)(counter + i) = make_uint2(k0.x + all.x, k0.y + all.y);
    if (all.x) dirty[i] = 1u;
    if (all.y) dirty[i + 1] = 1u;
}

struct Pose32 {
    float R[9], t[3];
};

// The reservoir entry of pixel p: its world point (integer mm, FP32 transform
// then round-half-even) and colour.
__device__ __forceinline__ Entry frame_entry(const Frame &fr, const Pose32 &pose, int p)
{
    const int u = p % fr.W, v = p / fr.W;
    float c[3];
    cam_point(fr, u, v, fr.depth[p], c);
    Entry e;
    float w0 = ((pose.R[0] * c[0] + pose.R[1] * c[1]) + pose.R[2] * c[2]) + pose.t[0];
    float w1 = ((pose.R[3] * c[0] + pose.R[4] * c[1]) + pose.R[5] * c[2]) + pose.t[1];
    float w2 = ((pose.R[6] * c[0] + pose.R[7] * c[1]) + pose.R[8] * c[2]) + pose.t[2];
    e.x = (int32_t)rintf(w0 * 1000.0f);
    e.y = (int32_t)rintf(w1 * 1000.0f);
    e.z = (int32_t)rintf(w2 * 1000.0f);
    e.rgb = (uint32_t)fr.rgb[p * 3] | ((uint32_t)fr.rgb[p * 3 + 1] << 8) | ((uint32_t)fr.rgb[p * 3 + 2] << 16);
    return e;
}

// a pixel that met a slot already taken by another pixel of the frame
struct Late {
    uint32_t cell;    // slot over all leaves
    uint32_t stamp;   // k + 1
    int32_t p;
};

// Per (pixel, tree): k and the slot. The slot's stamp takes the largest k + 1
// that maps to it. A stamp of an earlier frame is at most the leaf's counter
// at the frame's start, so the stamp found there tells whether another pixel
// of this frame was first: the first one writes its entry at once, a later one
// of larger k goes to its workgroup's list for k_late (a later one of smaller k
// has lost). (Slots, then a second pass that compared every pixel's k with its
// slot's stamp and wrote the winners: 22.7 + 16.9 us for a 640 x 480 frame
// in 5 trees; this and k_late: 26 + 5, mostly the
// chain of loads and the atomic's return. With one list for the frame its
// counter's atomics alone made it 58.)
constexpr int RES_THREADS = 256;

__global__ void __launch_bounds__(RES_THREADS) k_reservoir(const int32_t *__restrict__ leaves,
                                                           const uint16_t *__restrict__ rank,
                                                           const uint32_t *__restrict__ pref,
                                                           const uint32_t *__restrict__ base, int L, int R, int C,
                                                           int chunk, uint64_t seed, Frame fr, Pose32 pose,
                                                           uint32_t *__restrict__ stamp, Entry *__restrict__ res,
                                                           Late *__restrict__ late, uint32_t *__restrict__ n_late)
{
    __shared__ uint32_t wave_n[RES_THREADS / 64];
    const int P = fr.W * fr.H, p = blockIdx.x * RES_THREADS + threadIdx.x, t = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t ti = (int64_t)t * P + p;
    const int32_t leaf = p < P ? leaves[ti] : -1;
    bool again = false;
    Late l = {0u, 0u, p};
    if (leaf >= 0) {
        const int64_t li = (int64_t)t * L + leaf;
        const uint32_t k0 = base[li];
        const uint32_t k = k0 + pref[((int64_t)t * C + p / chunk) * L + leaf] + rank[ti];
        int32_t s = -1;
        if (k < (uint32_t)R) {
            s = (int32_t)k;
        } else {
            const U4 u = philox((uint64_t)t, (uint64_t)leaf, (uint64_t)k, 0, seed, TAG_RESERVOIR);
            const uint64_t j = uniform_int(u.x[0], (uint64_t)k + 1);
            if (j < (uint64_t)R) s = (int32_t)j;
        }
        if (s >= 0) {
            l.cell = (uint32_t)(li * R + s);
            l.stamp = k + 1u;
            const uint32_t was = atomicMax(&stamp[l.cell], l.stamp);
            if (was <= k0) res[l.cell] = frame_entry(fr, pose, p);
            else again = was < l.stamp;
        }
    }
    const uint64_t m = __ballot(again);
    if (lane == 0) wave_n[wave] = (uint32_t)__popcll(m);
    __syncthreads();
    const int64_t list = (int64_t)t * gridDim.x + blockIdx.x;
    uint32_t at = 0u, n = 0u;
#pragma unroll
    for (int w = 0; w < RES_THREADS / 64; ++w) {
        if (w < wave) at += wave_n[w];
        n += wave_n[w];
    }
    if (again) late[list * RES_THREADS + at + __popcll(m & ((1ull << lane) - 1ull))] = l;
    if (threadIdx.x == 0) n_late[list] = n;
}

// the listed pixels whose stamp has remained write over the slot's first
// entry; a wavefront per list
__global__ void __launch_bounds__(256) k_late(const Late *__restrict__ late, const uint32_t *__restrict__ n_late,
                                              int lists, const uint32_t *__restrict__ stamp, Frame fr, Pose32 pose,
                                              Entry *__restrict__ res)
{
    const int list = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (list >= lists) return;
    const uint32_t n = n_late[list];
    for (uint32_t i = threadIdx.x & 63; i < n; i += 64) {
        const Late l = late[(int64_t)list * RES_THREADS + i];
        if (stamp[l.cell] == l.stamp) res[l.cell] = frame_entry(fr, pose, l.p);
    }
}

// ---------------------------------------------------------------------------
// kernels: leaf modes (integer quick-shift, then Gaussian statistics)
// ---------------------------------------------------------------------------

constexpr int MODE_THREADS = 256;

// Leaves whose points lie within NEAR_EXTENT mm per axis and radii of at most
// NEAR_RADIUS mm take the tiled search: coordinates relative to the leaf's
// minimum then fit 16 bits together with the padding points at NEAR_PAD
// (farther than any radius from every point), squared distances 32 bits, and
// a squared distance up to the link radius's square (below 2^22) packs above a
// 10-bit point index. Rooms and radii of 5-10 cm are far inside; anything else
// takes the plain search over all pairs.
constexpr int NEAR_EXTENT = 28000, NEAR_RADIUS = 2000, NEAR_PAD = -4000;
constexpr uint32_t D2_CAP = (1u << 22) - 1u;
static_assert(MAX_R <= 1024, "a point index takes 10 bits");
static_assert(NEAR_EXTENT - NEAR_PAD <= 32767 && -NEAR_PAD > NEAR_RADIUS, "padding points are far and fit 16 bits");
static_assert((int64_t)NEAR_RADIUS * NEAR_RADIUS < (int64_t)D2_CAP, "a link distance packs above the index");

struct ModeParams {
    int32_t R, M, minc, rd, rl, reg;
};

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// One leaf in LDS. The search holds the points in Morton order, relative to
// the leaf's minimum ({x | y << 16, z, index << 22, order}; points come before
// one another by density, then by index: order = (2047 - density) << 10 |
// index), and the bounds of every 8 consecutive ones. Afterwards the points'
// space holds the clusters' sizes and candidate roots.
struct __align__(16) ModeLds {
    u32x4_t pt[MAX_R];
    int32_t par[MAX_R];      // sort exchange; then parent by original index, then root (-1: a root)
    uint4 box[MAX_R / 8];    // lo xy, hi xy, lo z, hi z (16-bit halves)
    uint32_t first[MAX_R / 8];   // the lowest order in the group
    int32_t red[MODE_THREADS / 64][6];
    int32_t n_cand;
    uint32_t next;
};

// dynamic LDS of the mode kernels: M accumulators of 13 sums
static inline size_t mode_smem(int M) { return (size_t)13 * 8 * M; }

__device__ __forceinline__ uint32_t spread3(uint32_t v)   // 7 bits, two zeros after each
{
    v = (v | (v << 8)) & 0x0000F00Fu;
    v = (v | (v << 4)) & 0x000C30C3u;
    return (v | (v << 2)) & 0x00249249u;
}

__device__ __forceinline__ i16x2 as_i16x2(uint32_t v) { return __builtin_bit_cast(i16x2, v); }
__device__ __forceinline__ uint32_t as_u32(i16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// squared distance of two points given as (xy, z)
__device__ __forceinline__ uint32_t near_d2(uint32_t axy, uint32_t az, uint32_t bxy, uint32_t bz)
{
    const i16x2 d = as_i16x2(axy) - as_i16x2(bxy);
    const int32_t dz = (int32_t)(az - bz);
    return (uint32_t)__builtin_amdgcn_sdot2(d, d, __mul24(dz, dz), false);
}

// Where point b comes before point a: their squared distance << 10 | b's
// index, so that the least is the nearest, then the lowest index
__device__ __forceinline__ uint32_t link_key(u32x4_t a, u32x4_t b)
{
    const uint32_t c = __builtin_amdgcn_alignbit(min(near_d2(a.x, a.y, b.x, b.y), D2_CAP), b.z, 22);
    return b.w < a.w ? c : 0xFFFFFFFFu;
}

// squared gap between two bounds (lo xy, hi xy, lo z, hi z)
__device__ __forceinline__ uint32_t box_gap2(uint4 a, uint4 b)
{
    const i16x2 zero = {0, 0};
    const i16x2 g = __builtin_elementwise_max(
        __builtin_elementwise_max(as_i16x2(a.x) - as_i16x2(b.y), as_i16x2(b.x) - as_i16x2(a.y)), zero);
    const i16x2 h = __builtin_elementwise_max(
        __builtin_elementwise_max(as_i16x2(a.z) - as_i16x2(b.w), as_i16x2(b.z) - as_i16x2(a.w)), zero);
    return (uint32_t)__builtin_amdgcn_sdot2(g, g, __builtin_amdgcn_sdot2(h, h, 0, false), false);
}

// one bitonic step at distance 4 M keys (lane ^ M) over a thread's four keys
// (key i = 4 tid + e in register e), for the merge of size k
template <int M>
__device__ __forceinline__ void mode_sort_lanes(uint32_t v[4], int tid, int k)
{
    const bool lower = ((tid & M) == 0) == (((4 * tid) & k) == 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t o = xor_lane<M>(v[e]);
        v[e] = lower ? min(v[e], o) : max(v[e], o);
    }
}

__device__ __forceinline__ void mode_sort_pair(uint32_t &a, uint32_t &b, bool asc)
{
    const uint32_t lo = min(a, b), hi = max(a, b);
    a = asc ? lo : hi;
    b = asc ? hi : lo;
}

// ascending bitonic sort of the first `len` keys (a power of two, 4 at
// least), key i = 4 tid + e in register e; distances of 256 keys and more go
// through `ex` between barriers
__device__ __forceinline__ void mode_sort(uint32_t v[4], int len, int tid, uint32_t *ex)
{
    {
        const bool asc = (tid & 1) == 0;   // bit 4 of the key index
        mode_sort_pair(v[0], v[1], true);
        mode_sort_pair(v[2], v[3], false);
        mode_sort_pair(v[0], v[2], asc);
        mode_sort_pair(v[1], v[3], asc);
        mode_sort_pair(v[0], v[1], asc);
        mode_sort_pair(v[2], v[3], asc);
    }
    for (int k = 8; k <= len; k <<= 1) {
        for (int j = k >> 1; j >= 256; j >>= 1) {
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 4; ++e) ex[4 * tid + e] = v[e];
            __syncthreads();
            const bool lower = (((4 * tid) & j) == 0) == (((4 * tid) & k) == 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t o = ex[(4 * tid + e) ^ j];
                v[e] = lower ? min(v[e], o) : max(v[e], o);
            }
        }
        if (k >= 256) mode_sort_lanes<32>(v, tid, k);
        if (k >= 128) mode_sort_lanes<16>(v, tid, k);
        if (k >= 64) mode_sort_lanes<8>(v, tid, k);
        if (k >= 32) mode_sort_lanes<4>(v, tid, k);
        if (k >= 16) mode_sort_lanes<2>(v, tid, k);
        mode_sort_lanes<1>(v, tid, k);
        const bool asc = ((4 * tid) & k) == 0;
        mode_sort_pair(v[0], v[2], asc);
        mode_sort_pair(v[1], v[3], asc);
        mode_sort_pair(v[0], v[1], asc);
        mode_sort_pair(v[2], v[3], asc);
    }
}

// Density and parent of every point by the tiled search: the points are
// sorted along a Morton curve, a wavefront takes 64 consecutive points (one a
// lane) and meets only those groups of 8 whose bounds come within the radius
// of its own, whose points it reads from LDS at one address for all lanes. On
// a full-size forest a third of all pairs is left (5 % are within 5 cm, 11 %
// within 10 cm), at 6 (density) and 9 (parent) VALU instructions a pair
// against about 33 for the branching plain search. The parent pass starts
// with the tile itself and then skips every group of which no lane can use a
// point: one that comes before its own and, by the group's bounds, within its
// best distance so far (about half of the groups that come within the link
// radius of the tile). k_modes of the 200-frame full-size forest took 64.5 ms
// with the plain search, 7.3 ms without that skip and takes 6.5 ms.
// Groups of 16 leave 6 % more pairs; tiles of 32 points would leave a quarter
// but need two lists a wavefront. Handing the (point, group) pairs that are
// left, 9 lanes of 64 per group met, to a queue that refills the wavefront
// met an eighth of the groups but spent as much on the queue (6.4 to 6.7 ms,
// and small leaves 15 % slower). x0, y0, z0: the leaf's minimum; shift: cells
// of 2^shift mm, 128 an axis at most.
__device__ __forceinline__ void near_search(ModeLds &S, const Entry (&mine)[4], int n, const ModeParams mp, int x0, int y0, int z0,
                            int shift)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n64 = (n + 63) & ~63, nt = (n + 7) >> 3;
    {
        uint32_t v[4];
        u32x4_t p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * tid + e;
            const uint32_t x = (uint32_t)(mine[e].x - x0), y = (uint32_t)(mine[e].y - y0),
                           z = (uint32_t)(mine[e].z - z0);
            p[e] = u32x4_t{x | (y << 16), z, (uint32_t)i << 22, 0u};
            v[e] = i < n ? ((spread3(x >> shift) << 2 | spread3(y >> shift) << 1 | spread3(z >> shift)) << 10) |
                               (uint32_t)i
                         : 0xFFFFFFFFu;
            if (i < n) S.pt[i] = p[e];
        }
        // up to 64 points are one tile: their order does not matter
        if (n > 64) {
            int len = 128;
            while (len < n) len <<= 1;
            mode_sort(v, len, tid, (uint32_t *)S.par);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (4 * tid + e < n) p[e] = S.pt[v[e] & 1023u];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * tid + e;
            if (i < n) S.pt[i] = p[e];
            else if (i < n64)
                S.pt[i] = u32x4_t{(uint32_t)(NEAR_PAD & 0xFFFF) * 0x10001u, (uint32_t)NEAR_PAD, 0u, 0u};
        }
    }
    __syncthreads();
    if (tid < nt) {
        i16x2 lo, hi, lz, hz;
        for (int q = 0; q < 8; ++q) {
            const int i = 8 * tid + q;
            const u32x2_t p = *(const u32x2_t *)&S.pt[i < n ? i : n - 1];
            const i16x2 xy = as_i16x2(p.x), z = as_i16x2(p.y);
            lo = q ? __builtin_elementwise_min(lo, xy) : xy;
            hi = q ? __builtin_elementwise_max(hi, xy) : xy;
            lz = q ? __builtin_elementwise_min(lz, z) : z;
            hz = q ? __builtin_elementwise_max(hz, z) : z;
        }
        S.box[tid] = make_uint4(as_u32(lo), as_u32(hi), as_u32(lz), as_u32(hz));
    }
    __syncthreads();
    const uint32_t rd2 = (uint32_t)(mp.rd * mp.rd), rl2 = (uint32_t)(mp.rl * mp.rl);
    for (int pass = 0; pass < 2; ++pass) {
        const uint32_t r2 = pass ? rl2 : rd2;
        for (int b = 64 * wave; b < n; b += MODE_THREADS) {
            uint4 tb = S.box[b >> 3];
            for (int q = 1; q < 8 && (b >> 3) + q < nt; ++q) {
                const uint4 o = S.box[(b >> 3) + q];
                tb.x = as_u32(__builtin_elementwise_min(as_i16x2(tb.x), as_i16x2(o.x)));
                tb.y = as_u32(__builtin_elementwise_max(as_i16x2(tb.y), as_i16x2(o.y)));
                tb.z = as_u32(__builtin_elementwise_min(as_i16x2(tb.z), as_i16x2(o.z)));
                tb.w = as_u32(__builtin_elementwise_max(as_i16x2(tb.w), as_i16x2(o.w)));
            }
            const u32x4_t me = S.pt[b + lane];
            const uint32_t i = me.z >> 22;
            const int own = b >> 3;      // the tile's first group
            if (!pass) {
                uint32_t cnt = 0u;
                for (int g = 0; g < nt; g += 64) {
                    uint64_t m = __ballot(g + lane < nt && box_gap2(tb, S.box[min(g + lane, nt - 1)]) <= r2);
                    while (m) {
                        const u32x4_t *pp = S.pt + 8 * (g + __builtin_ctzll(m));
                        m &= m - 1;
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            const u32x2_t w = *(const u32x2_t *)(pp + q);
                            cnt += near_d2(me.x, me.y, w.x, w.y) <= rd2 ? 1u : 0u;
                        }
                    }
                }
                // the padding comes before no point; other wavefronts only read x, y and z in this pass
                const uint32_t order = b + lane < n ? ((2047u - cnt) << 10) | i : 0xFFFFFFFFu;
                ((uint32_t *)&S.pt[b + lane])[3] = order;
                uint32_t lowest = min(order, xor_lane<1>(order));
                lowest = min(lowest, xor_lane<2>(lowest));
                lowest = min(lowest, xor_lane<4>(lowest));
                if ((lane & 7) == 0) S.first[own + (lane >> 3)] = lowest;
            } else {
                uint32_t best = (rl2 + 1u) << 10;
                auto meet = [&](int g) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) best = min(best, link_key(me, S.pt[8 * g + q]));
                };
                for (int g = own; g < min(own + 8, nt); ++g) meet(g);
                const uint4 at = make_uint4(me.x, me.x, me.y, me.y);
                for (int g = 0; g < nt; g += 64) {
                    uint64_t m = __ballot(g + lane < nt && ((g + lane) ^ own) >> 3 != 0 &&
                                          box_gap2(tb, S.box[min(g + lane, nt - 1)]) <= r2);
                    for (; m; m &= m - 1) {
                        const int o = g + __builtin_ctzll(m);
                        if (__any(S.first[o] < me.w && box_gap2(at, S.box[o]) <= best >> 10)) meet(o);
                    }
                }
                if (b + lane < n) S.par[i] = best < ((rl2 + 1u) << 10) ? (int32_t)(best & 1023u) : -1;
            }
        }
        __syncthreads();
    }
}

// the same over all pairs, for any coordinates and radii
__device__ __forceinline__ void plain_search(ModeLds &S, const Entry *__restrict__ pts, int n, const ModeParams mp)
{
    int32_t *rho = (int32_t *)S.pt;
    const int rd = mp.rd, rl = mp.rl;
    const int rd2 = rd * rd, rl2 = rl * rl;
    for (int i = threadIdx.x; i < n; i += MODE_THREADS) {
        const int xi = pts[i].x, yi = pts[i].y, zi = pts[i].z;
        int cnt = 0;
        for (int j = 0; j < n; ++j) {
            const int dx = pts[j].x - xi, dy = pts[j].y - yi, dz = pts[j].z - zi;
            if (abs(dx) <= rd && abs(dy) <= rd && abs(dz) <= rd && dx * dx + dy * dy + dz * dz <= rd2) cnt++;
        }
        rho[i] = cnt;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += MODE_THREADS) {
        const int xi = pts[i].x, yi = pts[i].y, zi = pts[i].z, ri = rho[i];
        int best = -1, bd = 0;
        for (int j = 0; j < n; ++j) {
            const int dx = pts[j].x - xi, dy = pts[j].y - yi, dz = pts[j].z - zi;
            if (abs(dx) > rl || abs(dy) > rl || abs(dz) > rl) continue;
            const int d2 = dx * dx + dy * dy + dz * dz;
            if (d2 > rl2 || j == i) continue;
            const int rj = rho[j];
            if (!(rj > ri || (rj == ri && j < i))) continue;
            if (best < 0 || d2 < bd || (d2 == bd && j < best)) {
                best = j;
                bd = d2;
            }
        }
        S.par[i] = best;
    }
    __syncthreads();
}

// One workgroup per leaf. Density and parent are exact integer comparisons
// (near_search or plain_search); clusters are the trees of the parent forest
// (roots by pointer jumping); clusters of at least `minc` points are ranked by
// (size descending, root ascending) and the first M become modes. Sums are
// exact integers relative to the leaf's minimum (modulo 2^64, as the
// covariance's numerator is), so their order does not matter.
__device__ __forceinline__ void leaf_modes(const Entry *__restrict__ pts, int n, const ModeParams mp, Mode *__restrict__ out,
                           uint32_t *__restrict__ rgb_out, int rgb_len, int32_t *__restrict__ n_out, ModeLds &S,
                           unsigned long long (*acc)[13])
{
    const int tid = threadIdx.x;
    if (n < mp.minc) {   // too few points for any cluster to be kept
        if (rgb_out && tid < rgb_len) rgb_out[tid] = RGB_NONE;
        if (tid == 0) *n_out = 0;
        return;
    }
    Entry mine[4];       // points 4 tid .. + 3
    int lo[3] = {INT32_MAX, INT32_MAX, INT32_MAX}, hi[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 4 * tid + e;
        mine[e] = i < n ? pts[i] : Entry{0, 0, 0, 0u};
        if (i < n) {
            lo[0] = min(lo[0], mine[e].x); hi[0] = max(hi[0], mine[e].x);
            lo[1] = min(lo[1], mine[e].y); hi[1] = max(hi[1], mine[e].y);
            lo[2] = min(lo[2], mine[e].z); hi[2] = max(hi[2], mine[e].z);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        for (int o = 32; o >= 1; o >>= 1) {
            lo[a] = min(lo[a], __shfl_xor(lo[a], o, 64));
            hi[a] = max(hi[a], __shfl_xor(hi[a], o, 64));
        }
        if ((tid & 63) == 0) {
            S.red[tid >> 6][a] = lo[a];
            S.red[tid >> 6][3 + a] = hi[a];
        }
    }
    if (tid == 0) S.n_cand = 0;
    for (int i = tid; i < mp.M * 13; i += MODE_THREADS) acc[i / 13][i % 13] = 0ull;
    __syncthreads();
    int64_t ext = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = S.red[0][a];
        hi[a] = S.red[0][3 + a];
        for (int w = 1; w < MODE_THREADS / 64; ++w) {
            lo[a] = min(lo[a], S.red[w][a]);
            hi[a] = max(hi[a], S.red[w][3 + a]);
        }
        lo[a] = __builtin_amdgcn_readfirstlane(lo[a]);   // (the same in every thread)
        hi[a] = __builtin_amdgcn_readfirstlane(hi[a]);
        ext = max(ext, (int64_t)hi[a] - (int64_t)lo[a]);
    }
    if (ext <= NEAR_EXTENT && mp.rd <= NEAR_RADIUS && mp.rl <= NEAR_RADIUS) {
        int shift = 4;
        while ((ext >> shift) > 127) ++shift;
        near_search(S, mine, n, mp, lo[0], lo[1], lo[2], shift);
    } else {
        plain_search(S, pts, n, mp);
    }
    // pointer jumping: par[i] becomes the root of i
    for (int it = 0; it < 13; ++it) {
        bool moved = false;
        for (int i = tid; i < n; i += MODE_THREADS) {
            const int a = S.par[i];
            if (a >= 0) {
                const int b = S.par[a];
                if (b >= 0) {
                    S.par[i] = b;
                    moved = true;
                }
            }
        }
        if (!__syncthreads_or(moved)) break;
    }
    uint32_t *size = (uint32_t *)S.pt, *cand_root = size + MAX_R;
    for (int i = tid; i < n; i += MODE_THREADS) size[i] = 0u;
    __syncthreads();
    for (int i = tid; i < n; i += MODE_THREADS) {
        const int r = S.par[i];
        atomicAdd(&size[r < 0 ? i : r], 1u);
    }
    __syncthreads();
    for (int i = tid; i < n; i += MODE_THREADS)
        if (S.par[i] < 0 && size[i] >= (uint32_t)mp.minc) cand_root[atomicAdd(&S.n_cand, 1)] = (uint32_t)i;
    __syncthreads();
    // rank candidates by (size desc, root asc); a rank below M is the mode
    // slot, kept as -2 - rank in the root's parent word (roots hold -1)
    const int nc = S.n_cand;
    for (int a = tid; a < nc; a += MODE_THREADS) {
        const int ra = (int)cand_root[a];
        const uint32_t sa = size[ra];
        int rank = 0;
        for (int b = 0; b < nc; ++b) {
            const int rb = (int)cand_root[b];
            const uint32_t sb = size[rb];
            if (sb > sa || (sb == sa && rb < ra)) rank++;
        }
        if (rank < mp.M) S.par[ra] = -2 - rank;
    }
    __syncthreads();
    const int nm = nc < mp.M ? nc : mp.M;
    // (read again: held through the search, its registers would be spilled)
    Entry again[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) again[e] = pts[min(4 * tid + e, n - 1)];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 4 * tid + e;
        if (i >= n) continue;
        const int r = S.par[i];
        const int m = -2 - (r < 0 ? r : S.par[r]);
        if (m < 0) continue;
        const Entry pt = again[e];
        const unsigned long long x = (uint32_t)pt.x - (uint32_t)lo[0], y = (uint32_t)pt.y - (uint32_t)lo[1],
                                 z = (uint32_t)pt.z - (uint32_t)lo[2];
        const uint32_t cl = pt.rgb;
        atomicAdd(&acc[m][0], x);
        atomicAdd(&acc[m][1], y);
        atomicAdd(&acc[m][2], z);
        atomicAdd(&acc[m][3], x * x);
        atomicAdd(&acc[m][4], x * y);
        atomicAdd(&acc[m][5], x * z);
        atomicAdd(&acc[m][6], y * y);
        atomicAdd(&acc[m][7], y * z);
        atomicAdd(&acc[m][8], z * z);
        atomicAdd(&acc[m][9], (unsigned long long)(cl & 255u));
        atomicAdd(&acc[m][10], (unsigned long long)((cl >> 8) & 255u));
        atomicAdd(&acc[m][11], (unsigned long long)((cl >> 16) & 255u));
        atomicAdd(&acc[m][12], 1ull);
    }
    __syncthreads();
    if (tid < nm) {
        const unsigned long long *a = acc[tid];
        const uint64_t nmm = a[12];
        Mode md;
        double dn = (double)nmm;
        for (int k = 0; k < 3; ++k) md.mu[k] = (float)((double)(int64_t)(a[k] + nmm * (uint64_t)(int64_t)lo[k]) / (dn * 1000.0));
        const int ia[6] = {0, 0, 0, 1, 1, 2}, ib[6] = {0, 1, 2, 1, 2, 2};
        double S6[6];
        for (int e = 0; e < 6; ++e) {
            const int64_t num = (int64_t)(nmm * a[3 + e] - a[ia[e]] * a[ib[e]]);
            double cv = (double)num / (dn * dn);
            if (ia[e] == ib[e]) cv = cv + (double)mp.reg;
            S6[e] = cv * 1e-6;
        }
        double A = S6[0], B = S6[1], Cc = S6[2], Dd = S6[3], E = S6[4], G = S6[5];
        double A00 = Dd * G - E * E;
        double A01 = Cc * E - B * G;
        double A02 = B * E - Cc * Dd;
        double A11 = A * G - Cc * Cc;
        double A12 = B * Cc - A * E;
        double A22 = A * Dd - B * B;
        double det = (A * A00 + B * A01) + Cc * A02;
        md.sinv[0] = (float)(A00 / det);
        md.sinv[1] = (float)(A01 / det);
        md.sinv[2] = (float)(A02 / det);
        md.sinv[3] = (float)(A11 / det);
        md.sinv[4] = (float)(A12 / det);
        md.sinv[5] = (float)(A22 / det);
        md.kappa = (float)(-log(dn / (double)n) + 0.5 * (3.0 * log(2.0 * M_PI) + log(det)));
        md.n = (int32_t)nmm;
        md.rgb = (uint32_t)(a[9] / nmm) | ((uint32_t)(a[10] / nmm) << 8) | ((uint32_t)(a[11] / nmm) << 16);
        out[tid] = md;
        if (rgb_out) rgb_out[tid] = rgb_code(md.rgb);
    } else if (rgb_out && tid < rgb_len) {
        rgb_out[tid] = RGB_NONE;
    }
    if (tid == 0) *n_out = nm;
}

// the flagged leaves as a list, 4 leaves a thread
__global__ void __launch_bounds__(256) k_dirty_list(const uint32_t *__restrict__ dirty, int n,
                                                    uint32_t *__restrict__ list, uint32_t *__restrict__ work)
{
    __shared__ uint32_t wave_n[4], at0;
    const int i = 4 * (int)(blockIdx.x * 256 + threadIdx.x), lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bool is[4];
    uint64_t m[4];
    uint32_t mine = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        is[e] = i + e < n && dirty[i + e] != 0u;
        m[e] = __ballot(is[e]);
        mine += (uint32_t)__popcll(m[e]);
    }
    if (lane == 0) wave_n[wave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) at0 = atomicAdd(&work[0], wave_n[0] + wave_n[1] + wave_n[2] + wave_n[3]);
    __syncthreads();
    uint32_t at = at0;
    for (int w = 0; w < wave; ++w) at += wave_n[w];
    const uint64_t before = (1ull << lane) - 1ull;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (is[e]) list[at + (uint32_t)__popcll(m[e] & before)] = (uint32_t)(i + e);
        at += (uint32_t)__popcll(m[e]);
    }
}

// Leaves of the dirty list; work[0] is the list's length. They are handed out
// by a ticket (work[1]) since their point counts differ by three orders of
// magnitude, unless reservoirs hold no more than a tile's points: such leaves
// take about 2 us each whatever they hold, and the tickets' additions to one
// address cost as much (20 480 leaves of 1 point 31 us, with tickets 100; of 16
// 97 and 117, of 64 118 and 124; leaves of 128 points 142 and 139, of 1024 in a
// deep forest's first frame 582 and 496). Clears each leaf's dirty flag and refreshes its summary for the
// learned proposal's inputs: {min(k, R), number of modes kept (<= 3)} and, for
// its first three modes (the heaviest: modes are ranked by size),
// {pi = n / min(k, R), -log(Sigma^-1_xx) / 10, -log(Sigma^-1_yy) / 10,
// -log(Sigma^-1_zz) / 10}
__global__ void __launch_bounds__(MODE_THREADS, 6) k_modes(const uint32_t *__restrict__ list,
                                                        uint32_t *__restrict__ work,
                                                        uint32_t *__restrict__ dirty,
                                                        const uint32_t *__restrict__ counter,
                                                        const Entry *__restrict__ res, ModeParams mp,
                                                        Mode *__restrict__ modes, uint32_t *__restrict__ mode_rgb,
                                                        int32_t *__restrict__ nmodes, float4 *__restrict__ leaf_in)
{
    extern __shared__ unsigned long long mode_acc[];
    __shared__ ModeLds S;
    const int tid = (int)threadIdx.x;
    const uint32_t n_list = work[0];
    const bool tickets = mp.R > 64;
    uint32_t it = blockIdx.x;
    while (it < n_list) {
        uint32_t ahead = 0u;   // the next leaf, asked for before this one's work
        if (tid == 0) ahead = tickets ? atomicAdd(&work[1], 1u) : it;
        const uint32_t li = list[it];
        const uint32_t k = counter[li];
        const int n = k < (uint32_t)mp.R ? (int)k : mp.R;
        const int ms = rgb_stride(mp.M);
        leaf_modes(res + (int64_t)li * mp.R, n, mp, modes + (int64_t)li * mp.M, mode_rgb + (int64_t)li * ms, ms,
                   nmodes + li, S, (unsigned long long(*)[13])mode_acc);
        if (tid == 0) {
            S.next = gridDim.x + ahead;
            dirty[li] = 0u;
        }
        __syncthreads();   // the modes, their count and the next ticket are visible
        it = S.next;
        if (tid < 4) {
            const int nm = nmodes[li];
            const int n3 = nm < 3 ? nm : 3;
            float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (tid == 0) {
                q.x = __uint_as_float((uint32_t)n);
                q.y = __int_as_float(n3);
            } else if (tid - 1 < n3) {
                const Mode md = modes[(int64_t)li * mp.M + tid - 1];
                q.x = (float)md.n / (float)n;
                q.y = -logf(md.sinv[0]) / 10.0f;
                q.z = -logf(md.sinv[3]) / 10.0f;
                q.w = -logf(md.sinv[5]) / 10.0f;
            }
            leaf_in[(int64_t)li * 4 + tid] = q;
        }
        __syncthreads();   // S is the next leaf's
    }
}

// the dirty list is empty again
__global__ void k_modes_done(uint32_t *__restrict__ work)
{
    work[threadIdx.x] = 0u;
}

__global__ void __launch_bounds__(MODE_THREADS) k_modes_points(const Entry *__restrict__ pts, int n, ModeParams mp,
                                                               Mode *__restrict__ out, int32_t *__restrict__ n_out)
{
    extern __shared__ unsigned long long mode_acc[];
    __shared__ ModeLds S;
    leaf_modes(pts, n, mp, out, nullptr, 0, n_out, S, (unsigned long long(*)[13])mode_acc);
}

static ModeParams mode_params(const Forest *f)
{
    ModeParams mp;
    mp.R = f->R;
    mp.M = f->M;
    mp.minc = f->p.min_cluster > 0 ? f->p.min_cluster : std::max(3, f->R / 64);
    mp.rd = f->p.dens_radius_mm;
    mp.rl = f->p.link_radius_mm;
    mp.reg = f->p.cov_reg_mm2;
    return mp;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

// workgroups of k_reservoir per tree
static int64_t res_blocks(int64_t P) { return (P + RES_THREADS - 1) / RES_THREADS; }

static void free_frame_scratch(Forest *f, size_t room = 0)
{
    dfree(f, &f->leaves, (size_t)f->T * f->cap_P, room);
    dfree(f, &f->packed, (size_t)PACKED_WORDS * f->cap_P, room);
    dfree(f, &f->rank, (size_t)f->T * f->cap_P, room);
    dfree(f, &f->late, (size_t)f->T * res_blocks(f->cap_P) * RES_THREADS * sizeof(Late), room);
    dfree(f, &f->n_late, (size_t)f->T * res_blocks(f->cap_P), room);
    f->cap_P = 0;
}

static void free_chunk_tables(Forest *f, size_t room = 0)
{
    dfree(f, &f->chunk_cnt, (size_t)f->T * f->cap_C * f->L, room);
    dfree(f, &f->chunk_pref, (size_t)f->T * f->cap_C * f->L, room);
    f->cap_C = 0;
}

static int ensure_frame_scratch(Forest *f, int64_t P, hipStream_t s)
{
    // (the capacities are set first: what a failure has to give back has their sizes)
    if (P > f->cap_P) {
        free_frame_scratch(f);
        f->cap_P = P;
        int rc = RELOC_OK;
        rc |= dalloc(f, &f->leaves, (size_t)f->T * P, s);
        rc |= dalloc(f, &f->packed, (size_t)PACKED_WORDS * P, s);
        rc |= dalloc(f, &f->rank, (size_t)f->T * P, s);
        rc |= dalloc(f, &f->late, (size_t)f->T * res_blocks(P) * RES_THREADS * sizeof(Late), s);
        rc |= dalloc(f, &f->n_late, (size_t)f->T * res_blocks(P), s);
        if (rc) {
            free_frame_scratch(f);
            return RELOC_E_NOMEM;
        }
    }
    const int chunk = chunk_pixels(P, f->T, f->L);
    const int64_t C = (P + chunk - 1) / chunk;
    if (C > f->cap_C) {
        free_chunk_tables(f);
        f->cap_C = C;
        int rc = RELOC_OK;
        rc |= dalloc(f, &f->chunk_cnt, (size_t)f->T * C * f->L, s);
        rc |= dalloc(f, &f->chunk_pref, (size_t)f->T * C * f->L, s);
        if (!rc && hipMemsetAsync(f->chunk_cnt, 0, (size_t)f->T * C * f->L * sizeof(uint16_t), s) != hipSuccess)
            rc = RELOC_E_HIP;
        if (rc) {
            free_chunk_tables(f);
            return rc == RELOC_E_HIP ? RELOC_E_HIP : RELOC_E_NOMEM;
        }
    }
    return RELOC_OK;
}

int update_modes(Forest *f, hipStream_t s)
{
    if (!f->maybe_dirty) return RELOC_OK;
    if (!f->res) return RELOC_E_STATE;
    ModeParams mp = mode_params(f);
    int grid = std::min(f->T * f->L, 256 * 8);
    RL_LAUNCH("k_dirty_list", k_dirty_list, dim3((unsigned)((f->T * f->L + 1023) / 1024)), dim3(256), 0, s, f->dirty,
              f->T * f->L, f->dirty_list, f->dirty_count);
    RL_LAUNCH("k_modes", k_modes, dim3(grid), dim3(MODE_THREADS), mode_smem(f->M), s, f->dirty_list, f->dirty_count,
                       f->dirty, f->counter, f->res, mp, f->modes, f->mode_rgb, f->nmodes, f->leaf_in);
    RL_LAUNCH("k_modes_done", k_modes_done, dim3(1), dim3(2), 0, s, f->dirty_count);
    RL_HIP(hipGetLastError());
    f->maybe_dirty = false;
    return RELOC_OK;
}

int traverse_frame(Forest *f, const Frame &fr, hipStream_t s)
{
    int64_t P = (int64_t)fr.W * fr.H;
    int rc = ensure_frame_scratch(f, P, s);
    if (rc) return rc;
    RL_LAUNCH("k_pack", k_pack, dim3((unsigned)((P + 1023) / 1024)), dim3(256), 0, s, fr, f->packed);
    RL_LAUNCH("k_leaves", k_leaves, dim3((unsigned)((P + LEAF_PIX * 256 - 1) / (LEAF_PIX * 256)), (unsigned)f->T),
              dim3(256), 0, s, f->nodes, f->deep, f->T, f->L, fr, f->packed, f->leaves);
    RL_HIP(hipGetLastError());
    return RELOC_OK;
}

int frame_from(const Forest *f, const uint16_t *depth, const uint8_t *rgb, const reloc_intrinsics *K, Frame &fr)
{
    return frame_of(f, depth, rgb, K, fr);
}

bool pose_is_se3(const double T[16]) { return is_se3(T); }

// every leaf of a forest empty again (the state of a new forest): counters,
// reservoirs, slot stamps, modes, the learned proposal's leaf summaries,
// the dirty list and the sample count
int forest_empty_leaves(Forest *f, hipStream_t s)
{
    const size_t TL = (size_t)f->T * f->L;
    if (f->dropped) return RELOC_E_STATE;
    if (hipMemsetAsync(f->counter, 0, TL * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->stamp, 0, TL * f->R * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->res, 0, TL * f->R * sizeof(Entry), s) != hipSuccess ||
        hipMemsetAsync(f->nmodes, 0, TL * sizeof(int32_t), s) != hipSuccess ||
        hipMemsetAsync(f->mode_rgb, 0xFF, TL * rgb_stride(f->M) * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->leaf_in, 0, TL * 4 * sizeof(float4), s) != hipSuccess ||
        hipMemsetAsync(f->dirty, 0, TL * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->dirty_count, 0, 2 * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->total_samples, 0, sizeof(unsigned long long), s) != hipSuccess)
        return RELOC_E_HIP;
    f->maybe_dirty = false;
    return RELOC_OK;
}

}  // namespace rl

using namespace rl;

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------

extern "C" int reloc_params_default(reloc_params *out)
{
    if (!out) return RELOC_E_ARG;
    params_default(out);
    return RELOC_OK;
}

extern "C" const char *reloc_status_string(int code)
{
    switch (code) {
    case RELOC_OK: return "ok";
    case RELOC_FAIL_NO_VALID_PIXELS: return "relocalisation failed: no valid depth in the frame";
    case RELOC_FAIL_NO_MODES: return "relocalisation failed: the forest has never been adapted";
    case RELOC_FAIL_NO_HYPOTHESIS: return "relocalisation failed: no hypothesis passed its checks";
    case RELOC_E_ARG: return "invalid argument";
    case RELOC_E_NOMEM: return "device allocation failed";
    case RELOC_E_HIP: return "HIP runtime error";
    case RELOC_E_STATE: return "operation not valid in this state";
    case RELOC_E_RANGE: return "value does not fit the packed device layout";
    case RELOC_E_IO: return "checkpoint file cannot be written or read, or is not a forest checkpoint";
    default: return "unknown status";
    }
}

static void forest_free(Forest *f, size_t room = 0)
{
    size_t TL = (size_t)f->T * f->L;
    dfree(f, &f->nodes, (size_t)f->T * (f->L - 1) + 8, room);
    dfree(f, &f->deep, (size_t)f->T * (f->L - 1), room);
    dfree(f, &f->counter, TL, room);
    dfree(f, &f->base, TL, room);
    dfree(f, &f->res, TL * f->R, room);
    dfree(f, &f->stamp, TL * f->R, room);
    dfree(f, &f->modes, TL * f->M, room);
    dfree(f, &f->nmodes, TL, room);
    dfree(f, &f->dirty, TL, room);
    dfree(f, &f->dirty_list, TL, room);
    dfree(f, &f->dirty_count, 2, room);
    dfree(f, &f->total_samples, 1, room);
    free_frame_scratch(f, room);
    free_chunk_tables(f, room);
    dfree(f, &f->mode_rgb, TL * rgb_stride(f->M), room);
    dfree(f, &f->leaf_in, TL * 4, room);
}

extern "C" int reloc_forest_create(const reloc_params *p, void *stream, reloc_forest **out)
{
    if (!p || !out) return RELOC_E_ARG;
    *out = nullptr;
    int rc = params_check(p);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    reloc_forest *f = new (std::nothrow) reloc_forest();
    if (!f) return RELOC_E_NOMEM;
    f->p = *p;
    f->T = p->n_trees; f->D = p->depth; f->L = 1 << p->depth; f->R = p->reservoir_size; f->M = p->max_modes;
    if (hipGetDevice(&f->device) != hipSuccess) { delete f; return RELOC_E_HIP; }
    size_t TL = (size_t)f->T * f->L;
    rc = RELOC_OK;
    rc |= dalloc(f, &f->nodes, (size_t)f->T * (f->L - 1) + 8, s);
    rc |= dalloc(f, &f->deep, (size_t)f->T * (f->L - 1), s);
    rc |= dalloc(f, &f->counter, TL, s);
    rc |= dalloc(f, &f->base, TL, s);
    rc |= dalloc(f, &f->res, TL * f->R, s);
    rc |= dalloc(f, &f->stamp, TL * f->R, s);
    rc |= dalloc(f, &f->modes, TL * f->M, s);
    rc |= dalloc(f, &f->nmodes, TL, s);
    rc |= dalloc(f, &f->dirty, TL, s);
    rc |= dalloc(f, &f->dirty_list, TL, s);
    rc |= dalloc(f, &f->dirty_count, 2, s);
    rc |= dalloc(f, &f->total_samples, 1, s);
    rc |= dalloc(f, &f->mode_rgb, TL * rgb_stride(f->M), s);
    rc |= dalloc(f, &f->leaf_in, TL * 4, s);
    if (rc) {
        forest_free(f);
        delete f;
        return RELOC_E_NOMEM;
    }
    if (hipMemsetAsync(f->counter, 0, TL * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->stamp, 0, TL * f->R * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->res, 0, TL * f->R * sizeof(Entry), s) != hipSuccess ||
        hipMemsetAsync(f->nmodes, 0, TL * sizeof(int32_t), s) != hipSuccess ||
        hipMemsetAsync(f->mode_rgb, 0xFF, TL * rgb_stride(f->M) * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->leaf_in, 0, TL * 4 * sizeof(float4), s) != hipSuccess ||
        hipMemsetAsync(f->dirty, 0, TL * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->dirty_count, 0, 2 * sizeof(uint32_t), s) != hipSuccess ||
        hipMemsetAsync(f->total_samples, 0, sizeof(unsigned long long), s) != hipSuccess) {
        forest_free(f);
        delete f;
        return RELOC_E_HIP;
    }
    int64_t nn = (int64_t)f->T * (f->L - 1) + 8;
    RL_LAUNCH("k_gen_nodes", k_gen_nodes, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, f->nodes, f->deep, f->T, f->L,
                       p->seed, p->offset_pxmm, p->thr_depth_mm, p->thr_rgb);
    if (hipGetLastError() != hipSuccess) {
        forest_free(f);
        delete f;
        return RELOC_E_HIP;
    }
    *out = f;
    return RELOC_OK;
}

extern "C" int reloc_forest_destroy(reloc_forest *f)
{
    if (!f) return RELOC_E_ARG;
    // (the wait fails while another thread captures a graph: nothing is kept then)
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    rl_free_plain(f);
    forest_free(f, idle ? kept_room(f->bytes, f->device) : 0);
    if (!idle) (void)hipGetLastError();   // (not left for the next launch's check)
    kept_expire();
    delete f;
    return RELOC_OK;
}

extern "C" int reloc_trim(void)
{
    kept_release([](const Block &, size_t) { return true; });
    return RELOC_OK;
}

extern "C" int reloc_forest_params(const reloc_forest *f, reloc_params *out)
{
    if (!f || !out) return RELOC_E_ARG;
    *out = f->p;
    return RELOC_OK;
}

extern "C" int reloc_forest_memory(const reloc_forest *f, uint64_t *bytes_out)
{
    if (!f || !bytes_out) return RELOC_E_ARG;
    *bytes_out = f->bytes;
    return RELOC_OK;
}

extern "C" int reloc_adapt_frame(reloc_forest *f, const uint16_t *depth_dev, const uint8_t *rgb_dev,
                                 const reloc_intrinsics *K, const double pose_c2w[16], void *stream)
{
    if (!f || !pose_c2w) return RELOC_E_ARG;
    if (f->dropped) return RELOC_E_STATE;
    Frame fr;
    int rc = frame_of(f, depth_dev, rgb_dev, K, fr);
    if (rc) return rc;
    if (!is_se3(pose_c2w)) return RELOC_E_ARG;
    hipStream_t s = (hipStream_t)stream;
    int64_t P = (int64_t)fr.W * fr.H;
    rc = traverse_frame(f, fr, s);
    if (rc) return rc;
    const int chunk = chunk_pixels(P, f->T, f->L), C = (int)((P + chunk - 1) / chunk);
    Pose32 ps;
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) ps.R[r * 3 + c] = (float)pose_c2w[r * 4 + c];
        ps.t[r] = (float)pose_c2w[r * 4 + 3];
    }
    Late *late = (Late *)f->late;
    auto rank_kernel = chunk == 2 * RANK_THREADS ? k_chunk_rank<2> : chunk == 4 * RANK_THREADS ? k_chunk_rank<4> : k_chunk_rank<8>;
    RL_LAUNCH("k_chunk_rank", rank_kernel, dim3(C, f->T), dim3(RANK_THREADS), rank_smem(f->L), s, f->leaves, (int)P, f->L,
              f->D, C, f->rank, f->chunk_cnt);
    const int64_t TL = (int64_t)f->T * f->L;
    RL_LAUNCH("k_leaf_scan", k_leaf_scan, dim3((unsigned)((TL + 127) / 128)), dim3(256), 0, s, f->T, f->L, C, f->chunk_cnt,
              f->chunk_pref, f->counter, f->base, f->dirty, f->total_samples);
    const int64_t nb = res_blocks(P), lists = nb * f->T;
    RL_LAUNCH("k_reservoir", k_reservoir, dim3((unsigned)nb, (unsigned)f->T), dim3(RES_THREADS), 0, s, f->leaves, f->rank,
              f->chunk_pref, f->base, f->L, f->R, C, chunk, f->p.seed, fr, ps, f->stamp, f->res, late, f->n_late);
    RL_LAUNCH("k_late", k_late, dim3((unsigned)((lists + 3) / 4)), dim3(256), 0, s, late, f->n_late, (int)lists, f->stamp,
              fr, ps, f->res);
    RL_HIP(hipGetLastError());
    f->maybe_dirty = true;
    return RELOC_OK;
}

extern "C" int reloc_update_modes(reloc_forest *f, void *stream)
{
    if (!f) return RELOC_E_ARG;
    return update_modes(f, (hipStream_t)stream);
}

extern "C" int reloc_forest_drop_reservoirs(reloc_forest *f, void *stream)
{
    if (!f) return RELOC_E_ARG;
    if (f->dropped) return RELOC_OK;
    hipStream_t s = (hipStream_t)stream;
    int rc = update_modes(f, s);
    if (rc) return rc;
    RL_HIP(hipStreamSynchronize(s));
    size_t TLR = (size_t)f->T * f->L * f->R;
    dfree(f, &f->res, TLR);
    dfree(f, &f->stamp, TLR);
    f->dropped = true;
    return RELOC_OK;
}

// ---- checkpoint: save and load ---------------------------------------------
//
// File layout (little-endian, this library's own format): a FileHeader, then
// the split nodes (u64 [T (L - 1) + 8]), leaf counters (u32 [T L]), mode
// counts (i32 [T L]), modes (Mode [T L M]), mode colour rows
// (u32 [T L rgb_stride(M)], as r | g << 8 | b << 16 or RGB_NONE), learned-input leaf summaries (float4 [T L 4])
// and, unless the reservoirs were dropped, the reservoirs (Entry [T L R]).
// Slot stamps are not stored: a stamp only has to be below every k + 1 that
// later frames can produce, and every later k is at least the leaf's counter,
// so the zero stamps of a new forest select the same winners.

namespace {

struct FileHeader {
    char magic[8];
    uint32_t version;
    uint32_t dropped;
    reloc_params p;
    uint64_t total_samples;
    uint64_t n_nodes, n_leaves, n_mode_slots, n_rgb, n_res;
};

constexpr char FILE_MAGIC[8] = {'R', 'L', 'F', 'O', 'R', 'E', 'S', 'T'};
constexpr uint32_t FILE_VERSION = 1;
constexpr size_t STAGE_BYTES = (size_t)64 << 20;

void clear_unused_modes(Mode *modes, const int32_t *count, size_t leaves, int M)
{
    for (size_t i = 0; i < leaves; ++i) {
        const int n = std::min(std::max(count[i], 0), M);
        memset((void *)(modes + i * M + n), 0, (size_t)(M - n) * sizeof(Mode));
    }
}

struct Staging {
    void *buf = nullptr;
    ~Staging()
    {
        if (buf) (void)hipHostFree(buf);
    }
};

// device -> file in chunks of whole units through pinned host memory, each
// handed to pass(buffer, offset, bytes) on the way
template <typename Pass>
int save_section(FILE *fp, const void *dev, size_t bytes, Staging &st, hipStream_t s, Pass pass, size_t unit = 4)
{
    const char *src = (const char *)dev;
    const size_t chunk = STAGE_BYTES / unit * unit;
    for (size_t off = 0; off < bytes; off += chunk) {
        const size_t n = std::min(chunk, bytes - off);
        RL_HIP(hipMemcpyAsync(st.buf, src + off, n, hipMemcpyDeviceToHost, s));
        RL_HIP(hipStreamSynchronize(s));
        pass(st.buf, off, n);
        if (fwrite(st.buf, 1, n, fp) != n) return RELOC_E_IO;
    }
    return RELOC_OK;
}

int save_section(FILE *fp, const void *dev, size_t bytes, Staging &st, hipStream_t s)
{
    return save_section(fp, dev, bytes, st, s, [](void *, size_t, size_t) {});
}

// file -> device in chunks through pinned host memory, every 32-bit word passed
// through `word` on the way where it is given
int load_section(FILE *fp, void *dev, size_t bytes, Staging &st, hipStream_t s,
                 uint32_t (*word)(uint32_t) = nullptr)
{
    char *dst = (char *)dev;
    for (size_t off = 0; off < bytes; off += STAGE_BYTES) {
        const size_t n = std::min(STAGE_BYTES, bytes - off);
        RL_HIP(hipStreamSynchronize(s));   // the previous chunk has left the staging buffer
        if (fread(st.buf, 1, n, fp) != n) return RELOC_E_IO;
        if (word)
            for (size_t i = 0; i < n / 4; ++i) ((uint32_t *)st.buf)[i] = word(((uint32_t *)st.buf)[i]);
        RL_HIP(hipMemcpyAsync(dst + off, st.buf, n, hipMemcpyHostToDevice, s));
    }
    RL_HIP(hipStreamSynchronize(s));
    return RELOC_OK;
}

FileHeader header_of(const Forest *f)
{
    FileHeader h;
    memset(&h, 0, sizeof(h));
    memcpy(h.magic, FILE_MAGIC, sizeof(FILE_MAGIC));
    h.version = FILE_VERSION;
    h.dropped = f->dropped ? 1u : 0u;
    h.p = f->p;
    const uint64_t TL = (uint64_t)f->T * f->L;
    h.n_nodes = (uint64_t)f->T * (f->L - 1) + 8;
    h.n_leaves = TL;
    h.n_mode_slots = TL * f->M;
    h.n_rgb = TL * rgb_stride(f->M);
    h.n_res = f->dropped ? 0 : TL * f->R;
    return h;
}

int save_forest(Forest *f, FILE *fp, hipStream_t s)
{
    int rc = update_modes(f, s);
    if (rc) return rc;
    Staging st;
    RL_HIP(hipHostMalloc(&st.buf, STAGE_BYTES, hipHostMallocDefault));
    FileHeader h = header_of(f);
    RL_HIP(hipMemcpyAsync(&h.total_samples, f->total_samples, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
    RL_HIP(hipStreamSynchronize(s));
    if (fwrite(&h, sizeof(h), 1, fp) != 1) return RELOC_E_IO;
    if ((rc = save_section(fp, f->nodes, h.n_nodes * sizeof(uint64_t), st, s))) return rc;
    if ((rc = save_section(fp, f->counter, h.n_leaves * sizeof(uint32_t), st, s))) return rc;
    if ((rc = save_section(fp, f->nmodes, h.n_leaves * sizeof(int32_t), st, s))) return rc;
    // (a leaf's unused mode slots hold whatever was there before: zeros in the file)
    std::unique_ptr<int32_t[]> count(new (std::nothrow) int32_t[h.n_leaves]);
    if (!count) return RELOC_E_NOMEM;
    RL_HIP(hipMemcpyAsync(count.get(), f->nmodes, h.n_leaves * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    const size_t leaf = f->M * sizeof(Mode);
    if ((rc = save_section(fp, f->modes, h.n_mode_slots * sizeof(Mode), st, s,
                           [&](void *buf, size_t off, size_t n) {
                               clear_unused_modes((Mode *)buf, count.get() + off / leaf, n / leaf, f->M);
                           },
                           leaf)))
        return rc;
    if ((rc = save_section(fp, f->mode_rgb, h.n_rgb * sizeof(uint32_t), st, s, [](void *buf, size_t, size_t n) {
             for (size_t i = 0; i < n / 4; ++i) ((uint32_t *)buf)[i] = rgb_of_code(((uint32_t *)buf)[i]);
         })))
        return rc;
    if ((rc = save_section(fp, f->leaf_in, h.n_leaves * 4 * sizeof(float4), st, s))) return rc;
    if (!f->dropped && (rc = save_section(fp, f->res, h.n_res * sizeof(Entry), st, s))) return rc;
    return RELOC_OK;
}

int load_forest(FILE *fp, hipStream_t s, reloc_forest **out)
{
    FileHeader h;
    if (fread(&h, sizeof(h), 1, fp) != 1) return RELOC_E_IO;
    if (memcmp(h.magic, FILE_MAGIC, sizeof(FILE_MAGIC)) != 0 || h.version != FILE_VERSION || h.dropped > 1u)
        return RELOC_E_IO;
    reloc_forest *f = nullptr;
    int rc = reloc_forest_create(&h.p, s, &f);
    if (rc) return rc;
    const FileHeader want = [&] {
        FileHeader w = header_of(f);
        if (h.dropped) w.n_res = 0;
        return w;
    }();
    if (h.n_nodes != want.n_nodes || h.n_leaves != want.n_leaves || h.n_mode_slots != want.n_mode_slots ||
        h.n_rgb != want.n_rgb || h.n_res != want.n_res) {
        reloc_forest_destroy(f);
        return RELOC_E_IO;
    }
    Staging st;
    std::vector<uint64_t> nodes(h.n_nodes);
    std::vector<DeepNode> deep((size_t)f->T * (f->L - 1));
    rc = hipHostMalloc(&st.buf, STAGE_BYTES, hipHostMallocDefault) == hipSuccess ? RELOC_OK : RELOC_E_NOMEM;
    if (!rc && fread(nodes.data(), sizeof(uint64_t), nodes.size(), fp) != nodes.size()) rc = RELOC_E_IO;
    if (!rc) {
        // split nodes are checked like reloc_debug_set_nodes checks them
        for (size_t i = 0; i < nodes.size() && !rc; ++i) {
            int32_t kind, dx, dy, thr;
            unpack_node(nodes[i], kind, dx, dy, thr);
            if (kind < 0 || kind > 3 || (int64_t)std::abs((int64_t)dx) > f->p.offset_pxmm ||
                (int64_t)std::abs((int64_t)dy) > f->p.offset_pxmm || pack_node(kind, dx, dy, thr) != nodes[i])
                rc = RELOC_E_RANGE;
        }
        for (size_t i = 0; i < deep.size() && !rc; ++i) deep[i] = deep_node(nodes[i]);
    }
    if (!rc && (hipMemcpyAsync(f->nodes, nodes.data(), nodes.size() * sizeof(uint64_t), hipMemcpyHostToDevice, s) !=
                    hipSuccess ||
                hipMemcpyAsync(f->deep, deep.data(), deep.size() * sizeof(DeepNode), hipMemcpyHostToDevice, s) !=
                    hipSuccess ||
                hipMemcpyAsync(f->total_samples, &h.total_samples, sizeof(uint64_t), hipMemcpyHostToDevice, s) !=
                    hipSuccess))
        rc = RELOC_E_HIP;
    if (!rc) rc = load_section(fp, f->counter, h.n_leaves * sizeof(uint32_t), st, s);
    if (!rc) rc = load_section(fp, f->nmodes, h.n_leaves * sizeof(int32_t), st, s);
    if (!rc) rc = load_section(fp, f->modes, h.n_mode_slots * sizeof(Mode), st, s);
    if (!rc) rc = load_section(fp, f->mode_rgb, h.n_rgb * sizeof(uint32_t), st, s, rgb_code);
    if (!rc) rc = load_section(fp, f->leaf_in, h.n_leaves * 4 * sizeof(float4), st, s);
    if (!rc && !h.dropped) rc = load_section(fp, f->res, h.n_res * sizeof(Entry), st, s);
    if (!rc && fgetc(fp) != EOF) rc = RELOC_E_IO;   // trailing bytes: not a file this version wrote
    if (!rc && hipStreamSynchronize(s) != hipSuccess) rc = RELOC_E_HIP;
    if (!rc && h.dropped) {
        const size_t TLR = (size_t)f->T * f->L * f->R;
        dfree(f, &f->res, TLR);
        dfree(f, &f->stamp, TLR);
        f->dropped = true;
    }
    if (rc) {
        reloc_forest_destroy(f);
        return rc;
    }
    f->maybe_dirty = false;
    *out = f;
    return RELOC_OK;
}

}  // namespace

extern "C" int reloc_forest_save(reloc_forest *f, const char *path, void *stream)
{
    if (!f || !path) return RELOC_E_ARG;
    FILE *fp = fopen(path, "wb");
    if (!fp) return RELOC_E_IO;
    int rc = save_forest(f, fp, (hipStream_t)stream);
    if (fclose(fp) != 0 && !rc) rc = RELOC_E_IO;
    return rc;
}

extern "C" int reloc_forest_load(const char *path, void *stream, reloc_forest **out)
{
    if (!path || !out) return RELOC_E_ARG;
    *out = nullptr;
    FILE *fp = fopen(path, "rb");
    if (!fp) return RELOC_E_IO;
    const int rc = load_forest(fp, (hipStream_t)stream, out);
    fclose(fp);
    return rc;
}

// ---- debug exports --------------------------------------------------------

extern "C" int reloc_debug_nodes(const reloc_forest *f, int32_t *kind, int32_t *dx, int32_t *dy, int32_t *thr)
{
    if (!f) return RELOC_E_ARG;
    size_t n = (size_t)f->T * (f->L - 1) + 8;
    uint64_t *h = (uint64_t *)malloc(n * sizeof(uint64_t));
    if (!h) return RELOC_E_NOMEM;
    if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(h, f->nodes, n * 8, hipMemcpyDeviceToHost) != hipSuccess) {
        free(h);
        return RELOC_E_HIP;
    }
    for (size_t i = 0; i < n; ++i) {
        int32_t a, b, c, d;
        unpack_node(h[i], a, b, c, d);
        if (kind) kind[i] = a;
        if (dx) dx[i] = b;
        if (dy) dy[i] = c;
        if (thr) thr[i] = d;
    }
    free(h);
    return RELOC_OK;
}

extern "C" int reloc_debug_set_nodes(reloc_forest *f, const int32_t *kind, const int32_t *dx, const int32_t *dy,
                                     const int32_t *thr)
{
    if (!f || !kind || !dx || !dy || !thr) return RELOC_E_ARG;
    size_t n = (size_t)f->T * (f->L - 1) + 8;
    uint64_t *h = (uint64_t *)malloc(n * sizeof(uint64_t));
    if (!h) return RELOC_E_NOMEM;
    for (size_t i = 0; i < n; ++i) {
        if (kind[i] < 0 || kind[i] > 3 || dx[i] < -NODE_OFF_MAX - 1 || dx[i] > NODE_OFF_MAX ||
            dy[i] < -NODE_OFF_MAX - 1 || dy[i] > NODE_OFF_MAX || thr[i] < -NODE_THR_MAX - 1 || thr[i] > NODE_THR_MAX ||
            (int64_t)std::abs((int64_t)dx[i]) > f->p.offset_pxmm || (int64_t)std::abs((int64_t)dy[i]) > f->p.offset_pxmm) {
            free(h);
            return RELOC_E_RANGE;
        }
        h[i] = pack_node(kind[i], dx[i], dy[i], thr[i]);
    }
    const size_t ns = (size_t)f->T * (f->L - 1);
    DeepNode *hd = (DeepNode *)malloc(ns * sizeof(DeepNode));
    if (!hd) {
        free(h);
        return RELOC_E_NOMEM;
    }
    for (size_t i = 0; i < ns; ++i) hd[i] = deep_node(h[i]);
    int rc = RELOC_OK;
    if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(f->nodes, h, n * 8, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(f->deep, hd, ns * sizeof(DeepNode), hipMemcpyHostToDevice) != hipSuccess)
        rc = RELOC_E_HIP;
    free(hd);
    free(h);
    return rc;
}

extern "C" int reloc_debug_leaves(reloc_forest *f, const uint16_t *depth_dev, const uint8_t *rgb_dev,
                                  const reloc_intrinsics *K, int32_t *leaves_host, void *stream)
{
    if (!f || !leaves_host) return RELOC_E_ARG;
    Frame fr;
    int rc = frame_of(f, depth_dev, rgb_dev, K, fr);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    rc = traverse_frame(f, fr, s);
    if (rc) return rc;
    int64_t P = (int64_t)fr.W * fr.H;
    RL_HIP(hipMemcpyAsync(leaves_host, f->leaves, (size_t)f->T * P * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    RL_HIP(hipStreamSynchronize(s));
    return RELOC_OK;
}

extern "C" int reloc_debug_features8(reloc_forest *f, const uint16_t *depth_dev, const uint8_t *rgb_dev,
                                     const reloc_intrinsics *K, int32_t *feat_host, void *stream)
{
    if (!f || !feat_host) return RELOC_E_ARG;
    Frame fr;
    int rc = frame_of(f, depth_dev, rgb_dev, K, fr);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    int64_t P = (int64_t)fr.W * fr.H;
    int32_t *d = nullptr;
    RL_HIP(device_malloc_async((void **)&d, (size_t)P * 8 * sizeof(int32_t), s));
    RL_LAUNCH("k_features8", k_features8, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s,
                       f->nodes + (int64_t)f->T * (f->L - 1), fr, d);
    hipError_t e = hipMemcpyAsync(feat_host, d, (size_t)P * 8 * sizeof(int32_t), hipMemcpyDeviceToHost, s);
    (void)hipFreeAsync(d, s);
    RL_HIP(e);
    RL_HIP(hipStreamSynchronize(s));
    return RELOC_OK;
}

extern "C" int reloc_debug_reservoir(const reloc_forest *f, int32_t t, int32_t leaf0, int32_t n, void *entries_host,
                                     uint32_t *counters_host)
{
    if (!f || t < 0 || t >= f->T || leaf0 < 0 || n < 0 || leaf0 + n > f->L) return RELOC_E_ARG;
    if (f->dropped && entries_host) return RELOC_E_STATE;
    RL_HIP(hipDeviceSynchronize());
    int64_t li = (int64_t)t * f->L + leaf0;
    if (entries_host)
        RL_HIP(hipMemcpy(entries_host, f->res + li * f->R, (size_t)n * f->R * sizeof(Entry), hipMemcpyDeviceToHost));
    if (counters_host)
        RL_HIP(hipMemcpy(counters_host, f->counter + li, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToHost));
    return RELOC_OK;
}

extern "C" int reloc_debug_modes(reloc_forest *f, int32_t t, int32_t leaf0, int32_t n, void *modes_host,
                                 int32_t *n_modes_host)
{
    if (!f || t < 0 || t >= f->T || leaf0 < 0 || n < 0 || leaf0 + n > f->L) return RELOC_E_ARG;
    int rc = update_modes(f, 0);
    if (rc) return rc;
    RL_HIP(hipDeviceSynchronize());
    int64_t li = (int64_t)t * f->L + leaf0;
    std::unique_ptr<int32_t[]> count(new (std::nothrow) int32_t[std::max(n, 1)]);
    if (!count) return RELOC_E_NOMEM;
    RL_HIP(hipMemcpy(count.get(), f->nmodes + li, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost));
    if (modes_host) {
        RL_HIP(hipMemcpy(modes_host, f->modes + li * f->M, (size_t)n * f->M * sizeof(Mode), hipMemcpyDeviceToHost));
        clear_unused_modes((Mode *)modes_host, count.get(), (size_t)n, f->M);
    }
    if (n_modes_host) memcpy(n_modes_host, count.get(), (size_t)n * sizeof(int32_t));
    return RELOC_OK;
}

extern "C" int reloc_debug_modes_from_points(reloc_forest *f, const void *entries_host, int32_t n, void *modes_host,
                                             int32_t *n_modes_host)
{
    if (!f || (!entries_host && n > 0) || !modes_host || !n_modes_host || n < 0 || n > MAX_R) return RELOC_E_ARG;
    Entry *d_pts = nullptr;
    Mode *d_modes = nullptr;
    int32_t *d_n = nullptr;
    RL_HIP(hipDeviceSynchronize());
    if (device_malloc((void **)&d_pts, (size_t)std::max(n, 1) * sizeof(Entry)) != hipSuccess) return RELOC_E_NOMEM;
    if (device_malloc((void **)&d_modes, (size_t)f->M * sizeof(Mode)) != hipSuccess ||
        device_malloc((void **)&d_n, sizeof(int32_t)) != hipSuccess) {
        (void)hipFree(d_pts);
        (void)hipFree(d_modes);
        return RELOC_E_NOMEM;
    }
    int rc = RELOC_OK;
    if (n > 0 && hipMemcpy(d_pts, entries_host, (size_t)n * sizeof(Entry), hipMemcpyHostToDevice) != hipSuccess)
        rc = RELOC_E_HIP;
    if (!rc) {
        ModeParams mp = mode_params(f);
        RL_LAUNCH("k_modes_points", k_modes_points, dim3(1), dim3(MODE_THREADS), mode_smem(mp.M), 0, d_pts, (int)n, mp, d_modes,
                           d_n);
        if (hipDeviceSynchronize() != hipSuccess ||
            hipMemcpy(n_modes_host, d_n, sizeof(int32_t), hipMemcpyDeviceToHost) != hipSuccess ||
            hipMemcpy(modes_host, d_modes, (size_t)f->M * sizeof(Mode), hipMemcpyDeviceToHost) != hipSuccess)
            rc = RELOC_E_HIP;
    }
    (void)hipFree(d_pts);
    (void)hipFree(d_modes);
    (void)hipFree(d_n);
    return rc;
}
