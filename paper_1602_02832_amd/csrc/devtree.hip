// Step 1 of the tree/Hermite scheme on the device (Fukushige & Kawai,
// Section 2): Peano-Hilbert keys, the sorted particle order, the octree,
// node moments, groups and the interaction lists, computed from particles
// already resident in device memory.  The definitions are those of the host
// builder (include/htree_host.h), and the results are bit-identical to it:
// the same keys and order, the same node sums in the same order, the same
// opening test with the same roundings, the same lists in the same order.
//
// Layout of the work (one stream, synchronous entry point):
//   1. root cube from a min/max reduction; 63-bit keys; stable radix sort of
//      (key, index) pairs; the particle state gathered into key order.
//   2. the octree without a pointer walk.  With L_k the first level at which
//      particle k's key leaves particle k-1's cell, the cells that begin at
//      particle k are those of levels L_k ... E_k, and pre-order is the order
//      of (first particle, level).  Per-particle counts and their prefix sums,
//      made where the state is gathered, give every cell, node and group its
//      pre-order number directly.
//   3. node moments, bottom-up in one launch: four lanes to a node add its
//      children's sums (or a leaf's particles) in order, small subtrees within
//      a work-group; above them the last child of a node to be done goes on
//      with the node.
//   4. lists: one work-group per group goes down the tree a level at a time,
//      visiting every cell once; the counts of list entries under each opened
//      cell are then summed upwards and the entries placed on the way down
//      again, so that the list comes out in pre-order.
// A rebuild queues all of it at once for what the arrays of the build before it
// hold, and looks at the counts at the end.
#include "htree_tree.h"
#include "wave_ops.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <cmath>
#include <string>

#include <rocprim/device/device_radix_sort.hpp>

namespace {

constexpr int kAxisBits = 21;      // bits per axis of the key
constexpr int kDeepest = 21;       // deepest cell level
constexpr int kNoCellLevel = 22;   // L_k of a particle whose key equals its predecessor's
constexpr int kWG = 256;
constexpr int kListWG = 512;
constexpr int64_t kMaxN = int64_t(1) << 26;   // every cell count fits in int32 (<= 22 N)

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HTD_HIP(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess) return fail(HTD_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

struct Cell {
    int32_t begin, end;   // particle range [begin, end) in key order
    int32_t skip;         // first cell after this cell's subtree (pre-order)
    int32_t node;         // node number, -1 for a single-particle cell
    int32_t level;
    int32_t split;        // 1 if the cell has children
    int32_t pad0, pad1;
};
static_assert(sizeof(Cell) == 32, "cell record");

struct Totals {
    int32_t cells, nodes, groups, pad;
};

struct Caps {             // what the arrays of cells and nodes hold
    int64_t cells, nodes;
};
__device__ inline bool fits(const Totals* t, const Caps& c) { return t->cells <= c.cells && t->nodes <= c.nodes; }

struct Counters {         // list phase
    unsigned long long staged;   // entries reserved in the staging array
    int32_t max_cut;             // most opened cells that did not fit a work-group's scratch
    int32_t taken;               // groups that work-groups have gone on with after their first
};

struct Root {
    double lo[3];
    double side;
    double scale;    // 2^21 / side
};

// A build's small state on the device: the tickets of the launches whose last
// work-group finishes their sums, and when each phase began.
constexpr int kStamps = 6;
struct Progress {
    Root root;
    Totals tot;
    Counters ctr;
    uint64_t stamp[kStamps];
    uint32_t bbox_done, counts_done, offsets_done, pad;
};
// What the host reads at the end of it (pinned memory).
struct Outcome {
    Root root;
    Totals tot;
    Counters ctr;
    uint64_t stamp[kStamps];
};

// True, in every thread, in the last of n_wgs work-groups to get here; what
// the others stored with agent-scope stores before can then be read with
// agent-scope loads.  The ticket is 0 again after the last one.
__device__ inline bool last_here(uint32_t* ticket, uint32_t n_wgs) {
    __shared__ uint32_t s_ticket;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores are where every XCD sees them
    __syncthreads();
    if (threadIdx.x == 0)
        s_ticket = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const bool last = s_ticket == n_wgs - 1;
    if (last && threadIdx.x == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::: "memory");
    return last;
}
template <class V>
__device__ inline void put_agent(V* p, V v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <class V>
__device__ inline V get_agent(const V* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Exclusive prefix sum over a work-group of WG threads, and its total.
template <int WG, class V>
__device__ inline V scan_group(V x, V* total) {
    __shared__ V s_wave[WG / 64];
    const V in = wave_ops::scan_inclusive(x);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63) s_wave[wave] = in;
    __syncthreads();
    V before = 0, sum = 0;
    for (int w = 0; w < WG / 64; ++w) {
        if (w == wave) before = sum;
        sum += s_wave[w];
    }
    __syncthreads();   // s_wave may be written again
    *total = sum;
    return before + in - x;
}

// ---------------------------------------------------------------- keys
__device__ inline uint64_t spread3(uint32_t v) {
    uint64_t s = v & 0x1fffffu;
    s = (s | s << 32) & 0x1f00000000ffffull;
    s = (s | s << 16) & 0x1f0000ff0000ffull;
    s = (s | s << 8) & 0x100f00f00f00f00full;
    s = (s | s << 4) & 0x10c30c30c30c30c3ull;
    s = (s | s << 2) & 0x1249249249249249ull;
    return s;
}

// Peano-Hilbert index of a lattice point (J. Skilling, "Programming the
// Hilbert curve", AIP Conf. Proc. 707, 2004): axes to transposed index, then
// the bits interleaved from the top with x first.
__device__ inline uint64_t ph_key(uint32_t x, uint32_t y, uint32_t z) {
    uint32_t c0 = x, c1 = y, c2 = z;
    for (uint32_t q = 1u << (kAxisBits - 1); q > 1; q >>= 1) {
        const uint32_t low = q - 1;
        {   // axis 0: invert or leave
            const uint32_t set = 0u - static_cast<uint32_t>((c0 & q) != 0);
            c0 ^= low & set;
        }
        {
            const uint32_t set = 0u - static_cast<uint32_t>((c1 & q) != 0);
            const uint32_t swap = (c0 ^ c1) & low & ~set;
            c0 ^= (low & set) | swap;
            c1 ^= swap;
        }
        {
            const uint32_t set = 0u - static_cast<uint32_t>((c2 & q) != 0);
            const uint32_t swap = (c0 ^ c2) & low & ~set;
            c0 ^= (low & set) | swap;
            c2 ^= swap;
        }
    }
    c1 ^= c0;
    c2 ^= c1;
    uint32_t flip = 0;
    for (uint32_t q = 1u << (kAxisBits - 1); q > 1; q >>= 1) flip ^= (q - 1) & (0u - static_cast<uint32_t>((c2 & q) != 0));
    c0 ^= flip;
    c1 ^= flip;
    c2 ^= flip;
    return (spread3(c0) << 2) | (spread3(c1) << 1) | spread3(c2);
}

__device__ inline double dmin(double a, double b) { return b < a ? b : a; }
__device__ inline double dmax(double a, double b) { return a < b ? b : a; }

// Componentwise min and max over a work-group (exact in any order), in thread 0.
template <int WG>
__device__ inline void box_of_group(double* lo, double* hi) {
    __shared__ double s_box[6][WG / 64];
    for (int d = 0; d < 3; ++d) {
        lo[d] = wave_ops::tree<32, 1>(lo[d], [](double p, double q) { return dmin(p, q); });
        hi[d] = wave_ops::tree<32, 1>(hi[d], [](double p, double q) { return dmax(p, q); });
    }
    if ((threadIdx.x & 63) == 0)
        for (int d = 0; d < 3; ++d) {
            s_box[d][threadIdx.x >> 6] = lo[d];
            s_box[3 + d][threadIdx.x >> 6] = hi[d];
        }
    __syncthreads();
    for (int d = 0; d < 3; ++d) {
        lo[d] = s_box[d][0];
        hi[d] = s_box[3 + d][0];
        for (int w = 1; w < WG / 64; ++w) {
            lo[d] = dmin(lo[d], s_box[d][w]);
            hi[d] = dmax(hi[d], s_box[3 + d][w]);
        }
    }
    __syncthreads();
}

// The root cube: side is the smallest power of two above the largest extent (1
// when all particles coincide).  Every work-group's box goes to part; the last
// one to be done reduces them.
constexpr int kBoxWGs = 512;   // at most: 12 ns a ticket
__global__ __launch_bounds__(kWG) void bbox_kernel(int64_t n, const double* __restrict__ x, double* part,
                                                   Progress* pr) {
    if (blockIdx.x == 0 && threadIdx.x == 0) pr->stamp[0] = wall_clock64();
    double lo[3], hi[3];
    for (int d = 0; d < 3; ++d) lo[d] = hi[d] = x[d];
#pragma unroll 4
    for (int64_t i = blockIdx.x * int64_t(kWG) + threadIdx.x; i < n; i += int64_t(gridDim.x) * kWG)
        for (int d = 0; d < 3; ++d) {
            lo[d] = dmin(lo[d], x[3 * i + d]);
            hi[d] = dmax(hi[d], x[3 * i + d]);
        }
    box_of_group<kWG>(lo, hi);
    if (threadIdx.x == 0)
        for (int d = 0; d < 3; ++d) {
            put_agent(part + 6 * blockIdx.x + d, lo[d]);
            put_agent(part + 6 * blockIdx.x + 3 + d, hi[d]);
        }
    if (!last_here(&pr->bbox_done, gridDim.x)) return;
    for (uint32_t b = threadIdx.x; b < gridDim.x; b += kWG)
        for (int d = 0; d < 3; ++d) {
            lo[d] = dmin(lo[d], get_agent(part + 6 * b + d));
            hi[d] = dmax(hi[d], get_agent(part + 6 * b + 3 + d));
        }
    box_of_group<kWG>(lo, hi);
    if (threadIdx.x != 0) return;
    const double ext = dmax(dmax(hi[0] - lo[0], hi[1] - lo[1]), hi[2] - lo[2]);
    double side = 1.0;
    if (ext > 0.0) {
        int e;
        frexp(ext, &e);
        side = ldexp(1.0, e);
    }
    for (int d = 0; d < 3; ++d) pr->root.lo[d] = lo[d];
    pr->root.side = side;
    pr->root.scale = ldexp(1.0, kAxisBits) / side;
}

__device__ inline uint64_t key_of(const double* __restrict__ x, int64_t i, const Root& root) {
    const double qmax = ldexp(1.0, kAxisBits) - 1.0;
    uint32_t q[3];
    for (int d = 0; d < 3; ++d) {
        double u = floor((x[3 * i + d] - root.lo[d]) * root.scale);
        u = dmin(dmax(u, 0.0), qmax);
        q[d] = static_cast<uint32_t>(u);
    }
    return ph_key(q[0], q[1], q[2]);
}

__global__ __launch_bounds__(kWG) void keys_kernel(int64_t n, const double* __restrict__ x, Progress* pr,
                                                   uint64_t* __restrict__ key, int32_t* __restrict__ idx) {
    const int64_t i = blockIdx.x * int64_t(kWG) + threadIdx.x;
    if (i >= n) return;
    key[i] = key_of(x, i, pr->root);
    idx[i] = static_cast<int32_t>(i);
    if (i == n - 1) {
        pr->ctr = Counters{0, 0, 0};
        pr->stamp[1] = wall_clock64();   // the sort follows
    }
}

// Up to kRankSort particles the keys are sorted, stably, by counting for each
// how many come before it, in two launches: runs of kRun keys in LDS as they
// are made, then every key's place among the other runs.  The library's sort
// takes five launches or more at these sizes, each waiting for the last.  Keys
// and sort, at 1024, 5000, 20011 and 32768 particles: 18, 19, 22 and 24 us
// against 17, 35, 46 and 46 us.  The work grows with n^2 / kRun, and above 64
// runs a wave has a second turn: at 50000, 58 us against 50 us.
constexpr int kRun = 512, kPiece = 128;
constexpr int64_t kRankSort = 64 * kRun;

// How many of the len keys of a sorted stretch come before key: those below
// it, and its equals if the stretch lies before it.  At N stretches at once,
// whose accesses do not depend on each other.
template <int MOST, int N, class At>
__device__ __forceinline__ void places(uint64_t key, const bool* before, const int* len, int* pos, At at) {
#pragma unroll
    for (int u = 0; u < N; ++u) pos[u] = 0;
    for (int step = MOST; step > 0; step >>= 1) {
        bool in[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int p = pos[u] + step;
            const uint64_t k = at(u, max(min(p, len[u]) - 1, 0));
            in[u] = p <= len[u] && (k < key || (before[u] && k == key));
        }
#pragma unroll
        for (int u = 0; u < N; ++u) pos[u] += in[u] ? step : 0;
    }
}

__global__ __launch_bounds__(kRun) void key_runs_kernel(int64_t n, const double* __restrict__ x, Progress* pr,
                                                        uint64_t* __restrict__ key, int32_t* __restrict__ idx) {
    __shared__ uint64_t s_key[2][kRun];
    __shared__ uint16_t s_from[2][kRun];
    const int t = threadIdx.x, lane = t & 63, piece = t / kPiece;
    const int64_t first = blockIdx.x * int64_t(kRun), i = first + t;
    if (i == 0) {
        pr->ctr = Counters{0, 0, 0};
        pr->stamp[1] = wall_clock64();
    }
    uint64_t mine = i < n ? key_of(x, i, pr->root) : uint64_t(1) << 63;   // above every key
    s_key[0][t] = mine;
    __syncthreads();
    {   // the place in the piece, by comparing with all of it
        const uint64_t* k = s_key[0] + piece * kPiece;
        const int own = t & (kPiece - 1) & ~63;   // the wave's own keys; equals before it count, behind it not
        int r = 0;
#pragma unroll 8
        for (int j = 0; j < own; ++j) r += k[j] <= mine;
#pragma unroll 8
        for (int j = 0; j < 64; ++j) r += k[own + j] < mine + (j < lane);
#pragma unroll 8
        for (int j = own + 64; j < kPiece; ++j) r += k[j] < mine;
        s_key[1][piece * kPiece + r] = mine;
        s_from[1][piece * kPiece + r] = static_cast<uint16_t>(t);
    }
    __syncthreads();
    {   // the place in the run, by searching the other pieces
        constexpr int N = kRun / kPiece;
        mine = s_key[1][t];
        const uint16_t from = s_from[1][t];
        bool before[N];
        int len[N], pos[N], r = 0;
        for (int u = 0; u < N; ++u) {
            before[u] = u < piece;
            len[u] = kPiece;
        }
        places<kPiece, N>(mine, before, len, pos, [&](int u, int k) { return s_key[1][u * kPiece + k]; });
        for (int u = 0; u < N; ++u) r += u == piece ? t & (kPiece - 1) : pos[u];
        s_key[0][r] = mine;
        s_from[0][r] = from;
    }
    __syncthreads();
    if (i < n) {
        key[i] = s_key[0][t];
        idx[i] = static_cast<int32_t>(first) + s_from[0][t];
    }
}

// A work-group places 64 keys, which are of one run; its waves share the runs.
// Every kStep-th key of every run is in LDS, so that a search goes to memory
// for the kStep keys at its end only.
constexpr int kMergeWG = 512, kStep = 32;
__global__ __launch_bounds__(kMergeWG) void merge_runs_kernel(int n, const uint64_t* __restrict__ runs,
                                                              const int32_t* __restrict__ run_idx,
                                                              uint64_t* __restrict__ key, int32_t* __restrict__ idx) {
    constexpr int N = 8, kWaves = kMergeWG / 64;
    __shared__ uint64_t s_step[kRankSort / kStep];
    __shared__ int s_place[kWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane, own = blockIdx.x * 64 / kRun, count = (n + kRun - 1) / kRun;
    const uint64_t mine = runs[min(i, n - 1)];
    for (int k = threadIdx.x; k < n / kStep; k += kMergeWG) s_step[k] = runs[k * kStep + kStep - 1];
    __syncthreads();
    int place = 0;
    for (int r0 = wave * N; r0 < count; r0 += kWaves * N) {
        bool before[N];
        int first[N], len[N], steps[N], pos[N];
        for (int u = 0; u < N; ++u) {
            const int run = min(r0 + u, count - 1);
            before[u] = run < own;
            first[u] = run * kRun;
            len[u] = min(kRun, n - first[u]);
            steps[u] = len[u] / kStep;
        }
        places<kRun / kStep, N>(mine, before, steps, pos,
                                [&](int u, int k) { return s_step[first[u] / kStep + k]; });
        for (int u = 0; u < N; ++u) {
            pos[u] *= kStep;
            first[u] += pos[u];
            len[u] = min(kStep, len[u] - pos[u]);
            steps[u] = pos[u];
        }
        places<kStep / 2, N>(mine, before, len, pos, [&](int u, int k) { return runs[min(first[u] + k, n - 1)]; });
        for (int u = 0; u < N; ++u)
            if (r0 + u < count) place += r0 + u == own ? i - own * kRun : steps[u] + pos[u];
    }
    s_place[wave][lane] = place;
    __syncthreads();
    if (wave != 0 || i >= n) return;
    for (int w = 1; w < kWaves; ++w) place += s_place[w][lane];
    key[place] = mine;
    idx[place] = run_idx[i];
}

__device__ inline uint64_t level_mask(int level) {
    const int sh = 3 * (kDeepest - level);
    return sh >= 63 ? 0ull : (~0ull << sh);
}

// The first level at which two keys of the sorted order part, the least of the
// levels at which neighbours part between them.
__device__ inline int parting(uint64_t a, uint64_t b) {
    const uint64_t diff = a ^ b;
    // digit i (0-based from the top) holds bits 60-3i .. 62-3i; the keys part at level i+1
    return diff == 0 ? kNoCellLevel : kDeepest - (63 - __clzll(diff)) / 3;
}

// How many of 0 ... top - 1 are `in`; those that are come first, and the first
// `have` are known to be.  Steps outwards from the near end in growing strides
// and narrows the bracket then, several accesses at a time, since each round
// waits for the last: most cells are small, and what is looked at lies near
// together.
template <class In>
__device__ inline int64_t extent(int64_t have, int64_t top, In in) {
    int64_t l = have, r = top;   // l are in, at most r are
    for (int64_t step = max(have, int64_t(1)); l < r; step *= 16) {
        int64_t p[4];
        bool ok[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            p[j] = min(l + step * ((2 << j) - 1), r);
            ok[j] = in(p[j] - 1);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (ok[j]) l = p[j];
            else r = min(r, p[j] - 1);
        }
        if (!ok[3]) break;
    }
    while (l < r) {
        const int64_t w = (r - l + 7) / 8, l0 = l, r0 = r;
        bool ok[7];
#pragma unroll
        for (int j = 0; j < 7; ++j) ok[j] = in(min(l0 + (j + 1) * w, r0) - 1);
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const int64_t p = min(l0 + (j + 1) * w, r0);
            if (ok[j]) l = p;
            else r = min(r, p - 1);
        }
    }
    return l;
}

// Counts over the kScanWG particles of a work-group, in one word: cells in the
// low 16 bits, nodes in the next 16, groups in the 16 above.  A particle's word
// holds the sums over the particles before it in the work-group, and above
// them its level L_k (6 bits), its cells (6) and whether a group begins (1).
constexpr int kScanWG = 512;
static_assert(kScanWG * (kDeepest + 1) < 1 << 16, "the counts of a work-group fit their fields");
__device__ inline int32_t cells_in(uint64_t w) { return static_cast<int32_t>(w & 0xffff); }
__device__ inline int32_t nodes_in(uint64_t w) { return static_cast<int32_t>((w >> 16) & 0xffff); }
__device__ inline int32_t groups_in(uint64_t w) { return static_cast<int32_t>((w >> 32) & 0xffff); }

// Particle state in key order; the cells, nodes and the group that begin at
// each particle, their sums over the particles before it in the work-group,
// and (by the last work-group to be done) the sums before every work-group.
// The gather of 104 bytes a particle from random places bounds it, and hides
// part of the counting.  At 2^20 and 20011 particles 143 and 15 us; a gather, a
// count that searched all n keys for the cell above, three scans and a kernel
// for their totals, nine launches, took 206 and 45 us.
__global__ __launch_bounds__(kScanWG) void particles_kernel(
    int64_t n, int n_leaf, int n_crit, const int32_t* __restrict__ perm32, const uint64_t* __restrict__ key,
    const double* __restrict__ x, const double* __restrict__ v, const double* __restrict__ a,
    const double* __restrict__ j, const double* __restrict__ m, int64_t* __restrict__ perm, double* __restrict__ sx,
    double* __restrict__ sv, double* __restrict__ sa, double* __restrict__ sj, double* __restrict__ sm,
    uint64_t* __restrict__ word, uint64_t* part, Totals* __restrict__ base, Progress* pr, Outcome* out) {
    if (blockIdx.x == 0 && threadIdx.x == 0) pr->stamp[2] = wall_clock64();
    const int64_t k = blockIdx.x * int64_t(kScanWG) + threadIdx.x;
    int L = 0;
    uint64_t count = 0, rest = 0;
    if (k < n) {
        const int64_t o = perm32[k];
        const uint64_t mine = key[k];
        if (k > 0) L = parting(mine, key[k - 1]);
        bool begins = L <= kDeepest, group = k == 0;
        if (begins && k > 0) {
            // the cell above: its particles from here on and before, as far as the answers need them
            const uint64_t mask = level_mask(L - 1), lo = mine & mask, hi = lo | (~mask & 0x7fffffffffffffffull);
            const int64_t far = max(int64_t(n_leaf), int64_t(n_crit)) + 1;
            int64_t above = extent(1, min(n - k, far), [&](int64_t i) { return key[k + i] <= hi; });
            if (above < far) above += extent(1, min(k, far), [&](int64_t i) { return key[k - 1 - i] >= lo; });
            begins = above > n_leaf;   // no cells in a leaf of up to n_leaf particles
            group = above > n_crit;    // no groups in a cell that is one, or in one
        }
        if (begins) {
            // levels L ... E: down to the last with more than n_leaf particles, and their children
            const int E = max(L, k + n_leaf >= n ? 0 : min(kDeepest, parting(mine, key[k + n_leaf])));
            const int nodes = k + 1 < n ? max(0, min(E, parting(mine, key[k + 1]) - 1) - L + 1) : 0;
            const uint64_t cells = E - L + 1;
            count = cells | static_cast<uint64_t>(nodes) << 16 | static_cast<uint64_t>(group) << 32;
            rest = static_cast<uint64_t>(L) << 48 | cells << 54 | static_cast<uint64_t>(group) << 60;
        }
        perm[k] = o;
        sm[k] = m[o];
        for (int d = 0; d < 3; ++d) {
            sx[3 * k + d] = x[3 * o + d];
            sv[3 * k + d] = v[3 * o + d];
            sa[3 * k + d] = a[3 * o + d];
            sj[3 * k + d] = j[3 * o + d];
        }
    }
    uint64_t sum;
    const uint64_t before = scan_group<kScanWG>(count, &sum);
    if (k < n) word[k] = before | rest;
    if (threadIdx.x == 0) put_agent(part + blockIdx.x, sum);
    if (!last_here(&pr->counts_done, gridDim.x)) return;
    int32_t at[3] = {0, 0, 0};
    for (uint32_t w = 0; w < gridDim.x; w += kScanWG) {
        const uint32_t i = w + threadIdx.x;
        const uint64_t c = i < gridDim.x ? get_agent(part + i) : 0;
        const int32_t here[3] = {cells_in(c), nodes_in(c), groups_in(c)};
        int32_t off[3];
        for (int q = 0; q < 3; ++q) {
            int32_t all;
            off[q] = at[q] + scan_group<kScanWG>(here[q], &all);
            at[q] += all;
        }
        if (i < gridDim.x) base[i] = Totals{off[0], off[1], off[2], 0};
    }
    if (threadIdx.x == 0) {
        const Totals tot{at[0], at[1], at[2], 0};
        pr->tot = tot;
        out->tot = tot;
        out->root = pr->root;
    }
}

// The cells and nodes that begin at each particle, from the deepest up: a
// cell's end lies past the one below it, a few times its size away at most
// where it has siblings.  A work-group keeps kTile keys from its first particle
// on in LDS, which most cells end in.  At 2^20 particles 49 us, 61 us without
// the LDS, 99 us with a search of all keys for every cell; at 20011, 15 us with
// any (a chain of dependent accesses for the few large cells).
constexpr int kTile = 4 * kWG;
__global__ __launch_bounds__(kWG) void cells_kernel(int64_t n, int n_leaf, const uint64_t* __restrict__ key,
                                                    const uint64_t* __restrict__ word,
                                                    const Totals* __restrict__ base, Caps caps, const Progress* pr,
                                                    Cell* __restrict__ cell, int32_t* __restrict__ node_level,
                                                    int64_t* __restrict__ node_begin, int64_t* __restrict__ node_end,
                                                    int32_t* __restrict__ node_cell, int64_t* __restrict__ group_first) {
    __shared__ uint64_t s_key[kTile], s_word[kTile];
    const int64_t first = blockIdx.x * int64_t(kWG), k = first + threadIdx.x;
    const int64_t ahead = min(int64_t(kTile), n - first);
    for (int64_t i = threadIdx.x; i < ahead; i += kWG) {
        s_key[i] = key[first + i];
        s_word[i] = word[first + i];
    }
    __syncthreads();
    if (k >= n || !fits(&pr->tot, caps)) return;
    if (k == 0) group_first[pr->tot.groups] = n;
    const uint64_t w = s_word[threadIdx.x];
    const int cells = static_cast<int>((w >> 54) & 63), L = static_cast<int>((w >> 48) & 63);
    if (cells == 0) return;
    const Totals b = base[k / kScanWG];
    if ((w >> 60) & 1) group_first[b.groups + groups_in(w)] = k;
    const int32_t c0 = b.cells + cells_in(w), q0 = b.nodes + nodes_in(w);
    const uint64_t mine = s_key[threadIdx.x];
    const int64_t near = ahead - threadIdx.x;
    int64_t cnt = 1;
    for (int l = L + cells - 1; l >= L; --l) {
        const uint64_t hi = mine | ~(level_mask(l) | ~0x7fffffffffffffffull);
        if (l == 0) cnt = n - k;
        else if (cnt < near) cnt = extent(cnt, near, [&](int64_t i) { return s_key[threadIdx.x + i] <= hi; });
        if (cnt >= near && cnt < n - k) cnt = extent(cnt, n - k, [&](int64_t i) { return key[k + i] <= hi; });
        const int64_t e = k + cnt;
        Cell c;
        c.begin = static_cast<int32_t>(k);
        c.end = static_cast<int32_t>(e);
        c.skip = e < n ? base[e / kScanWG].cells + cells_in(cnt < near ? s_word[threadIdx.x + cnt] : word[e])
                       : pr->tot.cells;
        c.node = cnt >= 2 ? q0 + (l - L) : -1;
        c.level = l;
        c.split = (cnt > n_leaf && l < kDeepest) ? 1 : 0;
        c.pad0 = c.pad1 = 0;
        cell[c0 + (l - L)] = c;
        if (c.node >= 0) {
            node_level[c.node] = l;
            node_begin[c.node] = k;
            node_end[c.node] = e;
            node_cell[c.node] = c0 + (l - L);
        }
    }
}

// What the list walk needs to know about a node, in one 64-byte record: its
// centre of mass, particle range, level and children (a single-particle child
// as its particle index, a child node q as ~q, kNone past the last), so that
// visiting a node is one access and opening it follows no chain of cells.
struct alignas(32) NodeTest {
    double x[3];
    uint32_t begin_level;   // first particle (26 bits), level above it
    uint32_t end;
};
struct alignas(64) NodeRec : NodeTest {
    int32_t kid[8];
};
constexpr int32_t kNone = INT32_MIN;
constexpr int kBeginBits = 26;
static_assert(sizeof(NodeTest) == 32 && sizeof(NodeRec) == 64, "node record");
static_assert(kMaxN <= int64_t(1) << kBeginBits && kDeepest < 32, "begin and level share a word");

__device__ inline int32_t first_of(const NodeTest& r) {
    return static_cast<int32_t>(r.begin_level & ((1u << kBeginBits) - 1));
}
__device__ inline int32_t size_of(const NodeTest& r) { return static_cast<int32_t>(r.end) - first_of(r); }
__device__ inline bool is_node(int32_t kid) { return kid < 0 && kid != kNone; }

// Every node's range, level and children (its centre of mass follows the moments).
__global__ __launch_bounds__(kWG) void node_recs_kernel(Caps caps, Progress* pr,
                                                        const int32_t* __restrict__ node_cell, const Cell* __restrict__ cell, NodeRec* __restrict__ rec,
                                                        int32_t* __restrict__ parent, int32_t* __restrict__ arrived) {
    const int32_t q = blockIdx.x * kWG + threadIdx.x;
    if (q == 0) pr->stamp[3] = wall_clock64();
    if (q >= pr->tot.nodes || !fits(&pr->tot, caps)) return;
    const int32_t ci = node_cell[q];
    const Cell c = cell[ci];
    NodeRec r;
    for (int d = 0; d < 3; ++d) r.x[d] = 0.0;
    r.begin_level = static_cast<uint32_t>(c.begin) | static_cast<uint32_t>(c.level) << kBeginBits;
    r.end = static_cast<uint32_t>(c.end);
    int32_t ch = c.split ? ci + 1 : c.skip, below = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {   // a cell has at most eight children
        r.kid[k] = kNone;
        if (ch < c.skip) {
            const Cell cc = cell[ch];
            r.kid[k] = cc.node >= 0 ? ~cc.node : cc.begin;
            if (cc.node >= 0) {
                parent[cc.node] = q;
                ++below;
            }
            ch = cc.skip;
        }
    }
    rec[q] = r;
    arrived[q] = -below;   // the last node child to be done gets -1
    if (q == 0) parent[0] = -1;
}

// Node moments, bottom-up, as the host builder defines them: a node's sums
// S = (m, m x[3], m v[3], m a[3], m jerk[3]) start from zero and add, for a
// split node, its children's S in key order (a single-particle child's S is
// 0 + its rounded products), otherwise its particles' rounded products in
// ascending order; the means are the sums divided by the mass.  No fused
// multiply-add anywhere, so the bits match.  raw holds S, 13 doubles per node.
//
// Four lanes (a DPP quad) to a node, one for each vector; every one sums the
// mass as well.  A work-group takes about kStride nodes in pre-order.  The
// nodes whose whole subtree is among them, most, are summed in it: every quad
// loads its node's single particles at once and then waits in LDS for the sums
// of its node children.  The others are the ancestors of the next work-group's
// first node, which is chosen as the shallowest of 2 kSlack: they are summed
// by whichever quad, of any work-group, finishes the last of their children
// and so takes the last ticket.  Their children's sums go through to where
// every XCD sees them (agent-scope stores and loads, which pass the L2s that
// are not coherent with each other), and the ticket is taken once they are
// there: about 3 us a level, which bounds the small sizes.  At 2^20 and 20011
// particles one launch per level from the deepest up took 336 and 124 us, with
// 28 and 4 us for the means after them; all sums through memory with sixteen
// lanes to a node, 250 and 40 us, with four, 270 and 51 us; this, 183 and 41 us
// (work-groups of 512 and 1024 threads: 193 and 233 us at 2^20).
#pragma clang fp contract(off)
struct NodeOut {
    double *m, *x, *v, *a, *j;
};
constexpr int kSumWG = 256;
constexpr int kQuads = kSumWG / 4;                // nodes that a work-group holds
constexpr int kSlack = 8;
constexpr int kStride = kQuads - 2 * kSlack;
static_assert(2 * kSlack <= 32, "half a wave looks at the places for a cut");

// A node's children's contributions: the single particles' as loaded, the node
// children's from where their sums are.
struct Kids {
    int32_t kid[8];
    double m[8], f[8][3];

    __device__ __forceinline__ void load(const NodeRec* rec, int32_t q) {
#pragma unroll
        for (int c = 0; c < 8; ++c) kid[c] = rec[q].kid[c];
    }
    __device__ __forceinline__ void load_particles(const double* sm, const double* src) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            m[c] = f[c][0] = f[c][1] = f[c][2] = 0.0;
            if (kid[c] < 0) continue;
            m[c] = sm[kid[c]];
            for (int d = 0; d < 3; ++d) f[c][d] = src[3 * int64_t(kid[c]) + d];
        }
    }
    // node_sum(q, k): sum k of node q, k = 0 the mass
    template <class Sum>
    __device__ __forceinline__ void add(double* M, double* s, Sum node_sum) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (!is_node(kid[c])) continue;
            m[c] = node_sum(~kid[c], 0);
            for (int d = 0; d < 3; ++d) f[c][d] = node_sum(~kid[c], 1 + d);
        }
        *M = s[0] = s[1] = s[2] = 0.0;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (kid[c] == kNone) continue;
            const bool node = is_node(kid[c]);
            *M = *M + (node ? m[c] : 0.0 + m[c]);
            for (int d = 0; d < 3; ++d) s[d] = s[d] + (node ? f[c][d] : 0.0 + m[c] * f[c][d]);
        }
    }
};

__global__ __launch_bounds__(kSumWG) void node_sums_kernel(Caps caps, const Progress* pr,
                                                           const int32_t* __restrict__ parent, int32_t* arrived,
                                                           const double* __restrict__ sm,
                                                           const double* __restrict__ sx, const double* __restrict__ sv,
                                                           const double* __restrict__ sa, const double* __restrict__ sj,
                                                           double* raw, NodeRec* rec, NodeOut o) {
    __shared__ int32_t s_left[kQuads];   // node children still to be summed, or kNone: not in this work-group
    __shared__ double s_sum[kQuads][13];
    const int32_t nodes = pr->tot.nodes;
    if (!fits(&pr->tot, caps) || blockIdx.x * int64_t(kStride) >= nodes) return;
    const int lane = threadIdx.x & 63, r = threadIdx.x & 3;
    // cuts: lanes 0-31 look at the places for this work-group's first node, the others for the next's
    const int64_t mark = (blockIdx.x + int64_t(lane >> 5)) * kStride;
    int64_t at = mark - kSlack + (lane & 31);
    const bool place = (lane & 31) < 2 * kSlack && at >= 0 && at < nodes;
    int best = place ? static_cast<int>(rec[at].begin_level >> kBeginBits) * 32 + (lane & 31) : INT32_MAX;
    for (int w = 16; w > 0; w >>= 1) best = min(best, __shfl_xor(best, w));
    const int32_t cut = static_cast<int32_t>(mark <= 0 ? 0 : mark >= nodes ? nodes : mark - kSlack + (best & 31));
    const int32_t q0 = wave_ops::read_lane(cut, 0), q1 = wave_ops::read_lane(cut, 32);
    // a node's subtree follows it: it ends before q1 if node q1 begins past the node's particles
    const int64_t beyond = q1 < nodes ? first_of(rec[q1]) : INT64_MAX;

    const int slot = threadIdx.x >> 2;
    int32_t q = q0 + slot;
    const bool on = q < q1;
    const double* src = r == 0 ? sx : r == 1 ? sv : r == 2 ? sa : sj;
    double* dst = r == 0 ? o.x : r == 1 ? o.v : r == 2 ? o.a : o.j;
    Kids K;
    double M = 0.0, s[3] = {0.0, 0.0, 0.0};
    int32_t p = -1;
    bool todo = false;
    if (on) {
        K.load(rec, q);
        p = parent[q];
        todo = static_cast<int64_t>(rec[q].end) <= beyond;
        int32_t below = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) below += is_node(K.kid[c]);
        if (r == 0) s_left[slot] = todo ? below : kNone;
    }
    const bool mine = todo, leaf = mine && K.kid[0] == kNone;
    if (leaf) {   // several particles
        const int64_t e = rec[q].end;
        for (int64_t k = first_of(rec[q]); k < e; ++k) {
            const double mk = sm[k];
            M = M + mk;
            for (int d = 0; d < 3; ++d) s[d] = s[d] + mk * src[3 * k + d];
        }
    } else if (mine) {
        K.load_particles(sm, src);
    }
    __syncthreads();
    const bool up_here = mine && p >= q0 && s_left[p - q0] != kNone;
    // Every turn sums the nodes whose children are done; a node's children are in this work-group,
    // and one without any needs none, so that each wave's last turn comes.
    while (__ballot(todo)) {
        if (todo && __hip_atomic_load(&s_left[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0) {
            asm volatile("" ::: "memory");
            if (!leaf) K.add(&M, s, [&](int32_t c, int k) { return s_sum[c - q0][k == 0 ? 0 : 3 * r + k]; });
            if (r == 0) s_sum[slot][0] = M;
            for (int d = 0; d < 3; ++d) s_sum[slot][1 + 3 * r + d] = s[d];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the sums are in LDS
            if (r == 0 && up_here)
                __hip_atomic_fetch_add(&s_left[p - q0], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            todo = false;
        }
    }
    if (!mine) return;   // summed by the last of its children
    for (;;) {
        const bool up = p >= 0 && !up_here;
        int32_t ticket = 0;
        Kids P;
        if (up) {
            double* S = raw + 13 * int64_t(q);
            if (r == 0) put_agent(S, M);
            for (int d = 0; d < 3; ++d) put_agent(S + 1 + 3 * r + d, s[d]);
            P.load(rec, p);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the sums are where every XCD sees them
            if (r == 0) ticket = __hip_atomic_fetch_add(arrived + p, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            P.load_particles(sm, src);
        }
        for (int d = 0; d < 3; ++d) {
            const double mean = s[d] / M;
            dst[3 * int64_t(q) + d] = mean;
            if (r == 0) rec[q].x[d] = mean;
        }
        if (r == 0) o.m[q] = M;
        if (!up || wave_ops::first_of_quad(ticket) != -1) return;   // nothing above, or a sibling is still on its way
        asm volatile("" ::: "memory");                              // the children's sums are read after the ticket
        P.add(&M, s, [&](int32_t c, int k) { return get_agent(raw + 13 * int64_t(c) + (k == 0 ? 0 : 3 * r + k)); });
        q = p;
        p = parent[q];
    }
}
#pragma clang fp contract(on)

// ---------------------------------------------------------------- lists
struct ListArgs {
    int64_t n;
    int32_t cut_cap;
    Caps caps;
    Progress* pr;
    const NodeRec* rec;
    const double* sx;
    const int64_t* group_first;
    int32_t* cut;             // per work-group: walk_words(cut_cap) int32
    int32_t* stage;
    int64_t stage_cap;
    int32_t* glen;
    int64_t* gstage;
    double theta2;
};

#pragma clang fp contract(off)
// The opening test of the host builder: accept a node iff side^2 < theta^2 d^2,
// d the distance from its centre of mass to the group's box; a node that
// overlaps the group never passes.
__device__ inline bool accepts(const ListArgs& A, const double* s2, const NodeTest& r, int64_t gb, int64_t ge,
                               const double* lo, const double* hi) {
    if (first_of(r) < ge && gb < static_cast<int64_t>(r.end)) return false;
    double gap[3];
    for (int d = 0; d < 3; ++d) {
        const double u = dmax(lo[d] - r.x[d], r.x[d] - hi[d]);
        gap[d] = dmax(u, 0.0);
    }
    const double d2 = (gap[0] * gap[0] + gap[1] * gap[1]) + gap[2] * gap[2];
    return s2[r.begin_level >> kBeginBits] < A.theta2 * d2;
}
#pragma clang fp contract(on)

// A group's walk: the opened cells level by level, each level in key order.
// onode: the node; ofirst: its first opened child (the opened children of a
// cell follow each other in the next level); okids: which children are opened
// (8 bits) and how many there are (0: a leaf of several particles); ocount:
// the list entries under it, later its place in the list.
struct Walk {
    int32_t *onode, *ofirst, *ocount;
    uint16_t* okids;
    int32_t cap;
};
constexpr int32_t kLdsOpened = 5600;   // 77 KB: two work-groups per CU
__host__ __device__ inline int64_t walk_words(int64_t cap) { return 3 * cap + (cap + 1) / 2; }

constexpr int kAhead = 2;                     // opened cells per eight lanes and round, their children in flight together
constexpr int kListWaves = kListWG / 64;
constexpr int kPerRound = kListWG / 8;        // opened cells that the work-group's lanes cover once

struct WalkShared {
    double s2[kDeepest + 1];
    int32_t open[kDeepest + 4];               // where each level's opened cells begin
    int32_t count[2][kAhead * kListWaves];    // opened cells by slot and wave, of this round and the last
    unsigned long long off;
};

// Visits the children of every opened cell of group [gb, ge) with box
// [lo, hi], eight lanes to a cell, and writes the group's list: down the
// levels, then the counts up, then the places down.  Returns false, with *need
// opened cells counted, if the walk does not fit w.
__device__ __forceinline__ bool walk_group(const ListArgs& A, int32_t g, int64_t gb, int64_t ge, const double* lo,
                                           const double* hi, const Walk& w, WalkShared& S, int32_t* need) {
    const int t = threadIdx.x, c = t & 7, lane = t & 63, wave = t >> 6;
    const uint64_t below = (1ull << lane) - 1ull, before8 = (1ull << (lane & 56)) - 1ull;
    if (t == 0) {
        w.onode[0] = 0;   // the root overlaps every group
        S.open[0] = 0;
        S.open[1] = 1;
    }
    __syncthreads();
    int levels = 0, round = 0;
    for (int32_t o0 = 0, o1 = 1; o0 < o1; ++levels) {
        int32_t fill = o1;
        for (int32_t s = o0; s < o1; s += kPerRound * kAhead, round ^= 1) {
            int32_t q[kAhead], kid[kAhead];
            NodeTest r[kAhead];
            uint64_t opened[kAhead], kids[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int32_t o = s + u * kPerRound + (t >> 3);
                q[u] = o < o1 ? w.onode[o] : -1;
                kid[u] = q[u] >= 0 ? A.rec[q[u]].kid[c] : kNone;
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (is_node(kid[u])) r[u] = A.rec[~kid[u]];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                opened[u] = __ballot(is_node(kid[u]) && !accepts(A, S.s2, r[u], gb, ge, lo, hi));
                kids[u] = __ballot(kid[u] != kNone);
                if (lane == 0) S.count[round][u * kListWaves + wave] = __popcll(opened[u]);
            }
            __syncthreads();
            int32_t at[kAhead];
            for (int u = 0; u < kAhead; ++u)
                for (int k = 0; k < kListWaves; ++k) {
                    if (k == wave) at[u] = fill;
                    fill += S.count[round][u * kListWaves + k];
                }
            if (fill > w.cap) continue;   // does not fit: the level is only counted
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (q[u] < 0) continue;
                if ((opened[u] >> lane) & 1) w.onode[at[u] + __popcll(opened[u] & below)] = ~kid[u];
                if (c != 0) continue;
                const int32_t o = s + u * kPerRound + (t >> 3);
                const uint32_t n = __popc(static_cast<uint32_t>(kids[u] >> lane) & 0xffu);
                w.ofirst[o] = at[u] + __popcll(opened[u] & before8);
                w.okids[o] = static_cast<uint16_t>((static_cast<uint32_t>(opened[u] >> lane) & 0xffu) | n << 8);
                if (n == 0) w.ocount[o] = size_of(A.rec[q[u]]);
            }
        }
        if (fill > w.cap) {
            *need = fill;
            return false;
        }
        o0 = o1;
        o1 = fill;
        if (t == 0) S.open[levels + 2] = fill;
        __syncthreads();
    }
    // up: entries under every opened cell
    for (int l = levels - 1; l >= 0; --l) {
        const int32_t o1 = S.open[l + 1];
        for (int32_t o = S.open[l] + t; o < o1; o += kListWG) {
            const uint32_t m = w.okids[o], n = m >> 8, k = __popc(m & 0xffu);
            if (n == 0) continue;   // a leaf: counted on the way down
            const int32_t f = w.ofirst[o];
            int32_t sum = static_cast<int32_t>(n - k);
            for (uint32_t i = 0; i < k; ++i) sum += w.ocount[f + i];
            w.ocount[o] = sum;
        }
        __syncthreads();
    }
    const int32_t len = w.ocount[0];
    __syncthreads();
    if (t == 0) {
        S.off = atomicAdd(&A.pr->ctr.staged, static_cast<unsigned long long>(len));
        w.ocount[0] = 0;
    }
    __syncthreads();
    const unsigned long long off = S.off;
    const bool fits = off + static_cast<unsigned long long>(len) <= static_cast<unsigned long long>(A.stage_cap);
    if (t == 0) {
        A.glen[g] = len;
        A.gstage[g] = fits ? static_cast<int64_t>(off) : -1;
    }
    if (!fits) return true;
    // down: the opened children's places in the list, and the entries
    int32_t* out = A.stage + off;
    for (int l = 0; l < levels; ++l) {
        const int32_t o1 = S.open[l + 1];
        for (int32_t s = S.open[l]; s < o1; s += kPerRound) {
            const int32_t o = s + (t >> 3);
            const bool on = o < o1;   // every lane takes part in the lane exchanges
            const int32_t q = on ? w.onode[o] : 0, kid = on ? A.rec[q].kid[c] : kNone;
            const uint32_t m = on ? w.okids[o] : 0u;
            const int32_t p0 = on ? w.ocount[o] : 0;
            const bool opened = (m >> c) & 1;
            const int32_t mine = on ? w.ofirst[o] + __popc(m & ((1u << c) - 1u)) : 0;
            const int32_t cnt = kid == kNone ? 0 : opened ? w.ocount[mine] : 1;
            int32_t x = cnt, y;   // inclusive prefix sum over the cell's eight lanes
            y = wave_ops::below_in_row<1>(x);
            x += c >= 1 ? y : 0;
            y = wave_ops::below_in_row<2>(x);
            x += c >= 2 ? y : 0;
            y = wave_ops::below_in_row<4>(x);
            x += c >= 4 ? y : 0;
            const int32_t p = p0 + x - cnt;
            if (opened) w.ocount[mine] = p;
            else if (kid != kNone) out[p] = kid < 0 ? static_cast<int32_t>(A.n) + ~kid : kid;
            if (on && m >> 8 == 0) {   // a leaf: its particles
                const NodeTest r = A.rec[q];
                for (int32_t k = c; k < size_of(r); k += 8) out[p0 + k] = first_of(r) + k;
            }
        }
        __syncthreads();
    }
    return true;
}

// One work-group per group.  The walk is bound by its chain of dependent
// accesses, a few per level: what it keeps is in LDS where it fits, in memory
// otherwise (a store and the load after the barrier cost about 1500 cycles
// there, under load).  Only opened cells are kept, a fifth of the visited
// ones, so that the lists of 2^20 particles (8700 entries in the mean, 15000
// at most) fit.  An earlier form kept the ordered cut itself in memory and
// moved every decided entry again in each of the up to 22 passes, with a chain
// of up to eight cells at every opened one: 1740 us at 2^20 particles, against
// 361 us with every work-group on its share of the groups, and 333 us with the
// groups handed out as work-groups become free.
__global__ __launch_bounds__(kListWG, 4) void lists_kernel(ListArgs A) {
    __shared__ int32_t s_onode[kLdsOpened], s_ofirst[kLdsOpened], s_ocount[kLdsOpened];
    __shared__ uint16_t s_okids[kLdsOpened];
    __shared__ WalkShared S;
    __shared__ double s_box[6][kListWaves];
    __shared__ int32_t s_next;
    const int t = threadIdx.x;
    const Totals tot = A.pr->tot;
    if (t == 0 && blockIdx.x == 0) A.pr->stamp[4] = wall_clock64();
    if (!fits(&tot, A.caps)) return;
    if (t <= kDeepest) {
        const double side = ldexp(A.pr->root.side, -t);
        S.s2[t] = side * side;
    }
    if (tot.nodes == 0) {   // a single particle
        if (t == 0 && blockIdx.x == 0) {
            const unsigned long long off = atomicAdd(&A.pr->ctr.staged, 1ull);
            if (off < static_cast<unsigned long long>(A.stage_cap)) A.stage[off] = 0;
            A.glen[0] = 1;
            A.gstage[0] = static_cast<int64_t>(off);
        }
        return;
    }
    for (int32_t g = blockIdx.x; g < tot.groups; g = s_next) {
        const int64_t gb = A.group_first[g], ge = A.group_first[g + 1];
        // group box: componentwise min and max of the members' positions
        double lo[3], hi[3];
        for (int d = 0; d < 3; ++d) lo[d] = hi[d] = A.sx[3 * gb + d];
        for (int64_t k = gb + t; k < ge; k += kListWG)
            for (int d = 0; d < 3; ++d) {
                lo[d] = dmin(lo[d], A.sx[3 * k + d]);
                hi[d] = dmax(hi[d], A.sx[3 * k + d]);
            }
        for (int d = 0; d < 3; ++d) {
            lo[d] = wave_ops::tree<32, 1>(lo[d], [](double p, double q) { return dmin(p, q); });
            hi[d] = wave_ops::tree<32, 1>(hi[d], [](double p, double q) { return dmax(p, q); });
        }
        if ((t & 63) == 0)
            for (int d = 0; d < 3; ++d) {
                s_box[d][t >> 6] = lo[d];
                s_box[3 + d][t >> 6] = hi[d];
            }
        __syncthreads();
        for (int d = 0; d < 3; ++d) {
            lo[d] = s_box[d][0];
            hi[d] = s_box[3 + d][0];
            for (int w = 1; w < kListWaves; ++w) {
                lo[d] = dmin(lo[d], s_box[d][w]);
                hi[d] = dmax(hi[d], s_box[3 + d][w]);
            }
        }
        int32_t need = 0;
        if (!walk_group(A, g, gb, ge, lo, hi, Walk{s_onode, s_ofirst, s_ocount, s_okids, kLdsOpened}, S, &need)) {
            __syncthreads();
            int32_t* m = A.cut + static_cast<int64_t>(blockIdx.x) * walk_words(A.cut_cap);
            const Walk w{m, m + A.cut_cap, m + 2 * static_cast<int64_t>(A.cut_cap),
                         reinterpret_cast<uint16_t*>(m + 3 * static_cast<int64_t>(A.cut_cap)), A.cut_cap};
            if (!walk_group(A, g, gb, ge, lo, hi, w, S, &need) && t == 0) {
                atomicMax(&A.pr->ctr.max_cut, need);
                A.glen[g] = 0;
                A.gstage[g] = -1;
            }
        }
        if (t == 0) s_next = static_cast<int32_t>(gridDim.x) + atomicAdd(&A.pr->ctr.taken, 1);
        __syncthreads();
    }
}

// Whether every list was walked and staged.
__device__ inline bool staged_all(const Progress* pr, const Caps& caps, int64_t stage_cap) {
    return fits(&pr->tot, caps) && pr->ctr.max_cut == 0 &&
           pr->ctr.staged <= static_cast<unsigned long long>(stage_cap);
}

// Where the lists begin: the sums of the lengths within each work-group's
// kOffWG groups, and by the last work-group to be done those before each
// work-group.  Also hands the build's outcome to the host.
constexpr int kOffWG = 1024;
__global__ __launch_bounds__(kOffWG) void offsets_kernel(Caps caps, int64_t stage_cap, Progress* pr,
                                                         const int32_t* __restrict__ glen, int64_t* __restrict__ local,
                                                         int64_t* part, int64_t* __restrict__ base, Outcome* out) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        out->ctr = pr->ctr;
        for (int i = 0; i < kStamps - 1; ++i) out->stamp[i] = pr->stamp[i];
        out->stamp[kStamps - 1] = wall_clock64();
    }
    const int32_t groups = pr->tot.groups, wgs = (groups + kOffWG - 1) / kOffWG;
    if (!staged_all(pr, caps, stage_cap)) return;
    // a work-group may have several turns: the grid is chosen before the groups are counted
    for (int32_t w = blockIdx.x; w < wgs; w += gridDim.x) {
        const int32_t g = w * kOffWG + threadIdx.x;
        int64_t sum;
        const int64_t off = scan_group<kOffWG>(g < groups ? int64_t(glen[g]) : 0, &sum);
        if (g < groups) local[g] = off;
        if (threadIdx.x == 0) put_agent(part + w, sum);
    }
    if (!last_here(&pr->offsets_done, gridDim.x)) return;
    int64_t at = 0;
    for (int32_t w = 0; w < wgs; w += kOffWG) {
        const int32_t i = w + threadIdx.x;
        int64_t all;
        const int64_t off = scan_group<kOffWG>(i < wgs ? get_agent(part + i) : int64_t(0), &all);
        if (i < wgs) base[i] = at + off;
        at += all;
    }
}

// CSR copy: group g's staged list to entries[list_off[g] ...].
__global__ __launch_bounds__(kWG) void csr_kernel(Caps caps, int64_t stage_cap, int64_t entries_cap,
                                                  const Progress* pr, const int32_t* __restrict__ glen,
                                                  const int64_t* __restrict__ local, const int64_t* __restrict__ base,
                                                  const int64_t* __restrict__ gstage,
                                                  const int32_t* __restrict__ stage, int64_t* __restrict__ list_off,
                                                  int32_t* __restrict__ entries) {
    const int64_t total = static_cast<int64_t>(pr->ctr.staged);
    if (!staged_all(pr, caps, stage_cap) || total > entries_cap) return;
    const int32_t groups = pr->tot.groups;
    if (blockIdx.x == 0 && threadIdx.x == 0) list_off[groups] = total;
    for (int32_t g = blockIdx.x; g < groups; g += gridDim.x) {
        const int64_t b = base[g / kOffWG] + local[g], len = glen[g], s = gstage[g];
        if (threadIdx.x == 0) list_off[g] = b;
        for (int64_t i = threadIdx.x; i < len; i += kWG) entries[b + i] = stage[s + i];
    }
}

template <class T>
struct DevBuf {
    T* p = nullptr;
    int64_t cap = 0;
    int grow(int64_t need) {
        if (need <= cap) return 0;
        if (p) (void)hipFree(p);
        p = nullptr;
        cap = 0;
        const int64_t want = need + need / 4 + 16;
        if (hipMalloc(&p, sizeof(T) * static_cast<size_t>(want)) != hipSuccess) {
            p = nullptr;
            return fail(HTD_ENOMEM, "device allocation of %lld bytes failed", (long long)(sizeof(T) * want));
        }
        cap = want;
        return 0;
    }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
        cap = 0;
    }
};

inline unsigned blocks_for(int64_t n, int wg) { return static_cast<unsigned>((n + wg - 1) / wg); }

}  // namespace

struct htd_tree {
    int device = 0;
    hipStream_t stream = nullptr;
    int64_t n_max = 0;
    // per particle
    DevBuf<uint64_t> key_in, key;
    DevBuf<int32_t> idx_in, idx;
    DevBuf<int64_t> perm;
    DevBuf<double> sx, sv, sa, sj, sm;
    DevBuf<uint64_t> word, cpart;   // per particle and per work-group: counts
    DevBuf<Totals> cbase;
    DevBuf<char> tmp;
    DevBuf<double> part;
    DevBuf<Progress> pr;
    Outcome* out = nullptr;         // pinned
    // cells and nodes
    DevBuf<Cell> cell;
    DevBuf<double> nm, nx, nv, na, nj;
    DevBuf<int32_t> nlev, ncid;   // per node: level, cell index
    DevBuf<double> nraw;            // per node: the 13 sums of its moments
    DevBuf<NodeRec> nrec;           // per node: what the list walk reads
    DevBuf<int32_t> npar, narr;     // per node: parent, children whose sums are done
    DevBuf<int64_t> nbeg, nend;
    // groups and lists
    DevBuf<int64_t> group_first, list_off, gstage, glocal, gpart, gbase;
    DevBuf<int32_t> glen, cut, stage, entries;
    int32_t cut_cap = 1 << 15;
    int n_list_wg = 512;
    // results of the last build
    int64_t n = 0, C = 0, M = 0, G = 0, L = 0;
    Root root_h{};
    hipEvent_t ev[2] = {};
    double tick_ms = 0;             // of the device's constant-rate counter
    float phase_ms[7] = {};
    bool built = false;
};

namespace {

// Temporary storage of the sort, sized before anything is queued (freeing a
// buffer a queued primitive still uses would be unsafe).
int reserve_tmp(htd_tree* t, int64_t n) {
    size_t a = 0;
    HTD_HIP(rocprim::radix_sort_pairs(nullptr, a, t->key_in.p, t->key.p, t->idx_in.p, t->idx.p,
                                      static_cast<size_t>(n), 0, 63, t->stream));
    return t->tmp.grow(static_cast<int64_t>(a));
}

int grow_particles(htd_tree* t, int64_t n) {
    int rc = 0;
    const int64_t scans = (n + kScanWG - 1) / kScanWG, offs = (n + kOffWG - 1) / kOffWG;
    if ((rc = t->key_in.grow(n)) || (rc = t->key.grow(n)) || (rc = t->idx_in.grow(n)) || (rc = t->idx.grow(n)) ||
        (rc = t->perm.grow(n)) || (rc = t->sx.grow(3 * n)) || (rc = t->sv.grow(3 * n)) || (rc = t->sa.grow(3 * n)) ||
        (rc = t->sj.grow(3 * n)) || (rc = t->sm.grow(n)) || (rc = t->word.grow(n)) || (rc = t->cpart.grow(scans)) ||
        (rc = t->cbase.grow(scans)) || (rc = t->part.grow(6 * kBoxWGs)) || (rc = t->group_first.grow(n + 1)) ||
        (rc = t->list_off.grow(n + 1)) || (rc = t->gstage.grow(n + 1)) || (rc = t->glocal.grow(n + 1)) ||
        (rc = t->gpart.grow(offs)) || (rc = t->gbase.grow(offs)) || (rc = t->glen.grow(n + 1)))
        return rc;
    return 0;
}

int grow_nodes(htd_tree* t, int64_t cells, int64_t nodes) {
    int rc = 0;
    const int64_t M1 = std::max<int64_t>(nodes, 1);
    if ((rc = t->cell.grow(cells)) || (rc = t->nm.grow(M1)) || (rc = t->nx.grow(3 * M1)) ||
        (rc = t->nv.grow(3 * M1)) || (rc = t->na.grow(3 * M1)) || (rc = t->nj.grow(3 * M1)) ||
        (rc = t->nlev.grow(M1)) || (rc = t->ncid.grow(M1)) || (rc = t->nraw.grow(13 * M1)) || (rc = t->nrec.grow(M1)) ||
        (rc = t->npar.grow(M1)) || (rc = t->narr.grow(M1)) || (rc = t->nbeg.grow(M1)) || (rc = t->nend.grow(M1)))
        return rc;
    return 0;
}

// Work-groups of the list walk: one per group up to n_list_wg, fewer (down to
// 64) where their scratch would pass 32 GB.
int64_t list_wgs(const htd_tree* t, int64_t groups) {
    const int64_t fit = (int64_t(32) << 30) / (4 * walk_words(t->cut_cap));
    return std::min<int64_t>(groups, std::min<int64_t>(t->n_list_wg, std::max<int64_t>(fit, 64)));
}

// What the cell and node arrays hold, up to a quarter above the last counts
// (the kernels on nodes are launched for as many as may be there).
Caps caps_of(const htd_tree* t) {
    const int64_t arrays = std::min({t->nm.cap, t->nx.cap / 3, t->nv.cap / 3, t->na.cap / 3, t->nj.cap / 3, t->nlev.cap,
                                     t->ncid.cap, t->nraw.cap / 13, t->nrec.cap, t->npar.cap, t->narr.cap, t->nbeg.cap,
                                     t->nend.cap, int64_t(INT32_MAX)});
    return {t->cell.cap, std::min(arrays, t->M + t->M / 4 + 16)};
}

// How much of the rest of a build to queue: everything from the cells on, the
// lists on, or the copy into entries alone.
enum class From { cells, lists, copy };

// Queues it for what the arrays hold, with `groups` groups expected (any number
// is done).  The kernels do nothing where the arrays turn out to be too small.
int queue_rest(htd_tree* t, From from, int64_t n, int n_leaf, double theta, int64_t groups) {
    hipStream_t s = t->stream;
    Progress* pr = t->pr.p;
    const Caps caps = caps_of(t);
    const int64_t M = std::max<int64_t>(caps.nodes, 1);
    if (from == From::cells) {
        cells_kernel<<<blocks_for(n, kWG), kWG, 0, s>>>(n, n_leaf, t->key.p, t->word.p, t->cbase.p, caps, pr, t->cell.p,
                                                        t->nlev.p, t->nbeg.p, t->nend.p, t->ncid.p, t->group_first.p);
        node_recs_kernel<<<blocks_for(M, kWG), kWG, 0, s>>>(caps, pr, t->ncid.p, t->cell.p, t->nrec.p, t->npar.p,
                                                            t->narr.p);
        node_sums_kernel<<<blocks_for(M, kStride), kSumWG, 0, s>>>(
            caps, pr, t->npar.p, t->narr.p, t->sm.p, t->sx.p, t->sv.p, t->sa.p, t->sj.p, t->nraw.p, t->nrec.p,
            NodeOut{t->nm.p, t->nx.p, t->nv.p, t->na.p, t->nj.p});
    }
    if (from != From::copy) {
        ListArgs A{};
        A.n = n;
        A.cut_cap = t->cut_cap;
        A.caps = caps;
        A.pr = pr;
        A.rec = t->nrec.p;
        A.sx = t->sx.p;
        A.group_first = t->group_first.p;
        A.cut = t->cut.p;
        A.stage = t->stage.p;
        A.stage_cap = t->stage.cap;
        A.glen = t->glen.p;
        A.gstage = t->gstage.p;
        A.theta2 = theta * theta;
        lists_kernel<<<static_cast<unsigned>(list_wgs(t, groups)), kListWG, 0, s>>>(A);
        offsets_kernel<<<blocks_for(groups, kOffWG), kOffWG, 0, s>>>(caps, t->stage.cap, pr, t->glen.p, t->glocal.p,
                                                                     t->gpart.p, t->gbase.p, t->out);
    }
    if (t->entries.cap > 0)
        csr_kernel<<<static_cast<unsigned>(std::min<int64_t>(groups, 4096)), kWG, 0, s>>>(
            caps, t->stage.cap, t->entries.cap, pr, t->glen.p, t->glocal.p, t->gbase.p, t->gstage.p, t->stage.p,
            t->list_off.p, t->entries.p);
    HTD_HIP(hipGetLastError());
    return 0;
}

int build(htd_tree* t, int64_t n, const double* x, const double* v, const double* a, const double* jerk,
          const double* m, int n_leaf, int n_crit, double theta) {
    hipStream_t s = t->stream;
    Progress* pr = t->pr.p;
    if (int rc = grow_particles(t, n)) return rc;
    if (n > kRankSort)
        if (int rc = reserve_tmp(t, n)) return rc;
    HTD_HIP(hipEventRecord(t->ev[0], s));
    // 1. root cube, keys, sort; 2. the particle state in key order, counts
    bbox_kernel<<<std::min<unsigned>(kBoxWGs, blocks_for(n, kWG)), kWG, 0, s>>>(n, x, t->part.p, pr);
    if (n <= kRankSort) {
        const bool one = n <= kRun;
        key_runs_kernel<<<blocks_for(n, kRun), kRun, 0, s>>>(n, x, pr, one ? t->key.p : t->key_in.p,
                                                            one ? t->idx.p : t->idx_in.p);
        if (!one)
            merge_runs_kernel<<<blocks_for(n, 64), kMergeWG, 0, s>>>(static_cast<int>(n), t->key_in.p, t->idx_in.p, t->key.p, t->idx.p);
        HTD_HIP(hipGetLastError());
    } else {
        keys_kernel<<<blocks_for(n, kWG), kWG, 0, s>>>(n, x, pr, t->key_in.p, t->idx_in.p);
        HTD_HIP(hipGetLastError());
        size_t bytes = static_cast<size_t>(t->tmp.cap);
        HTD_HIP(rocprim::radix_sort_pairs(t->tmp.p, bytes, t->key_in.p, t->key.p, t->idx_in.p, t->idx.p,
                                          static_cast<size_t>(n), 0, 63, s));
    }
    particles_kernel<<<blocks_for(n, kScanWG), kScanWG, 0, s>>>(
        n, n_leaf, n_crit, t->idx.p, t->key.p, x, v, a, jerk, m, t->perm.p, t->sx.p, t->sv.p, t->sa.p, t->sj.p,
        t->sm.p, t->word.p, t->cpart.p, t->cbase.p, pr, t->out);
    HTD_HIP(hipGetLastError());
    // 3., 4. cells, node moments and lists.  Where the arrays of an earlier build are there, all of
    // it is queued for what they hold before the host knows the counts; a part that does not fit
    // is queued again with larger arrays.
    if (int rc = t->stage.grow(std::max<int64_t>(t->stage.cap, 64 * n))) return rc;
    const bool blind = t->G > 0 && n >= t->n / 2 && n / 2 <= t->n &&
                       t->cut.cap >= list_wgs(t, t->G) * walk_words(t->cut_cap);
    From from = From::cells;
    for (int attempt = 0;; ++attempt) {
        if (attempt > 0 || blind) {
            if (attempt > 0 && from != From::copy) {
                if (int rc = t->cut.grow(list_wgs(t, t->G) * walk_words(t->cut_cap))) return rc;
                HTD_HIP(hipMemsetAsync(&pr->ctr, 0, sizeof(Counters), s));
            }
            if (int rc = queue_rest(t, from, n, n_leaf, theta, t->G)) return rc;
            HTD_HIP(hipEventRecord(t->ev[1], s));
        }
        HTD_HIP(hipStreamSynchronize(s));
        const Outcome o = *t->out;
        const Caps had = caps_of(t);
        if (o.tot.cells < 1 || o.tot.groups < 1) return fail(HTD_EHIP, "tree construction produced no cells");
        t->C = o.tot.cells;
        t->M = o.tot.nodes;
        t->G = o.tot.groups;
        if (t->C > had.cells || t->M > had.nodes || (attempt == 0 && !blind)) {
            if (int rc = grow_nodes(t, t->C, t->M)) return rc;
            continue;
        }
        const int64_t staged = static_cast<int64_t>(o.ctr.staged);
        if (o.ctr.max_cut == 0 && staged <= t->stage.cap) {
            t->L = staged;
            if (staged <= t->entries.cap) break;
            if (int rc = t->entries.grow(std::max<int64_t>(staged, 1))) return rc;
            from = From::copy;
            continue;
        }
        if (attempt >= 32) return fail(HTD_ERANGE, "interaction lists did not fit after %d attempts", attempt + 1);
        from = From::lists;
        if (o.ctr.max_cut > 0) {
            // a group's opened cells outgrew the per-work-group scratch.  They were counted up to
            // the level that did not fit, so the next size at least doubles, up to all nodes.
            if (int64_t(o.ctr.max_cut) > INT32_MAX / 2) return fail(HTD_ERANGE, "a group's list exceeds 2^30 entries");
            t->cut_cap = static_cast<int32_t>(std::min<int64_t>(t->M, 2 * int64_t(o.ctr.max_cut)));
            t->cut.release();
        }
        if (staged > t->stage.cap) {
            t->stage.release();
            if (int rc = t->stage.grow(staged)) return rc;
        }
    }
    t->root_h = t->out->root;
    float ms = 0;
    HTD_HIP(hipEventElapsedTime(&ms, t->ev[0], t->ev[1]));
    t->phase_ms[6] = t->phase_ms[5] = ms;
    for (int i = 0; i < kStamps - 1; ++i) {
        const auto ticks = static_cast<int64_t>(t->out->stamp[i + 1] - t->out->stamp[i]);
        t->phase_ms[i] = static_cast<float>(static_cast<double>(std::max<int64_t>(ticks, 0)) * t->tick_ms);
        t->phase_ms[5] -= t->phase_ms[i];
    }
    t->n = n;
    t->built = true;
    return 0;
}

template <class T>
int copy_out(T* dst, const T* src, int64_t count, hipStream_t s) {
    if (!dst || count <= 0) return 0;
    HTD_HIP(hipMemcpyAsync(dst, src, sizeof(T) * static_cast<size_t>(count), hipMemcpyDeviceToHost, s));
    return 0;
}

}  // namespace

extern "C" {

const char* htd_last_error(void) { return g_err.c_str(); }

int htd_create(htd_tree** out, int32_t device, void* stream, int64_t n_max) {
    if (!out) return fail(HTD_EINVAL, "out is NULL");
    *out = nullptr;
    if (n_max < 1 || n_max > kMaxN) return fail(HTD_EINVAL, "n_max %lld outside [1, 2^26]", (long long)n_max);
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count < 1) return fail(HTD_EHIP, "no HIP device");
    if (device < 0 || device >= count) return fail(HTD_EINVAL, "device %d outside [0, %d)", device, count);
    HTD_HIP(hipSetDevice(device));
    htd_tree* t = new (std::nothrow) htd_tree();
    if (!t) return fail(HTD_ENOMEM, "host allocation failed");
    t->device = device;
    t->stream = static_cast<hipStream_t>(stream);
    t->n_max = n_max;
    for (auto& e : t->ev)
        if (hipEventCreate(&e) != hipSuccess) {
            htd_destroy(t);
            return fail(HTD_EHIP, "hipEventCreate failed");
        }
    int khz = 0;
    if (hipHostMalloc(&t->out, sizeof(Outcome)) != hipSuccess ||
        hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device) != hipSuccess || khz < 1) {
        htd_destroy(t);
        return fail(HTD_EHIP, "pinned memory or the counter's rate is not available");
    }
    t->tick_ms = 1.0 / khz;
    int rc = grow_particles(t, n_max);
    if (rc == 0) rc = t->pr.grow(1);
    if (rc == 0 && hipMemset(t->pr.p, 0, sizeof(Progress)) != hipSuccess) rc = fail(HTD_EHIP, "hipMemset failed");
    if (rc) {
        htd_destroy(t);
        return rc;
    }
    *out = t;
    return 0;
}

int htd_destroy(htd_tree* t) {
    if (!t) return 0;
    (void)hipSetDevice(t->device);
    if (t->stream) (void)hipStreamSynchronize(t->stream);
    else (void)hipDeviceSynchronize();
    for (auto& e : t->ev)
        if (e) (void)hipEventDestroy(e);
    t->key_in.release(); t->key.release(); t->idx_in.release(); t->idx.release(); t->perm.release();
    t->sx.release(); t->sv.release(); t->sa.release(); t->sj.release(); t->sm.release(); t->word.release();
    t->cpart.release(); t->cbase.release(); t->tmp.release(); t->part.release(); t->pr.release();
    t->cell.release(); t->nm.release(); t->nx.release(); t->nv.release(); t->na.release(); t->nj.release();
    t->nlev.release(); t->ncid.release(); t->nraw.release(); t->nrec.release(); t->npar.release();
    t->narr.release(); t->nbeg.release();
    t->nend.release(); t->group_first.release(); t->list_off.release(); t->gstage.release(); t->glocal.release();
    t->gpart.release(); t->gbase.release(); t->glen.release(); t->cut.release(); t->stage.release();
    t->entries.release();
    if (t->out) (void)hipHostFree(t->out);
    delete t;
    return 0;
}

int htd_build(htd_tree* t, int64_t n, const double* d_x, const double* d_v, const double* d_a, const double* d_jerk,
              const double* d_m, int32_t n_leaf, int32_t n_crit, double theta) {
    if (!t) return fail(HTD_EINVAL, "tree is NULL");
    if (n < 1 || n > t->n_max) return fail(HTD_EINVAL, "n = %lld outside [1, %lld]", (long long)n, (long long)t->n_max);
    if (!d_x || !d_v || !d_a || !d_jerk || !d_m) return fail(HTD_EINVAL, "a particle array is NULL");
    if (n_leaf < 1 || n_crit < 1) return fail(HTD_EINVAL, "n_leaf and n_crit must be positive");
    if (!(theta >= 0.0) || !std::isfinite(theta)) return fail(HTD_EINVAL, "theta must be finite and >= 0");
    HTD_HIP(hipSetDevice(t->device));
    t->built = false;
    return build(t, n, d_x, d_v, d_a, d_jerk, d_m, n_leaf, n_crit, theta);
}

int htd_sizes(const htd_tree* t, int64_t* n_node, int64_t* n_group, int64_t* n_entries, int64_t* n_cell) {
    if (!t) return fail(HTD_EINVAL, "tree is NULL");
    if (!t->built) return fail(HTD_ESTATE, "no successful build");
    if (n_node) *n_node = t->M;
    if (n_group) *n_group = t->G;
    if (n_entries) *n_entries = t->L;
    if (n_cell) *n_cell = t->C;
    return 0;
}

int htd_root(const htd_tree* t, double* lo, double* side) {
    if (!t) return fail(HTD_EINVAL, "tree is NULL");
    if (!t->built) return fail(HTD_ESTATE, "no successful build");
    if (lo)
        for (int d = 0; d < 3; ++d) lo[d] = t->root_h.lo[d];
    if (side) *side = t->root_h.side;
    return 0;
}

int htd_get(const htd_tree* t, int64_t* perm, uint64_t* keys, double* node_m, double* node_x, double* node_v,
            double* node_a, double* node_j, int32_t* node_level, int64_t* node_begin, int64_t* node_end,
            int64_t* group_first, int64_t* list_off, int32_t* entries) {
    if (!t) return fail(HTD_EINVAL, "tree is NULL");
    if (!t->built) return fail(HTD_ESTATE, "no successful build");
    HTD_HIP(hipSetDevice(t->device));
    hipStream_t s = t->stream;
    int rc = 0;
    if ((rc = copy_out(perm, t->perm.p, t->n, s)) || (rc = copy_out(keys, t->key.p, t->n, s)) ||
        (rc = copy_out(node_m, t->nm.p, t->M, s)) || (rc = copy_out(node_x, t->nx.p, 3 * t->M, s)) ||
        (rc = copy_out(node_v, t->nv.p, 3 * t->M, s)) || (rc = copy_out(node_a, t->na.p, 3 * t->M, s)) ||
        (rc = copy_out(node_j, t->nj.p, 3 * t->M, s)) || (rc = copy_out(node_level, t->nlev.p, t->M, s)) ||
        (rc = copy_out(node_begin, t->nbeg.p, t->M, s)) || (rc = copy_out(node_end, t->nend.p, t->M, s)) ||
        (rc = copy_out(group_first, t->group_first.p, t->G + 1, s)) ||
        (rc = copy_out(list_off, t->list_off.p, t->G + 1, s)) || (rc = copy_out(entries, t->entries.p, t->L, s)))
        return rc;
    HTD_HIP(hipStreamSynchronize(s));
    return 0;
}

int htd_device_view(const htd_tree* t, htd_view* out) {
    if (!t || !out) return fail(HTD_EINVAL, "NULL argument");
    if (!t->built) return fail(HTD_ESTATE, "no successful build");
    out->perm = t->perm.p;
    out->keys = t->key.p;
    out->x = t->sx.p;
    out->v = t->sv.p;
    out->a = t->sa.p;
    out->jerk = t->sj.p;
    out->m = t->sm.p;
    out->node_m = t->nm.p;
    out->node_x = t->nx.p;
    out->node_v = t->nv.p;
    out->node_a = t->na.p;
    out->node_j = t->nj.p;
    out->group_first = t->group_first.p;
    out->list_off = t->list_off.p;
    out->entries = t->entries.p;
    return 0;
}

int htd_phase_ms(const htd_tree* t, double* ms) {
    if (!t || !ms) return fail(HTD_EINVAL, "NULL argument");
    if (!t->built) return fail(HTD_ESTATE, "no successful build");
    for (int i = 0; i < 7; ++i) ms[i] = t->phase_ms[i];
    return 0;
}

int htd_device_bytes(const htd_tree* t, size_t* bytes) {
    if (!t || !bytes) return fail(HTD_EINVAL, "NULL argument");
    size_t b = 0;
    auto add = [&](const auto& buf) { b += sizeof(*buf.p) * static_cast<size_t>(buf.cap); };
    add(t->key_in), add(t->key), add(t->idx_in), add(t->idx), add(t->perm);
    add(t->sx), add(t->sv), add(t->sa), add(t->sj), add(t->sm), add(t->word), add(t->cpart), add(t->cbase);
    add(t->tmp), add(t->part), add(t->pr), add(t->cell);
    add(t->nm), add(t->nx), add(t->nv), add(t->na), add(t->nj), add(t->nlev), add(t->ncid), add(t->nraw), add(t->nrec);
    add(t->npar), add(t->narr);
    add(t->nbeg), add(t->nend), add(t->group_first), add(t->list_off), add(t->gstage), add(t->glocal), add(t->gpart), add(t->gbase);
    add(t->glen), add(t->cut), add(t->stage), add(t->entries);
    *bytes = b;
    return 0;
}

}  // extern "C"
