// HIP kernels of the MLS-MPM substep for gfx950 (MI355X).
//
// One substep (Algorithm 1, inner loop: particle to grid, grid velocity,
// grid to particle, integrate) runs as
//   k_p2g   particle-to-grid: APIC + MLS stress scatter of one binned chunk of
//           particles into an LDS tile (integer fixed-point accumulation with
//           ds_add_u32, exact and order independent), flushed to the global
//           grid with float atomics;
//   k_grid  grid velocity: v = p/m, gravity, SDF colliders, walls; it zeroes
//           (m, p) after reading them, so no separate clear pass exists;
//   k_g2p   grid-to-particle fused with the integration: velocity and APIC
//           matrix from an LDS tile of grid velocities, x += dt v,
//           F <- (I + dt C) F, Hencky + von Mises return map, and the affine
//           momentum A = m C - dt V (4/dx^2) tau(F) the next P2G scatters.
// Particles are binned by grid block (Morton order inside a scene) every
// few substeps by a counting sort (k_keys .. k_gather).
#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "mpm_device.hpp"
#include <hip/hip_ext.h>

namespace mpm {

// Timing of the substep kernels: events handed in by time_next_launch are
// recorded by the runtime at the start and the end of the next substep
// kernel launched on this thread (hipExtLaunchKernelGGL), so they time the
// kernel itself rather than the queue around it.
static thread_local hipEvent_t t_ev[2] = {nullptr, nullptr};

void time_next_launch(hipEvent_t start, hipEvent_t stop)
{
    t_ev[0] = start;
    t_ev[1] = stop;
}

template <typename... KArgs, typename... Args>
static void launch_timed(void (*kernel)(KArgs...), int n_wg, int nt, hipStream_t st, Args... args)
{
    hipEvent_t a = t_ev[0], b = t_ev[1];
    t_ev[0] = t_ev[1] = nullptr;
    if (a && b) hipExtLaunchKernelGGL(kernel, dim3(n_wg), dim3(nt), 0, st, a, b, 0, args...);
    else kernel<<<n_wg, nt, 0, st>>>(args...);
}

// ====================================================================== sort
// Runs of equal keys in consecutive lanes (the particles are nearly sorted
// from the previous sort): one atomic per run instead of one per particle.
struct KeyRun {
    int head_lane;   // first lane of this lane's run
    int len;         // run length (valid at the head lane)
};

__device__ __forceinline__ KeyRun key_run(unsigned key)
{
    const int lane = threadIdx.x & 63;
    const unsigned prev = __shfl_up(key, 1, 64);
    const bool head = lane == 0 || prev != key;
    const unsigned long long heads = __ballot(head);
    const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
    KeyRun r;
    r.head_lane = 63 - __clzll(heads & upto);
    const unsigned long long after = heads & ~upto;
    const int next = after ? __ffsll((long long)after) - 1 : 64;
    r.len = next - lane;
    return r;
}

__device__ __forceinline__ unsigned particle_key(const SortArgs &a, int j)
{
    int s = a.psc[j];
    const SceneDev &S = a.scenes[s];
    int b[3], cl = 0;
    float f;
    for (int d = 0; d < 3; d++) particle_base(S, a.x[d * a.x_comp + j * a.x_part], b[d], f, cl);
    return (unsigned)a.scene_bin_off[s] + morton3(b[0] / a.B, b[1] / a.B, b[2] / a.B);
}

// Particles per thread of k_keys and k_scatter: 8 where that still fills the chip, else 1.
constexpr int SORT_PER = 8, SORT_PER_MIN = 1 << 19;

// A workgroup's own counts per bin, an open-addressed table in LDS (as many
// slots as the workgroup has particles, so a free one is always found): a scene
// in creation order has its particles in random bins, a few dozen of them, and
// one global atomic per particle (or run of equal keys) on so few addresses is
// what these two kernels spent their time on (7.7 million particles in creation
// order: keys 350 -> 55 us, scatter 556 -> 69).
template <int PER>
struct BinTable {
    static constexpr int SLOTS = PER == 1 ? 2 * WG : PER * WG;
    static constexpr unsigned FREE = 0xFFFFFFFFu;   // no bin has this number
    unsigned key[SLOTS];
    int cnt[SLOTS];
    __device__ void clear()
    {
        for (int q = threadIdx.x; q < SLOTS; q += WG) {
            key[q] = FREE;
            cnt[q] = 0;
        }
    }
    __device__ int slot(unsigned k)
    {
        int h = (int)((k * 2654435761u) >> 8) & (SLOTS - 1);
        for (;;) {
            const unsigned old = atomicCAS(&key[h], FREE, k);
            if (old == FREE || old == k) return h;
            h = (h + 1) & (SLOTS - 1);
        }
    }
};

template <int PER>
__global__ __launch_bounds__(WG) void k_keys(SortArgs a)
{
    __shared__ BinTable<PER> tab;
    tab.clear();
    const int base = xcd_remap(blockIdx.x, gridDim.x) * (WG * PER) + threadIdx.x;
    unsigned key[PER];
#pragma unroll
    for (int i = 0; i < PER; i++) key[i] = base + i * WG < a.N ? particle_key(a, base + i * WG) : tab.FREE;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const bool valid = base + i * WG < a.N;
        if (valid) a.keys[base + i * WG] = key[i];
        const KeyRun r = key_run(key[i]);
        if (valid && r.head_lane == (int)(threadIdx.x & 63)) atomicAdd(&tab.cnt[tab.slot(key[i])], r.len);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < tab.SLOTS; q += WG)
        if (tab.cnt[q] > 0) atomicAdd(&a.count[tab.key[q]], tab.cnt[q]);
}

// Grid blocks that receive mass from particles at home in their bin: the
// block itself and its upper neighbours (a stencil spans base .. base + 2).
// Mass a drifted particle puts one block lower is queued on the overflow
// list by P2G itself.
__device__ __forceinline__ int dilate_bin(const SortArgs &a, int b)
{
    int s = scene_of_bin(a.scene_bin_off, a.n_scenes, b);
    const SceneDev &S = a.scenes[s];
    int off = a.scene_bin_off[s];
    uint32_t m = (uint32_t)(b - off);
    int bx = compact3(m), by = compact3(m >> 1), bz = compact3(m >> 2);
    int nb = S.nb, hit = 0;
    for (int dx = -1; dx <= 0; dx++)
        for (int dy = -1; dy <= 0; dy++)
            for (int dz = -1; dz <= 0; dz++) {
                int x = bx + dx, y = by + dy, z = bz + dz;
                if (x < 0 || y < 0 || z < 0 || x >= nb || y >= nb || z >= nb) continue;
                hit |= a.count[off + morton3(x, y, z)] > 0;
            }
    a.L.bflag[off + (bx * nb + by) * nb + bz] = hit ? 2 : 0;
    return hit;
}

__global__ __launch_bounds__(WG) void k_dilate(SortArgs a)
{
    int b = blockIdx.x * WG + threadIdx.x;
    if (b < a.T) a.dil[b] = (unsigned char)dilate_bin(a, b);
}

static constexpr int SCAN_PER = 8;
static constexpr int SCAN_TILE = WG * SCAN_PER;

// Particles per item of a block with c of them: a.cut (a.CH where the scenes'
// material is dense at rest), or a.CH where the block holds over 12 particles a
// cell all the same, compressed or placed on top of each other.  An item's P2G
// takes its fixed-point scale from its own scatter bound and fullest cell, so in
// dense material a piece has a finer scale than its block, and the rounding of
// its terms would follow the launch configuration (6,000 fluid particles at 40 a
// cell: velocity gradients moved by 2e-5, 6,360 -> 3,160 us).  Where the single
// term's limit sets the scale it is the last bit of the block's largest term.
__device__ __forceinline__ int item_size(const SortArgs &a, int c)
{
    return c <= 12 * a.B * a.B * a.B ? a.cut : a.CH;
}

__device__ __forceinline__ int3 bin_triple(const SortArgs &a, int b, int dil)
{
    const int c = a.count[b], ch = item_size(a, c);
    return make_int3(c, (c + ch - 1) / ch, dil);
}

__device__ __forceinline__ int3 bin_triple(const SortArgs &a, int b)
{
    return b < a.T ? bin_triple(a, b, (int)a.dil[b]) : make_int3(0, 0, 0);
}

__device__ __forceinline__ int3 add3(int3 x, int3 y) { return make_int3(x.x + y.x, x.y + y.y, x.z + y.z); }

// Exclusive scan of one int3 per thread over the workgroup; returns the total.
template <int NT = WG>
__device__ int3 block_exscan3(int3 v, int3 &excl)
{
    __shared__ int3 wsum[NT / 64];
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int3 inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        int3 t;
        t.x = __shfl_up(inc.x, o, 64);
        t.y = __shfl_up(inc.y, o, 64);
        t.z = __shfl_up(inc.z, o, 64);
        if (lane >= o) inc = add3(inc, t);
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int3 before = make_int3(0, 0, 0), total = make_int3(0, 0, 0);
    for (int i = 0; i < NT / 64; i++) {
        if (i < w) before = add3(before, wsum[i]);
        total = add3(total, wsum[i]);
    }
    excl = make_int3(before.x + inc.x - v.x, before.y + inc.y - v.y, before.z + inc.z - v.z);
    __syncthreads();
    return total;
}

__global__ __launch_bounds__(WG) void k_scan_tiles(SortArgs a)
{
    int base = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_PER;
    int3 s = make_int3(0, 0, 0);
    for (int i = 0; i < SCAN_PER; i++) s = add3(s, bin_triple(a, base + i));
    int3 ex;
    int3 tot = block_exscan3(s, ex);
    if (threadIdx.x == 0) a.tsum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(WG) void k_scan_top(SortArgs a, int ntiles)
{
    int3 carry = make_int3(0, 0, 0);
    for (int base = 0; base < ntiles; base += WG) {
        int i = base + threadIdx.x;
        int3 v = i < ntiles ? a.tsum[i] : make_int3(0, 0, 0);
        int3 ex;
        int3 tot = block_exscan3(v, ex);
        if (i < ntiles) a.tsum[i] = add3(ex, carry);
        carry = add3(carry, tot);
    }
    if (threadIdx.x == 0) {
        *a.L.n_items = carry.y;
        *a.L.n_gitems = carry.z;
        a.L.scene_item_begin[a.n_scenes] = carry.y;
        a.L.scene_gitem_begin[a.n_scenes] = carry.z;
    }
}

// v: the bin's counts (bin_triple), run: their sums over the bins before it.
__device__ void emit_bin(const SortArgs &a, int b, int3 v, int3 run)
{
    a.pstart[b] = run.x;
    int sc = scene_of_bin(a.scene_bin_off, a.n_scenes, b);
    int off = a.scene_bin_off[sc];
    if (b == off) {
        a.L.scene_item_begin[sc] = run.y;
        a.L.scene_gitem_begin[sc] = run.z;
    }
    if (v.x > 0 || v.z > 0) {
        const SceneDev &S = a.scenes[sc];
        uint32_t m = (uint32_t)(b - off);
        int bx = compact3(m), by = compact3(m >> 1), bz = compact3(m >> 2);
        int lb = (bx * S.nb + by) * S.nb + bz;
        const int ch = item_size(a, v.x);
        for (int c = 0; c < v.y; c++) {
            Item it;
            it.scene = sc;
            it.block = lb;
            it.start = run.x + c * ch;
            it.count = min(ch, v.x - c * ch);
            a.L.items[run.y + c] = it;
        }
        if (v.z) a.L.gitems[run.z] = make_int2(sc, lb);
    }
}

__global__ __launch_bounds__(WG) void k_scan_emit(SortArgs a)
{
    int base = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_PER;
    int3 v[SCAN_PER];
    int3 s = make_int3(0, 0, 0);
    for (int i = 0; i < SCAN_PER; i++) {
        v[i] = bin_triple(a, base + i);
        s = add3(s, v[i]);
    }
    int3 ex;
    block_exscan3(s, ex);
    int3 run = add3(ex, a.tsum[blockIdx.x]);
    for (int i = 0; i < SCAN_PER; i++) {
        if (base + i < a.T) emit_bin(a, base + i, v[i], run);
        run = add3(run, v[i]);
    }
}

// Inside its bin a particle's slot is scrambled (local rank r -> r * 104729 mod
// bin size, a bijection unless the prime divides the size, which then keeps
// r), so a bin's
// particles end up in an order unrelated to space: consecutive lanes of a
// P2G wave then land on distant cells, and their LDS atomics rarely collide
// on an address or a bank.  (In the order of the previous sort they arrive
// clustered cell by cell.)
constexpr long long BIN_SCRAMBLE = 104729;   // prime

template <int PER>
__global__ __launch_bounds__(WG) void k_scatter(SortArgs a)
{
    __shared__ BinTable<PER> tab;
    __shared__ int2 bin[BinTable<PER>::SLOTS];   // start and size of the slot's bin
    tab.clear();
    // a contiguous share per XCD: a scene's part of perm fills in one L2
    const int base = xcd_remap(blockIdx.x, gridDim.x) * (WG * PER) + threadIdx.x;
    const int lane = threadIdx.x & 63;
    unsigned key[PER];
    int slot[PER], local[PER];
#pragma unroll
    for (int i = 0; i < PER; i++) key[i] = base + i * WG < a.N ? a.keys[base + i * WG] : tab.FREE;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const KeyRun r = key_run(key[i]);
        int sl = 0, off = 0;
        if (base + i * WG < a.N && r.head_lane == lane) {
            sl = tab.slot(key[i]);
            off = atomicAdd(&tab.cnt[sl], r.len);
        }
        // the run takes the workgroup's ranks [off, off + len) of its bin in lane order
        slot[i] = __shfl(sl, r.head_lane, 64);
        local[i] = __shfl(off, r.head_lane, 64) + (lane - r.head_lane);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < tab.SLOTS; q += WG) {
        const int n = tab.cnt[q];
        if (n == 0) continue;
        const unsigned k = tab.key[q];
        const int b0 = a.pstart[k];
        bin[q] = make_int2(b0, ((int)k + 1 < a.T ? a.pstart[k + 1] : a.N) - b0);
        tab.cnt[q] = atomicSub(&a.count[k], n) - n;   // the workgroup's ranks in its bin
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; i++) {
        if (base + i * WG >= a.N) continue;
        const int2 b = bin[slot[i]];
        const long long mul = (b.y % BIN_SCRAMBLE) ? BIN_SCRAMBLE : 1;   // a bijection for any size
        const long long at = (long long)(tab.cnt[slot[i]] + local[i]) * mul;
        a.perm[b.x + (b.y <= 40000 ? (int)((unsigned)at % (unsigned)b.y) : (int)(at % b.y))] = base + i * WG;
    }
}

// Order inside a work item so that the lanes of a P2G wave scatter into
// distinct LDS banks.  A particle's bank class is the tile address of its
// base node mod 64; every stencil offset adds the same constant to all
// lanes, so lanes with distinct classes hit distinct banks.  Particles are
// ranked inside their class and laid out by (rank, class): the first 64
// slots hold rank 0 of every class present, the next ones rank 1, and so on.
// Slot of (rank r, class c) = sum_c' min(count[c'], r) + #{c' < c : count[c'] > r}.
// Edge of a work item's node tile (P2G sums, G2P velocities) for grid blocks of
// edge B: the tile starts one node below the block, and a particle is handled
// in it while its base cell lies at tile coordinates 0 .. B, i.e. in the
// block (1 .. B, where the sort put it) or one cell below; its stencil then
// reaches tile nodes 0 .. B + 2.  Particles past that range since the last
// re-sort take the global path.  The material of the substep workloads sinks
// and is pushed down: the allowance below is the one that matters (on the
// measured runs at most 0.07 % of the particles leave this range between
// re-sorts every 50 substeps, 0.6 % with the allowance above instead).
template <int B> constexpr int tile_edge() { return B + 3; }
// Largest base-cell tile coordinate of a particle handled in the tile.
template <int B> constexpr int tile_bmax() { return tile_edge<B>() - 3; }

constexpr int BANK_CLASSES = 64;

template <int B>
__global__ __launch_bounds__(WG) void k_bank_order(SortArgs a)
{
    constexpr int T = tile_edge<B>();
    __shared__ int cnt[BANK_CLASSES];
    __shared__ unsigned short rank[8192];
    __shared__ unsigned char cls[8192];
    const int n_items = *a.L.n_items;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const Item item = a.L.items[it];
        if (threadIdx.x < BANK_CLASSES) cnt[threadIdx.x] = 0;
        __syncthreads();
        const SceneDev &S = a.scenes[item.scene];
        const int nb = S.nb;
        const int org[3] = {(item.block / (nb * nb)) * B - 1, ((item.block / nb) % nb) * B - 1, (item.block % nb) * B - 1};
        for (int li = threadIdx.x; li < item.count; li += WG) {
            const int j = a.perm[item.start + li];
            int tb[3], cl = 0;
            float f;
            for (int d = 0; d < 3; d++) {
                int b;
                particle_base(S, a.x[d * a.x_comp + j * a.x_part], b, f, cl);
                tb[d] = min(max(b - org[d], 0), T - 1);
            }
            const int c = ((tb[0] * T + tb[1]) * T + tb[2]) % BANK_CLASSES;
            cls[li] = (unsigned char)c;
            rank[li] = (unsigned short)atomicAdd(&cnt[c], 1);
        }
        __syncthreads();
        for (int li = threadIdx.x; li < item.count; li += WG) {
            const int c = cls[li], r = rank[li];
            int pos = 0;
            for (int q = 0; q < BANK_CLASSES; q++) {
                const int k = cnt[q];
                pos += min(k, r) + ((q < c && k > r) ? 1 : 0);
            }
            a.perm2[item.start + pos] = a.perm[item.start + li];
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(WG) void k_gather(SortArgs a)
{
    // contiguous share per XCD: the sources of a bin (scattered over that
    // bin's old range) are fetched into one L2 rather than into all eight
    int p = xcd_remap(blockIdx.x, gridDim.x) * WG + threadIdx.x;
    if (p >= a.N) return;
    int j = a.perm2[p];
    // all loads before any store: the compiler cannot tell that the two
    // buffers do not overlap, and would otherwise wait for each store
    const float *__restrict__ src = a.P;
    float *__restrict__ dst = a.Pn;
    float v[NCOMP];
#pragma unroll
    for (int c = 0; c < NCOMP; c++) v[c] = src[(long long)c * a.pstride + j];
#pragma unroll
    for (int c = 0; c < NCOMP; c++) dst[(long long)c * a.pstride + p] = v[c];
}

// Dispatch order of the work items for P2G and G2P: most particles first.
// Those kernels take one item per workgroup in workgroup order (the
// dispatcher deals workgroups to the XCDs in turn, so each XCD gets every
// eighth item of the order), and items range from a few dozen particles to
// a full chunk: in block order the largest ones could start last and hold
// the end of the launch.  A counting sort by particle count in 64 classes
// (order inside a class: arbitrary).  Where blocks are cut below the chunk, half
// of the classes are for the items up to the cut, half for the whole blocks past
// it: 64 classes of the chunk would put the pieces of a small context into one.
constexpr int ORDER_CLASSES = 64;

__device__ __forceinline__ int order_class(const SortArgs &a, int count)
{
    constexpr int H = ORDER_CLASSES / 2;
    if (a.cut >= a.CH) return min(ORDER_CLASSES - 1, (int)((long long)count * ORDER_CLASSES / (a.CH + 1)));
    return count <= a.cut ? count * H / (a.cut + 1) : H + (count - a.cut - 1) * H / (a.CH - a.cut);
}

__global__ __launch_bounds__(1024) void k_item_order(SortArgs a)
{
    __shared__ int cnt[ORDER_CLASSES];
    const int n = *a.L.n_items;
    if (threadIdx.x < ORDER_CLASSES) cnt[threadIdx.x] = 0;
    __syncthreads();
    for (int it = threadIdx.x; it < n; it += blockDim.x) atomicAdd(&cnt[order_class(a, a.L.items[it].count)], 1);
    __syncthreads();
    if (threadIdx.x == 0) {
        int s = 0;   // classes from the largest down: cnt[c] becomes the first slot of class c
        for (int c = ORDER_CLASSES - 1; c >= 0; c--) {
            const int k = cnt[c];
            cnt[c] = s;
            s += k;
        }
    }
    __syncthreads();
    for (int it = threadIdx.x; it < n; it += blockDim.x)
        a.L.order[atomicAdd(&cnt[order_class(a, a.L.items[it].count)], 1)] = it;
}

// k_dilate, the three scan kernels and k_item_order in one workgroup, for few
// bins: five dependent launches of a few microseconds each were most of a small
// context's sort (8,192 particles, 512 bins: 23.7 us and the gaps between them
// -> 10.9 us).  Up to two bins a thread: at 4,096 bins the eight counts that each
// reads for its neighbours wait on one CU, 21.5 us against about as much.
constexpr int SMALL_PER = 2, SMALL_BINS = SMALL_PER * 1024;

__global__ __launch_bounds__(1024) void k_plan_small(SortArgs a)
{
    __shared__ int cls[ORDER_CLASSES];
    static_assert(ORDER_CLASSES == 64, "one class per lane");
    const int t = threadIdx.x, per = (a.T + 1023) / 1024, base = t * per;
    if (t < ORDER_CLASSES) cls[t] = 0;
    int3 v[SMALL_PER], sum = make_int3(0, 0, 0), run;
#pragma unroll
    for (int i = 0; i < SMALL_PER; i++) {
        v[i] = make_int3(0, 0, 0);
        if (i < per && base + i < a.T) v[i] = bin_triple(a, base + i, dilate_bin(a, base + i));
        sum = add3(sum, v[i]);
    }
    const int3 total = block_exscan3<1024>(sum, run);
    if (t == 0) {
        *a.L.n_items = total.y;
        *a.L.n_gitems = total.z;
        a.L.scene_item_begin[a.n_scenes] = total.y;
        a.L.scene_gitem_begin[a.n_scenes] = total.z;
    }
    const int item0 = run.y;
#pragma unroll
    for (int i = 0; i < SMALL_PER; i++) {
        if (i >= per || base + i >= a.T) break;
        emit_bin(a, base + i, v[i], run);
        run = add3(run, v[i]);
    }
    // the items' dispatch order, as k_item_order's: f(item, class) over this thread's items
    auto own_items = [&](auto f) {
        int it = item0;
#pragma unroll
        for (int i = 0; i < SMALL_PER; i++) {
            const int ch = item_size(a, v[i].x);
            for (int c = 0; c < v[i].y; c++, it++) f(it, order_class(a, min(ch, v[i].x - c * ch)));
        }
    };
    own_items([&](int, int c) { atomicAdd(&cls[c], 1); });
    __syncthreads();
    if (t < ORDER_CLASSES) {
        // classes from the largest down: lane t holds class 63 - t, its first slot is the sum before it
        const int n = cls[ORDER_CLASSES - 1 - t];
        int inc = n;
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(inc, o, 64);
            if (t >= o) inc += u;
        }
        cls[ORDER_CLASSES - 1 - t] = inc - n;
    }
    __syncthreads();
    own_items([&](int it, int c) { a.L.order[atomicAdd(&cls[c], 1)] = it; });
}

// Scale bound of every new work item (the P2G fixed-point scale), from the
// freshly gathered particles.
__global__ __launch_bounds__(WG) void k_item_bounds(SortArgs a)
{
    __shared__ float red[WG / 64];
    const int n_items = *a.L.n_items;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const Item item = a.L.items[it];
        const SceneDev &S = a.scenes[item.scene];
        float b = 0.0f;
        for (int li = threadIdx.x; li < item.count; li += WG) {
            const long long j = item.start + li;
            float v[3], A[9];
            for (int d = 0; d < 3; d++) v[d] = a.Pn[(V0 + d) * a.pstride + j];
            for (int e = 0; e < 9; e++) A[e] = a.Pn[(A00 + e) * a.pstride + j];
            b = fmaxf(b, scatter_bound(S.mass, S.dx, v, A));
        }
        b = wave_max(b);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = b;
        __syncthreads();
        if (threadIdx.x == 0) {
            a.L.ibound[it] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
            a.L.icell[it] = 0;   // per-cell counts unknown: the next P2G counts
        }
        __syncthreads();
    }
}

// A non-finite x, v, C or F (or an F whose stress is not defined) sets the
// scene's FLAG_NONFINITE: inside a substep the fixed-point P2G would turn it
// into finite garbage rather than propagate it.
__device__ __forceinline__ void init_particle(const SceneDev *scenes, int s, const float (&x)[3], const float (&v)[3],
                                              const float (&C)[9], const float (&F)[9], float *P, long long ps, int slot,
                                              int id, int *flags)
{
    const SceneDev &S = scenes[s];
    const Material mat = material_of(S);
    const float mass = S.mass, kstress = S.kstress;   // before the stores, which may alias the scene for the compiler
    float G[9], tau[9];
#pragma unroll
    for (int e = 0; e < 9; e++) G[e] = F[e] - (e % 4 == 0 ? 1.0f : 0.0f);
    int bad = 0;
    state_stress(G, mat, tau, bad);
    float chk = 0.0f;   // NaN or infinity in any input makes it fail the test below
#pragma unroll
    for (int d = 0; d < 3; d++) {
        chk += fabsf(x[d]) + fabsf(v[d]);
        P[(X0 + d) * ps + slot] = x[d];
        P[(V0 + d) * ps + slot] = v[d];
    }
#pragma unroll
    for (int e = 0; e < 9; e++) chk += fabsf(G[e]) + fabsf(C[e]) + fabsf(tau[e]);
    if (bad || !(chk <= 3.0e38f)) atomicOr(flags + s, (int)FLAG_NONFINITE);
#pragma unroll
    for (int e = 0; e < 9; e++) {
        P[(A00 + e) * ps + slot] = fmaf(mass, C[e], -kstress * tau[e]);
        P[(G00 + e) * ps + slot] = G[e];
    }
    P[PID * ps + slot] = __int_as_float(id);
}

template <int N>
__device__ __forceinline__ void load_row(float (&r)[N], const float *src)
{
    __builtin_memcpy(r, src, sizeof(r));   // the widest loads that a 4-byte alignment allows
}

// k_gather for a state handed in as rows: each particle goes straight to its
// sorted slot, its 24 floats in 5 or 6 cache lines where the gather from
// component arrays in creation order takes 25 (7.7 million particles: in and
// gather 460 + 995 -> 550 us).
__global__ __launch_bounds__(WG) void k_gather_rows(SortArgs a, StateRows w, int *flags)
{
    const int p = xcd_remap(blockIdx.x, gridDim.x) * WG + threadIdx.x;
    if (p >= a.N) return;
    const long long j = a.perm2[p];
    float x[3], v[3], C[9], F[9];
    load_row(x, w.x + 3 * j);
    load_row(v, w.v + 3 * j);
    load_row(C, w.C + 9 * j);
    load_row(F, w.F + 9 * j);
    init_particle(a.scenes, a.psc[p], x, v, C, F, a.Pn, a.pstride, p, (int)j, flags);
}

hipError_t launch_sort(const SortArgs &a, const StateRows *rows, int *flags, hipStream_t st)
{
    int gN = (a.N + WG - 1) / WG, gT = (a.T + WG - 1) / WG;
    int ntiles = (a.T + SCAN_TILE - 1) / SCAN_TILE;
    // xcd_remap needs a multiple of 8 workgroups
    const bool wide = a.N >= SORT_PER_MIN;
    const int gS = (wide ? (a.N + WG * SORT_PER - 1) / (WG * SORT_PER) + 7 : gN + 7) & ~7;
    if (a.N > 0) {
        if (wide) k_keys<SORT_PER><<<gS, WG, 0, st>>>(a);
        else k_keys<1><<<gS, WG, 0, st>>>(a);
    }
    if (a.T <= SMALL_BINS) {
        k_plan_small<<<1, 1024, 0, st>>>(a);
    } else {
        k_dilate<<<gT, WG, 0, st>>>(a);
        k_scan_tiles<<<ntiles, WG, 0, st>>>(a);
        k_scan_top<<<1, WG, 0, st>>>(a, ntiles);
        k_scan_emit<<<ntiles, WG, 0, st>>>(a);
        k_item_order<<<1, 1024, 0, st>>>(a);
    }
    if (a.N > 0) {
        const int gN8 = (gN + 7) & ~7;    // xcd_remap (gather) needs a multiple of 8 workgroups
        if (wide) k_scatter<SORT_PER><<<gS, WG, 0, st>>>(a);
        else k_scatter<1><<<gS, WG, 0, st>>>(a);
        if (a.B == 4) k_bank_order<4><<<2048, WG, 0, st>>>(a);
        else k_bank_order<8><<<2048, WG, 0, st>>>(a);
        if (rows) k_gather_rows<<<gN8, WG, 0, st>>>(a, *rows, flags);
        else k_gather<<<gN8, WG, 0, st>>>(a);
        k_item_bounds<<<2048, WG, 0, st>>>(a);
    }
    return hipGetLastError();
}

// ====================================================================== substep pieces
__device__ __forceinline__ void load_particle_xvA(const StepArgs &a, int jj, float x[3], float v[3], float A[9])
{
    const float *P = a.P;
    const long long ps = a.pstride;
    const unsigned jo = (unsigned)jj << 2;
#pragma unroll
    for (int d = 0; d < 3; d++) {
        x[d] = pload(P, ps, X0 + d, jo);
        v[d] = pload(P, ps, V0 + d, jo);
    }
#pragma unroll
    for (int e = 0; e < 9; e++) A[e] = pload(P, ps, A00 + e, jo);
}

// Length of the overflow list of substep k.  Two counters alternate by
// substep parity: the G2P of substep k clears counter k & 1 (its grid update
// has consumed the list) while a P2G fused into the same launch already
// fills the list of substep k + 1; at the end of every substep both are zero.
__device__ __forceinline__ int *ovf_count(const StepArgs &a, int k) { return a.L.n_ovf + (k & 1); }

// What the scatter paths write, read from the kernel's argument segment where
// it is needed (the kernels' only argument is their StepArgs): kept live over
// the particle loops these pointers would push the loops' own scalars out of
// the scalar registers (each use of a spilled one is a vector instruction).
struct GridOut {
    float *gm, *gpx, *gpy, *gpz;
    unsigned char *touched;
    int *bflag, *n_ovf, *flags;
    int2 *ovf;
    int ovf_cap;
};

__device__ __forceinline__ GridOut grid_out(int k)
{
    typedef const __attribute__((address_space(4))) StepArgs args_t;
    args_t *p = (args_t *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return {p->gm, p->gpx, p->gpy, p->gpz, p->L.touched, p->L.bflag, p->L.n_ovf + (k & 1), p->flags, p->L.ovf, p->L.ovf_cap};
}

// Put a grid block that is not on the static update list on the overflow
// list (once per substep) of the substep that scatters.
__device__ __forceinline__ void queue_block(const GridOut &o, int s, int bin_off, int lb)
{
    int *fl = o.bflag + bin_off + lb;
    if (*fl == 0 && atomicCAS(fl, 0, 1) == 0) {
        int pos = atomicAdd(o.n_ovf, 1);
        if (pos < o.ovf_cap) o.ovf[pos] = make_int2(s, lb);
        else atomicOr(o.flags + s, (int)FLAG_OVERFLOW_FULL);
    }
}

// Quadratic B-spline weight of node o (0, 1, 2) for the offset f: bspline_w's
// polynomials, for any f (a particle past the grid's edge has a clamped base
// cell and an offset outside [0.5, 1.5); its weights still sum to 1).
__device__ __forceinline__ float bspline_at(float f, float o)
{
    const float u = f - o, e = fmaf(o - 1.0f, u, 1.5f);
    return o == 1.0f ? 0.75f - u * u : 0.5f * e * e;
}

// Slow path of P2G: scatter one particle straight into the global grid and
// queue any block that is not already on the grid-update list.  home: grid
// block of the particle's work item; that block and its upper neighbours are
// on the list from the sort on, so only blocks outside them are checked (each
// check waits for a global round trip).  The scene constants are copied into
// registers first: the atomics may alias the scene record for the compiler,
// which would otherwise reload it, waiting for every atomic issued so far,
// before each one.
template <int B>
__device__ void p2g_global(const GridOut &o, int s, const SceneDev &S, const float v[3], const float A[9], const int b[3],
                           const float f[3], int3 home)
{
    const float mass = uniform_f(S.mass), dx = uniform_f(S.dx);
    const int nb = uniform_i(S.nb), bin_off = uniform_i(S.bin_off);
    const SceneDev Sg = {0, 0, uniform_i(S.res), nb, uniform_ll(S.grid_off)};
    // rolled: unrolled, the 27 nodes' temporaries cost the kernels around it their registers
#pragma unroll 1
    for (int n = 0; n < 27; n++) {
        const int q[3] = {n / 9, n / 3 % 3, n % 3};
        float wt = 1.0f, d[3];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            wt *= bspline_at(f[k], (float)q[k]);
            d[k] = ((float)q[k] - f[k]) * dx;
        }
        const long long idx = node_index(Sg, B, b[0] + q[0], b[1] + q[1], b[2] + q[2]);
        atomicAdd(o.gm + idx, wt * mass);
        atomicAdd(o.gpx + idx, wt * (mass * v[0] + A[0] * d[0] + A[1] * d[1] + A[2] * d[2]));
        atomicAdd(o.gpy + idx, wt * (mass * v[1] + A[3] * d[0] + A[4] * d[1] + A[5] * d[2]));
        atomicAdd(o.gpz + idx, wt * (mass * v[2] + A[6] * d[0] + A[7] * d[1] + A[8] * d[2]));
    }
#pragma unroll 1
    for (int cx = 0; cx < 2; cx++)
#pragma unroll 1
        for (int cy = 0; cy < 2; cy++)
#pragma unroll 1
            for (int cz = 0; cz < 2; cz++) {
                const int bx = (b[0] + 2 * cx) / B, by = (b[1] + 2 * cy) / B, bz = (b[2] + 2 * cz) / B;
                if ((cx && bx == b[0] / B) || (cy && by == b[1] / B) || (cz && bz == b[2] / B)) continue;
                const int lb = (bx * nb + by) * nb + bz;
                o.touched[bin_off + lb] = 1;
                if ((unsigned)(bx - home.x) > 1u || (unsigned)(by - home.y) > 1u || (unsigned)(bz - home.z) > 1u)
                    queue_block(o, s, bin_off, lb);
            }
}


// Slow lanes of a wave up to this many take the wave-wide slow paths below
// (about 120 instructions a particle for the scatter and 80 for the gather),
// more the lane-by-lane ones (950 and 750 instructions for any number of
// lanes): on the 256-scene workload 0.3 % of the particles change their base
// cell in a substep and up to 1 % have left their tile before the next
// re-sort, one or two lanes of every sixth to every second wave.
constexpr int COOP_LANES = 8;

__device__ __forceinline__ float lane_f(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }

// p2g_global for the lanes of `mask`, one particle after the other, its 27
// nodes on 27 lanes (every lane of the wave must be active).
template <int B>
__device__ void p2g_global_wave(const GridOut &o, int s, const SceneDev &S, unsigned long long mask, const float v[3],
                                const float A[9], const int b[3], const float f[3], int3 home)
{
    const float mass = uniform_f(S.mass), dx = uniform_f(S.dx);
    const int nb = uniform_i(S.nb), bin_off = uniform_i(S.bin_off);
    const SceneDev Sg = {0, 0, uniform_i(S.res), nb, uniform_ll(S.grid_off)};
    int lane = threadIdx.x & 63;
    asm("" : "+v"(lane));   // opaque: what follows from it is formed here, not kept over the particle loop
    const int ox = lane / 9, oy = lane / 3 % 3, oz = lane % 3;
    const float of[3] = {(float)ox, (float)oy, (float)oz};
    while (mask) {
        const int l = __ffsll(mask) - 1;
        mask &= mask - 1;
        int bs[3];
        float w = 1.0f, d[3];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            bs[k] = __builtin_amdgcn_readlane(b[k], l);
            const float fs = lane_f(f[k], l);
            w *= bspline_at(fs, of[k]);
            d[k] = (of[k] - fs) * dx;
        }
        float p[3];
#pragma unroll
        for (int c = 0; c < 3; c++)
            p[c] = mass * lane_f(v[c], l) + lane_f(A[3 * c], l) * d[0] + lane_f(A[3 * c + 1], l) * d[1] + lane_f(A[3 * c + 2], l) * d[2];
        if (lane < 27) {
            const long long idx = node_index(Sg, B, bs[0] + ox, bs[1] + oy, bs[2] + oz);
            atomicAdd(o.gm + idx, w * mass);
            atomicAdd(o.gpx + idx, w * p[0]);
            atomicAdd(o.gpy + idx, w * p[1]);
            atomicAdd(o.gpz + idx, w * p[2]);
        }
        if (lane < 8) {
            const int cx = lane >> 2, cy = (lane >> 1) & 1, cz = lane & 1;
            const int bx = (bs[0] + 2 * cx) / B, by = (bs[1] + 2 * cy) / B, bz = (bs[2] + 2 * cz) / B;
            if (!((cx && bx == bs[0] / B) || (cy && by == bs[1] / B) || (cz && bz == bs[2] / B))) {
                const int lb = (bx * nb + by) * nb + bz;
                o.touched[bin_off + lb] = 1;
                if ((unsigned)(bx - home.x) > 1u || (unsigned)(by - home.y) > 1u || (unsigned)(bz - home.z) > 1u)
                    queue_block(o, s, bin_off, lb);
            }
        }
    }
}

// G2P's gather for the lanes of `mask` (particles outside the tile), two
// particles at a time, their 27 nodes on the two halves of the wave (every
// lane must be active): vp = sum w v, So[c][e] = sum w v_c o_e.
template <int B>
__device__ void gather_wave(const StepArgs &a, const SceneDev &Sn, unsigned long long mask, const int b[3], const float f[3],
                            float vp[3], float So[3][3])
{
    int lane = threadIdx.x & 63;
    asm("" : "+v"(lane));   // as above
    const int n = lane & 31;
    const bool hi = lane >= 32;
    const int o[3] = {n / 9, n / 3 % 3, n % 3};
    while (mask) {
        const int l0 = __ffsll(mask) - 1;
        mask &= mask - 1;
        const int l1 = mask ? __ffsll(mask) - 1 : l0;
        if (mask) mask &= mask - 1;
        int bs[3];
        float w = 1.0f;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            bs[k] = (hi ? __builtin_amdgcn_readlane(b[k], l1) : __builtin_amdgcn_readlane(b[k], l0)) + o[k];
            w *= bspline_at(hi ? lane_f(f[k], l1) : lane_f(f[k], l0), (float)o[k]);
        }
        float t[12];
#pragma unroll
        for (int q = 0; q < 3; q++) t[q] = 0.0f;
        if (n < 27) {
            const long long idx = node_index(Sn, B, bs[0], bs[1], bs[2]);
            t[0] = w * a.gvx[idx];
            t[1] = w * a.gvy[idx];
            t[2] = w * a.gvz[idx];
        }
#pragma unroll
        for (int c = 0; c < 3; c++)
#pragma unroll
            for (int e = 0; e < 3; e++) t[3 + 3 * c + e] = (float)o[e] * t[c];
#pragma unroll
        for (int q = 0; q < 12; q++) {
            float r = t[q];                     // lanes 31 and 63 end with the sums of their halves
            r = dpp_add<0x111, 0xf>(r);
            r = dpp_add<0x112, 0xf>(r);
            r = dpp_add<0x114, 0xf>(r);
            r = dpp_add<0x118, 0xf>(r);
            r = dpp_add<0x142, 0xa>(r);
            const float s0 = lane_f(r, 31), s1 = lane_f(r, 63);
            float &dst = q < 3 ? vp[q] : So[(q - 3) / 3][(q - 3) % 3];
            dst = lane == l0 ? s0 : (lane == l1 ? s1 : dst);
        }
    }
}

// Rounding by addition: RND = 1.5 * 2^23, whose float spacing is 1 for sums in [2^23, 2^24).
constexpr float RND = 12582912.0f;
constexpr unsigned long long RND_PAIR = 0x4B4000004B400000ull;   // RND's bits in both halves

// Base cells a particle of a P2G tile can have (tile coordinates 0 .. tile_bmax).
template <int B> constexpr int p2g_cells() { return (tile_bmax<B>() + 1) * (tile_bmax<B>() + 1) * (tile_bmax<B>() + 1); }

// Items with more particles than this count their particles per base cell
// before scattering (below it the per-term limit already sets the scale).
constexpr int P2G_COUNT_MIN = 256;

// Power-of-two fixed-point scales of the P2G tile, keeping every node sum
// below 2^30: |contribution| <= w * bound with the weights of a node summing
// to at most wsum; and every single term within 2^22 (w <= 0.421875; rounded
// by the RND addition of scatter_packed).  A particle may be scattered into
// the tile while its scatter bound b satisfies b * sp <= lim.
struct TileScale {
    float msc;   // Sm m: mass-scaled weights
    float kd, km;   // kk dx and kk m with kk = Sp / (Sm m), the momentum scale relative to the mass-scaled weight
    float sp;    // Sp
    float lim;
    float im, ip;   // 1 / Sm, 1 / Sp
};

__device__ __forceinline__ TileScale tile_scale(const SceneK &K, float wsum, float bmax)
{
    TileScale ts;
    ts.lim = fminf(1073741824.0f / wsum, 4194304.0f / 0.421875f);
    int em = ilogbf(ts.lim / K.mass);
    em = min(max(em, -120), 120);
    int ep = bmax > 0.0f ? ilogbf(ts.lim / bmax) : 120;
    ep = min(max(ep, -120), 120);
    const float Sm = ldexpf(1.0f, em), Sp = ldexpf(1.0f, ep);
    const float kk = Sp / (Sm * K.mass);
    ts.kd = uniform_f(kk * K.dx);
    ts.km = uniform_f(kk * K.mass);
    ts.msc = Sm * K.mass;
    ts.sp = Sp;
    ts.im = 1.0f / Sm;
    ts.ip = 1.0f / Sp;
    return ts;
}

// One particle's 27 stencil terms into the tile t64 (per node two 64-bit sums,
// (p_x, m) and (p_y, p_z) as (hi, lo), each the exact sum of 32-bit fixed-point
// terms packed as hi * 2^32 + lo: an integer sum, so both halves are recovered
// exactly while they fit in 32 bits); tb0: the sums of the particle's base
// cell, f its offset from it in cells.
template <int B>
__device__ __forceinline__ void scatter_packed(long long *tb0, const float f[3], const TileScale &ts, const float v[3],
                                               const float A[9])
{
    constexpr int T = tile_edge<B>(), T3 = T * T * T;
    float wx[3], wy[3], wz[3];
    bspline_w(f[0], wx);
    bspline_w(f[1], wy);
    bspline_w(f[2], wz);
#pragma unroll
    for (int o = 0; o < 3; o++) wx[o] *= ts.msc;
    // r(o) = kk * (m v + A (o - f) dx); increments along each axis.  The roundings are written out (the
    // increments rounded before they are added, the order of the fused sum): left to the compiler they
    // follow the code around this function, and a last bit that turns here is 1e-3 of a network output
    // whose inputs are rounded to BF16
    float Ad[3][3], r0[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {
#pragma unroll
        for (int e = 0; e < 3; e++) {
#pragma clang fp contract(off)
            Ad[c][e] = ts.kd * A[3 * c + e];
        }
        r0[c] = fmaf(ts.km, v[c], -fmaf(Ad[c][2], f[2], fmaf(Ad[c][0], f[0], Ad[c][1] * f[1])));
    }
    // r at offset (ox, oy, oz): r0 + ox Ad_x + oy Ad_y + oz Ad_z, one add per axis step
    // (offset 0 adds nothing, 1 adds Ad, 2 adds 2 Ad)
    auto step = [](float r, float d, int o) { return o == 0 ? r : (o == 1 ? r + d : fmaf(2.0f, d, r)); };
#pragma unroll
    for (int ox = 0; ox < 3; ox++)
#pragma unroll
        for (int oy = 0; oy < 3; oy++) {
            float wxy = wx[ox] * wy[oy];
            float rxy[3];
#pragma unroll
            for (int c = 0; c < 3; c++) rxy[c] = step(step(r0[c], Ad[c][0], ox), Ad[c][1], oy);
#pragma unroll
            for (int oz = 0; oz < 3; oz++) {
                float w = wxy * wz[oz];
                int o = (ox * T + oy) * T + oz;
                // x + RND (|x| <= 2^22) holds round(x) in its low mantissa bits: bits = RND_BITS + round(x).
                // A pair of such bit patterns as hi * 2^32 + lo, minus RND_BITS * (2^32 + 1), is
                // round(x_hi) * 2^32 + round(x_lo) exactly (one 64-bit subtraction per pair).
                const unsigned b0 = __float_as_uint(fmaf(wxy, wz[oz], RND));   // mass term
                const unsigned b1 = __float_as_uint(fmaf(w, step(rxy[0], Ad[0][2], oz), RND));
                const unsigned b2 = __float_as_uint(fmaf(w, step(rxy[1], Ad[1][2], oz), RND));
                const unsigned b3 = __float_as_uint(fmaf(w, step(rxy[2], Ad[2][2], oz), RND));
                atomicAdd((unsigned long long *)(tb0 + o), ((unsigned long long)b1 << 32 | b0) - RND_PAIR);
                atomicAdd((unsigned long long *)(tb0 + T3 + o), ((unsigned long long)b2 << 32 | b3) - RND_PAIR);
            }
        }
}

// The tile's node sums into the global grid: marks the grid blocks that
// received mass, queues lower neighbour blocks off the update list.
template <int B, int NT>
__device__ void flush_packed(const GridOut &o, int s, const SceneDev &S, const int org[3], const long long *t64,
                             const TileScale &ts)
{
    constexpr int T = tile_edge<B>(), T3 = T * T * T;
    const int home[3] = {(org[0] + 1) / B, (org[1] + 1) / B, (org[2] + 1) / B};
    // neighbour blocks (home - 1 .. home + 1 per axis, bit (cx * 3 + cy) * 3 + cz) below the home
    // block along some axis that received mass: queued once per wave after the node loop (the
    // home block and its upper neighbours are on the update list already)
    unsigned lower = 0;
    // scene constants in registers: the grid atomics may alias the scene record for the
    // compiler, which would otherwise reload it (waiting for the atomics) on every node
    const int res = uniform_i(S.res), nb = uniform_i(S.nb), bin_off = uniform_i(S.bin_off);
    const SceneDev Sg = {0, 0, res, nb, uniform_ll(S.grid_off)};
    for (int n = threadIdx.x; n < T3; n += NT) {
        int m0, p0, p1, p2;
        unpack2(t64[n], p0, m0);
        unpack2(t64[T3 + n], p1, p2);
        if ((m0 | p0 | p1 | p2) == 0) continue;
        int tx = n / (T * T), ty = (n / T) % T, tz = n % T;
        int gi = org[0] + tx, gj = org[1] + ty, gk = org[2] + tz;
        if (gi < 0 || gj < 0 || gk < 0 || gi >= res || gj >= res || gk >= res) continue;
        const int lb = ((gi / B) * nb + (gj / B)) * nb + (gk / B);
        o.touched[bin_off + lb] = 1;
        if (tx == 0 || ty == 0 || tz == 0)
            lower |= 1u << (((gi / B - home[0] + 1) * 3 + (gj / B - home[1] + 1)) * 3 + (gk / B - home[2] + 1));
        const long long idx = node_index(Sg, B, gi, gj, gk);
        atomicAdd(o.gm + idx, (float)m0 * ts.im);
        atomicAdd(o.gpx + idx, (float)p0 * ts.ip);
        atomicAdd(o.gpy + idx, (float)p1 * ts.ip);
        atomicAdd(o.gpz + idx, (float)p2 * ts.ip);
    }
    lower = wave_or(lower);
    const int lane = threadIdx.x & 63;
    if (lane < 27 && ((lower >> lane) & 1u)) {
        const int lb = ((home[0] - 1 + lane / 9) * nb + (home[1] - 1 + (lane / 3) % 3)) * nb + (home[2] - 1 + lane % 3);
        queue_block(o, s, bin_off, lb);
    }
}

template <int B, int NT = WG>
__device__ void p2g_item(const StepArgs &a, int it, const Item &item, int *tile, int *cells)
{
    constexpr int T = tile_edge<B>(), T3 = T * T * T, NC = p2g_cells<B>();
    const int t = threadIdx.x;
    const int s = item.scene;
    const SceneDev &S = a.scenes[s];
    const int nb = S.nb;
    const int bx = item.block / (nb * nb), by = (item.block / nb) % nb, bz = item.block % nb;
    const int org[3] = {bx * B - 1, by * B - 1, bz * B - 1};
    const int3 home = make_int3(bx, by, bz);
    const SceneK K = scene_k(S);
    const TileBox box = tile_box(K, org, tile_bmax<B>());
    // largest particle count of a base cell, left by the G2P that moved the
    // particles (0 after a re-sort or a surrogate step: count here)
    const int known = item.count > P2G_COUNT_MIN ? a.L.icell[it] : 0;
    const bool count_cells = item.count > P2G_COUNT_MIN && known <= 0;

    // the first particle's state is in flight while the tile is cleared; the
    // next one's is loaded while the current one scatters
    float xn[3] = {}, vn[3] = {}, An[9] = {};
    if (t < item.count) load_particle_xvA(a, item.start + t, xn, vn, An);
    // LDS tile: per node two 64-bit sums, (p_x, m) and (p_y, p_z) as (hi, lo),
    // each the exact sum of 32-bit fixed-point terms packed as hi * 2^32 + lo
    // (an integer sum, so both halves are recovered exactly while they fit in
    // 32 bits)
    long long *t64 = (long long *)tile;
    for (int n = t; n < 2 * T3; n += NT) t64[n] = 0;
    if (count_cells) {
        for (int n = t; n < NC + 1; n += NT) cells[n] = 0;   // cells[NC]: the maximum
    }
    // bound of this item's particles, left by the previous G2P (or the sort)
    const float bmax = a.L.ibound[it];
    __syncthreads();
    if (t == 0 && !a.keep_bound && !a.chain) a.L.ibound[it] = 0.0f;   // this substep's G2P accumulates the next bound

    // Node sums of weights: a node receives w <= 0.5, 0.75, 0.5 per axis from
    // particles whose base cell is 0, 1, 2 cells below it, so the weights
    // reaching one node add up to at most 1.75^3 = 5.359375 times the largest
    // number of particles sharing a base cell (and never more than
    // 0.421875 * count).  Large items count their particles per base cell
    // first (the same in-tile test as the scatter below).
    float wsum = 0.421875f * (float)item.count;
    if (count_cells) {
        for (int base = 0; base < item.count; base += NT) {
            const int li = base + t;
            if (li >= item.count) break;
            const unsigned jo = (unsigned)(item.start + li) << 2;
            float x[3], fb[3], f[3];
#pragma unroll
            for (int d = 0; d < 3; d++) x[d] = pload(a.P, a.pstride, X0 + d, jo);
            if (tile_base(K, box, x, fb, f)) atomicAdd(cells + tile_index<tile_bmax<B>() + 1>(fb, org), 1);
        }
        __syncthreads();
        int mx = 0;
        for (int n = t; n < NC; n += NT) mx = max(mx, cells[n]);
        mx = wave_max_i(mx);
        if ((t & 63) == 0) atomicMax(cells + NC, mx);
        __syncthreads();
        if (a.chain && t == 0) a.L.icell[it] = cells[NC];   // the fused G2P's scale
        wsum = fminf(wsum, 5.359375f * (float)max(cells[NC], 1));
    } else if (known > 0) {
        wsum = fminf(wsum, 5.359375f * (float)known);
    }

    const TileScale ts = tile_scale(K, wsum, bmax);

    const int lane = t & 63;
    for (int k0 = t - lane; k0 < item.count; k0 += NT) {   // wave-uniform: the wave's next 64 particles
        const int li = k0 + lane;
        const bool act = li < item.count;
        float x[3], v[3], A[9], fb[3], f[3];
#pragma unroll
        for (int d = 0; d < 3; d++) {
            x[d] = xn[d];
            v[d] = vn[d];
        }
#pragma unroll
        for (int e = 0; e < 9; e++) A[e] = An[e];
        if (li + NT < item.count) load_particle_xvA(a, item.start + li + NT, xn, vn, An);
        const bool in = tile_base(K, box, x, fb, f);
        const unsigned long long slow = __ballot(act && !in);
        if (slow) {
            int bp[3] = {0, 0, 0}, cl = 0;
            float fp[3] = {0.0f, 0.0f, 0.0f};
            if (act && !in) {
#pragma unroll
                for (int d = 0; d < 3; d++) particle_base(K, x[d], bp[d], fp[d], cl);
                if (cl) atomicOr(a.flags + s, (int)FLAG_CLAMPED);
            }
            const GridOut o = grid_out(a.substep);
            if (__popcll(slow) <= COOP_LANES) p2g_global_wave<B>(o, s, S, slow, v, A, bp, fp, home);
            else if (act && !in) p2g_global<B>(o, s, S, v, A, bp, fp, home);
        }
        if (act && in) scatter_packed<B>(t64 + tile_index<T>(fb, org), f, ts, v, A);
    }
    const GridOut go = grid_out(a.substep);
    __syncthreads();
    flush_packed<B, NT>(go, s, S, org, t64, ts);
    __syncthreads();
}

template <int B, int NT>
__global__ __launch_bounds__(NT, 5) void k_p2g(StepArgs a)
{
    constexpr int T = tile_edge<B>(), T3 = T * T * T;
    __shared__ __align__(16) int tile[4 * T3];
    __shared__ int cells[p2g_cells<B>() + 1];
    const int n_items = *a.L.n_items;
    const int G = active_wgs(n_items);
    if ((int)blockIdx.x >= G) return;
    // items in dispatch order, most particles first (L.order)
    for (int r = blockIdx.x; r < n_items; r += G) {
        const int it = a.L.order[r];
        Item item = a.L.items[it];
        if (!a.active[item.scene]) continue;
        p2g_item<B, NT>(a, it, item, tile, cells);
    }
}

// ---------------------------------------------------------------- grid update
// cl: this wave's LDS copy of the scene's colliders (at most
// MAX_COLLIDERS_PER_SCENE).
// The node loop stores to the grid; reading the colliders and the scene
// constants from LDS and registers keeps the compiler from reloading them
// from global memory (and waiting for the stores) on every node.
// EXTRA = false: a plain substep (no capture, no surrogate arrays), built
// without that code so that it keeps its registers and occupancy.
template <int B, bool EXTRA = true>
__device__ void grid_block(const StepArgs &a, int s, int lb, int lane, ColliderNow *cl)
{
    const SceneDev &S = a.scenes[s];
    unsigned char *tf = a.L.touched + S.bin_off + lb;
    if (!*tf) return;          // no P2G wrote into this block: every (m, p) in it is zero
    const int nb = S.nb;
    const int bx = lb / (nb * nb), by = (lb / nb) % nb, bz = lb % nb;
    const int n_col = __builtin_amdgcn_readfirstlane(S.n_col);
    const int bound = __builtin_amdgcn_readfirstlane(S.bound);
    const SceneK K = scene_k(S);
    const float gdt[3] = {K.dt * uniform_f(S.g[0]), K.dt * uniform_f(S.g[1]), K.dt * uniform_f(S.g[2])};
    const long long goff = S.grid_off;
    {
        // this substep's collider poses, one lane per collider
        if (lane < n_col) {
            ColliderNow cn;
            collider_at(a.cols[S.col_off + lane], (float)a.substep * K.dt, cn);
            cl[lane] = cn;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // B^3 is a multiple of 64: every lane runs every iteration, so the wave sums of the
    // collider wrenches below see all lanes (a lane on an empty node adds zero)
    for (int l = lane; l < B * B * B; l += 64) {
        long long idx = goff + (long long)lb * (B * B * B) + l;
        float m = a.gm[idx], px = a.gpx[idx], py = a.gpy[idx], pz = a.gpz[idx];
        const bool live = !(m == 0.0f && px == 0.0f && py == 0.0f && pz == 0.0f);
        if (!__any(live)) continue;
        int ii[3] = {bx * B + l / (B * B), by * B + (l / B) % B, bz * B + l % B};
        if (EXTRA && a.cap && live) {
            long long c = a.cap_off[s] + ((long long)ii[0] * K.res + ii[1]) * K.res + ii[2];
            a.cap[4 * c] = m;
            a.cap[4 * c + 1] = px;
            a.cap[4 * c + 2] = py;
            a.cap[4 * c + 3] = pz;
        }
        float v[3] = {0.0f, 0.0f, 0.0f};
        if (m > 0.0f) {
            v[0] = px / m;
            v[1] = py / m;
            v[2] = pz / m;
        }
        for (int d = 0; d < 3; d++) v[d] += gdt[d];
        float xi[3] = {ii[0] * K.dx, ii[1] * K.dx, ii[2] * K.dx};
        for (int c = 0; c < (a.contact == 1 ? 0 : n_col); c++) {   // contact 1: particle penalty only
            const float v0[3] = {v[0], v[1], v[2]};
            const bool hit = collide_node(cl[c], xi, v, a.sdf) && live && m > 0.0f;
            // two-way coupling: the collider receives minus the momentum its projection gives
            // the node, and minus its moment about the collider centre; one wave sum and one
            // atomic per component, only where the wave touched this collider
            if (a.wrench && __any(hit)) {
                float dp[3], r[3];
                for (int d = 0; d < 3; d++) {
                    dp[d] = hit ? m * (v[d] - v0[d]) : 0.0f;
                    r[d] = xi[d] - cl[c].c[d];
                }
                const float w6[6] = {dp[0], dp[1], dp[2], r[1] * dp[2] - r[2] * dp[1], r[2] * dp[0] - r[0] * dp[2],
                                     r[0] * dp[1] - r[1] * dp[0]};
                float *acc = a.wrench + 6 * (long long)(S.col_off + c);
                float tot[6];
#pragma unroll
                for (int j = 0; j < 6; j++) tot[j] = wave_total(w6[j]);
                if (lane == 0)
#pragma unroll
                    for (int j = 0; j < 6; j++) atomicAdd(acc + j, -tot[j]);
            }
        }
        if (!live) continue;
        for (int d = 0; d < 3; d++) {
            if (ii[d] < bound && v[d] < 0.0f) v[d] = 0.0f;
            if (ii[d] >= K.res - bound && v[d] > 0.0f) v[d] = 0.0f;
        }
        const long long c = EXTRA && a.dense ? sur_index(a, s, K.res, ii[0], ii[1], ii[2]) : -1;
        if (EXTRA && a.dense && c < 0 && a.out_mass && m > 0.0f) atomicAdd(a.out_mass + s, m);   // outside the box
        if (EXTRA && c >= 0) {   // (m, p / m) of the P2G, before gravity, colliders and walls
            const float im = m > 0.0f ? 1.0f / m : 0.0f;
            *(float4 *)(a.dense + 4 * c) = make_float4(m, px * im, py * im, pz * im);
            if (a.feat) {
                const float inv = S.vol / (S.mass * S.dx * S.dx * S.dx);   // 1 / (rho dx^3)
                float *fp = a.feat + c * a.cf;
                fp[0] = m * inv;
                fp[1] = px * inv * (1.0f / SUR_VEL);
                fp[2] = py * inv * (1.0f / SUR_VEL);
                fp[3] = pz * inv * (1.0f / SUR_VEL);
            }
        }
        a.gvx[idx] = v[0];
        a.gvy[idx] = v[1];
        a.gvz[idx] = v[2];
        a.gm[idx] = 0.0f;
        a.gpx[idx] = 0.0f;
        a.gpy[idx] = 0.0f;
        a.gpz[idx] = 0.0f;
    }
    if (lane == 0) *tf = 0;
}

// The wave that takes the first static grid block of scene s also leaves the
// scene's collider poses of this substep in a.colnow for the G2P (penalty
// contact reads them there).
__device__ __forceinline__ void publish_colliders(const StepArgs &a, int w, int s, int lane)
{
    if (w != a.L.scene_gitem_begin[s]) return;
    const SceneDev &S = a.scenes[s];
    if (lane < S.n_col) {
        ColliderNow cn;
        collider_at(a.cols[S.col_off + lane], (float)a.substep * S.dt, cn);
        ((ColliderNow *)a.colnow)[S.col_off + lane] = cn;
    }
}

template <int B, bool EXTRA>
__global__ __launch_bounds__(WG, (B == 8 && !EXTRA) ? 7 : 1) void k_grid(StepArgs a)
{
    const int lane = threadIdx.x & 63;
    __shared__ ColliderNow cls[WG / 64][MAX_COLLIDERS_PER_SCENE];
    const int ng = *a.L.n_gitems;
    const int no = min(*ovf_count(a, a.substep), a.L.ovf_cap);
    const int G = active_wgs((ng + no + WG / 64 - 1) / (WG / 64));
    if ((int)blockIdx.x >= G) return;
    const int nw = G * (WG / 64);
    const int w0 = xcd_remap(blockIdx.x, G) * (WG / 64) + (threadIdx.x >> 6);
    for (int w = w0; w < ng + no; w += nw) {
        int2 e = w < ng ? a.L.gitems[w] : a.L.ovf[w - ng];
        if (w < ng) publish_colliders(a, w, e.x, lane);
        grid_block<B, EXTRA>(a, e.x, e.y, lane, cls[threadIdx.x >> 6]);
        if (w >= ng && lane == 0) a.L.bflag[a.scenes[e.x].bin_off + e.y] = 0;
    }
}

// ---------------------------------------------------------------- G2P + integration
// PEN: particle penalty contact after the position update (MPM_OPT_CONTACT 1 or 2).
// cells: LDS of p2g_cells<B>() + 1 ints; the item's particles are counted per
// base cell of their new position (as the next P2G's tile sees them) and the
// largest count is left in L.icell[it] for that P2G's fixed-point scale.
// FUSE: the P2G of substep a.substep + 1 follows in the same pass: each
// particle, once advanced, is scattered from registers into the fixed-point
// LDS tile t64 (as p2g_item's), which is flushed to the grid at the end of the
// item; only x and G are stored (v and A live on in the grid, and the G2P
// that ends the run of fused substeps stores them).  The tile's scale has to
// be fixed before any particle has moved, so it comes from the state this
// G2P starts from: the largest particle count of a base cell (L.icell) and
// the scatter bound (L.ibound, with 1/8 headroom).  Both stay bounds of the
// scattered state because a particle goes into the tile only if it kept its
// base cell (so no cell gains particles) and its bound stays within the
// scale; any other particle is scattered straight into the grid.  The item's
// L.ibound and L.icell are then replaced by those of the advanced state.
template <int B, bool PF, bool PEN, int NT = WG, bool FUSE = false>
__device__ void g2p_item(const StepArgs &a, int it, const Item &item, float *vt, float *pf, int *cells,
                         long long *t64 = nullptr)
{
    constexpr int T = tile_edge<B>(), T3 = T * T * T, NC = p2g_cells<B>();
    const int t = threadIdx.x;
    const int s = item.scene;
    const SceneDev &S = a.scenes[s];
    const int nb = S.nb;
    const int bx = item.block / (nb * nb), by = (item.block / nb) % nb, bz = item.block % nb;
    const int org[3] = {bx * B - 1, by * B - 1, bz * B - 1};
    const int3 home = make_int3(bx, by, bz);
    const long long ps = a.pstride;
    const int lane = t & 63;
    float *pw = PF ? pf + uniform_i(t >> 6) * (PF_COMPS * 64) : nullptr;
    // scene constants in registers before any copy into LDS (the copies may alias memory for
    // the compiler, which would reload them after each one)
    const Material mat = material_of(S);
    const SceneK K = scene_k(S);
    const TileBox box = tile_box(K, org, tile_bmax<B>());
    const SceneDev Sn = {0, 0, K.res, uniform_i(S.nb), uniform_ll(S.grid_off)};   // for node_index
    TileScale ts{};
    if (FUSE) {
        const int known = item.count > P2G_COUNT_MIN ? a.L.icell[it] : 0;
        float wsum = 0.421875f * (float)item.count;
        if (known > 0) wsum = fminf(wsum, 5.359375f * (float)known);
        // floor: 2^-20 of the momentum of a particle crossing a cell per substep (a state at rest
        // has bound 0)
        const float floor_b = 9.5367431640625e-7f * K.mass * K.dx / K.dt;
        ts = tile_scale(K, wsum, fmaxf(1.125f * a.L.ibound[it], floor_b));
        for (int n = t; n < 2 * T3; n += NT) t64[n] = 0;
    }
    for (int n = t; n < NC + 1; n += NT) cells[n] = 0;
    {
        const int res = Sn.res;
        // the wave's first 64 particles: x and G copied into LDS while the tile is staged
        if (PF) pf_issue(a.P, ps, item.start + (t - lane), item.count - (t - lane), lane, pw);
        // tile nodes copied straight into LDS, all in flight at once; nodes outside the grid are zeroed
        for (int n0 = t - lane; n0 < T3; n0 += NT) {
            const int n = n0 + lane;
            if (n >= T3) break;
            int gi = org[0] + n / (T * T), gj = org[1] + (n / T) % T, gk = org[2] + n % T;
            if (gi >= 0 && gj >= 0 && gk >= 0 && gi < res && gj < res && gk < res) {
                long long idx = node_index(Sn, B, gi, gj, gk);
                lds_copy(a.gvx + idx, vt + n0);
                lds_copy(a.gvy + idx, vt + T3 + n0);
                lds_copy(a.gvz + idx, vt + 2 * T3 + n0);
            } else {
                vt[n] = 0.0f;
                vt[T3 + n] = 0.0f;
                vt[2 * T3 + n] = 0.0f;
            }
        }
        wait_vmem();
    }
    __syncthreads();
    if (FUSE && t == 0) a.L.ibound[it] = 0.0f;   // read by every thread above; the advanced state's bound follows
    int bad_any = 0, cl_any = 0;
    float bnd = 0.0f;
    // penalty contact: this substep's collider poses of the scene (uniform), the per-lane sums of
    // the momentum and its moment given to the particles, and which colliders were touched
    const ColliderNow *cn = (const ColliderNow *)a.colnow + S.col_off;
    const int pen_ncol = PEN ? uniform_i(S.n_col) : 0;
    const float pen_rate = 0.25f / K.dt;
    float pacc[PEN ? MAX_COLLIDERS_PER_SCENE : 1][6] = {};
    unsigned pen_hit = 0;
    // wave-uniform loop: lane li = k0 + lane of each 64-particle batch
    for (int k0 = t - lane; k0 < item.count; k0 += NT) {
        const int li = k0 + lane;
        const unsigned jo = (unsigned)(item.start + li) << 2;
        float *const P = a.P;
        float x[3], G[9];
        if (PF) {
#pragma unroll
            for (int d = 0; d < 3; d++) x[d] = pw[d * 64 + lane];
#pragma unroll
            for (int e = 0; e < 9; e++) G[e] = pw[(3 + e) * 64 + lane];
            wait_lds();
            // the next batch streams into LDS while this one computes
            pf_issue(P, ps, item.start + k0 + NT, item.count - (k0 + NT), lane, pw);
        }
        const bool act = li < item.count;
        if (!PF && act) {
#pragma unroll
            for (int d = 0; d < 3; d++) x[d] = pload(P, ps, X0 + d, jo);
#pragma unroll
            for (int e = 0; e < 9; e++) G[e] = pload(P, ps, G00 + e, jo);
        }
        float fb[3], f[3], vp[3] = {0.0f, 0.0f, 0.0f};
        float So[3][3] = {{0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}};   // sum w v_c o_e
        const bool in = tile_base(K, box, x, fb, f);
        const unsigned long long out = __ballot(act && !in);
        const bool coop = __popcll(out) <= COOP_LANES;
        int b[3] = {0, 0, 0};
        if (out) {
            // outside the tile (drifted since the re-sort): the nodes straight from the grid
            if (act && !in) {
                int cl = 0;
#pragma unroll
                for (int d = 0; d < 3; d++) particle_base(K, x[d], b[d], f[d], cl);
                cl_any |= cl;
            }
            if (coop) gather_wave<B>(a, Sn, out, b, f, vp, So);
        }
        bool slow = false;          // scattered by the slow path below
        float fn[3], An[9];
        if (act) {
        float wx[3], wy[3], wz[3];
        bspline_w(f[0], wx);
        bspline_w(f[1], wy);
        bspline_w(f[2], wz);
        if (in) {
            // separable gather: reduce over z, then y, then x
            const float *vb = vt + tile_index<T>(fb, org);
            const float wz2 = 2.0f * wz[2], wy2 = 2.0f * wy[2], wx2 = 2.0f * wx[2];
#pragma unroll
            for (int ox = 0; ox < 3; ox++) {
                float A[3] = {0.0f, 0.0f, 0.0f}, By[3] = {0.0f, 0.0f, 0.0f}, Bz[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int oy = 0; oy < 3; oy++) {
                    const int o = (ox * T + oy) * T;
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        const float v0 = vb[c * T3 + o], v1 = vb[c * T3 + o + 1], v2 = vb[c * T3 + o + 2];
                        const float az = fmaf(wz[0], v0, fmaf(wz[1], v1, wz[2] * v2));
                        const float bzv = fmaf(wz[1], v1, wz2 * v2);
                        A[c] = fmaf(wy[oy], az, A[c]);
                        if (oy == 1) By[c] = fmaf(wy[1], az, By[c]);
                        if (oy == 2) By[c] = fmaf(wy2, az, By[c]);
                        Bz[c] = fmaf(wy[oy], bzv, Bz[c]);
                    }
                }
#pragma unroll
                for (int c = 0; c < 3; c++) {
                    vp[c] = fmaf(wx[ox], A[c], vp[c]);
                    if (ox == 1) So[c][0] = fmaf(wx[1], A[c], So[c][0]);
                    if (ox == 2) So[c][0] = fmaf(wx2, A[c], So[c][0]);
                    So[c][1] = fmaf(wx[ox], By[c], So[c][1]);
                    So[c][2] = fmaf(wx[ox], Bz[c], So[c][2]);
                }
            }
        } else if (!coop) {
            // the nodes straight from the grid, with the scene constants in registers (the particle stores may
            // alias the scene record for the compiler, which would reload it and wait for them)
#pragma unroll 1
            for (int q = 0; q < 9; q++) {
                const int ox = q / 3, oy = q % 3;
                float g[3][3];
#pragma unroll
                for (int oz = 0; oz < 3; oz++) {
                    const long long idx = node_index(Sn, B, b[0] + ox, b[1] + oy, b[2] + oz);
                    g[oz][0] = a.gvx[idx];
                    g[oz][1] = a.gvy[idx];
                    g[oz][2] = a.gvz[idx];
                }
                const float wxy = bspline_at(f[0], (float)ox) * bspline_at(f[1], (float)oy);
#pragma unroll
                for (int oz = 0; oz < 3; oz++) {
                    const float w = wxy * wz[oz];
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        const float tv = w * g[oz][c];
                        vp[c] += tv;
                        So[c][0] += (float)ox * tv;
                        So[c][1] += (float)oy * tv;
                        So[c][2] += (float)oz * tv;
                    }
                }
            }
        }
        // C = (4/dx^2) sum w v (x_i - x_p)^T = (4/dx) (So - vp f^T)
        const float Dd = 4.0f * K.inv_dx;
        float C[9];
#pragma unroll
        for (int c = 0; c < 3; c++)
#pragma unroll
            for (int e = 0; e < 3; e++) C[3 * c + e] = Dd * fmaf(-vp[c], f[e], So[c][e]);
#pragma unroll
        for (int d = 0; d < 3; d++) x[d] = fmaf(K.dt, vp[d], x[d]);
        // base cell of the new position in this item's P2G tile: the same one as before for all but
        // a few particles of a substep
        float fbn[3];
        const bool inn = tile_base(K, box, x, fbn, fn);
        const bool kept = in && fbn[0] == fb[0] && fbn[1] == fb[1] && fbn[2] == fb[2];
        if (inn) atomicAdd(cells + tile_index<tile_bmax<B>() + 1>(fbn, org), 1);
        if (PEN) {
            // inside collider c at the new position: v += -phi n / (4 dt), a spring of stiffness
            // m / (4 dt^2) along the outward normal (the stored v, hence the next scatter bound,
            // includes it)
#pragma unroll
            for (int c = 0; c < (PEN ? MAX_COLLIDERS_PER_SCENE : 1); c++) {
                if (c >= pen_ncol) break;
                float nrm[3];
                const float phi = sdf_eval(cn[c], x, nrm, a.sdf);
                if (phi < 0.0f) {
                    float dp[3], r[3];
#pragma unroll
                    for (int d = 0; d < 3; d++) {
                        const float dv = -phi * pen_rate * nrm[d];
                        vp[d] += dv;
                        dp[d] = K.mass * dv;
                        r[d] = x[d] - cn[c].c[d];
                    }
                    pacc[c][0] += dp[0];
                    pacc[c][1] += dp[1];
                    pacc[c][2] += dp[2];
                    pacc[c][3] += r[1] * dp[2] - r[2] * dp[1];
                    pacc[c][4] += r[2] * dp[0] - r[0] * dp[2];
                    pacc[c][5] += r[0] * dp[1] - r[1] * dp[0];
                    pen_hit |= 1u << c;
                }
            }
        }
        // F <- (I + dt C) F  ->  G <- G + dt C + dt C G
        float Gt[9];
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                float acc = C[3 * i + k];
#pragma unroll
                for (int e = 0; e < 3; e++) acc = fmaf(C[3 * i + e], G[3 * e + k], acc);
                Gt[3 * i + k] = fmaf(K.dt, acc, G[3 * i + k]);
            }
        float tau[9], Gn[9];
        int bad = 0;
        if (mat.model == 0) {
            tau_neo_hookean(Gt, mat.mu, mat.la, tau, bad);
#pragma unroll
            for (int e = 0; e < 9; e++) Gn[e] = Gt[e];
        } else if (mat.model == 2) {
            fluid_update(Gt, mat, Gn, tau, bad);
        } else {
            hencky_update<!FUSE>(Gt, mat, Gn, tau, bad);
        }
        bad |= !(isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]));
        bad_any |= bad;
        // the prefetch has had the whole computation to land; waiting here (not at
        // the top of the next batch) keeps the wait off this batch's stores (lane 0 of a wave is
        // active in every batch, so the wave always waits)
        if (PF) wait_vmem();
#pragma unroll
        for (int d = 0; d < 3; d++) {
            pstore(P, ps, X0 + d, jo, x[d]);
            if (!FUSE) pstore(P, ps, V0 + d, jo, vp[d]);
        }
#pragma unroll
        for (int e = 0; e < 9; e++) {
            An[e] = fmaf(K.mass, C[e], -K.kstress * tau[e]);
            if (!FUSE) pstore(P, ps, A00 + e, jo, An[e]);
            pstore(P, ps, G00 + e, jo, Gn[e]);
        }
        // a non-finite v or A (the next P2G would scatter it as garbage)
        const float sb = scatter_bound(K.mass, K.dx, vp, An);
        bad_any |= !(sb <= 3.0e38f);
        bnd = fmaxf(bnd, sb);
        if (FUSE) {
            slow = !(kept && sb * ts.sp <= ts.lim);
        }
        }   // act
        if (FUSE) {
            const unsigned long long sm = __ballot(slow);
            if (sm) {
                int bn[3] = {0, 0, 0}, cln = 0;
                float fs[3] = {0.0f, 0.0f, 0.0f};
                if (slow)
#pragma unroll
                    for (int d = 0; d < 3; d++) particle_base(K, x[d], bn[d], fs[d], cln);
                const GridOut o = grid_out(a.substep + 1);
                if (__popcll(sm) <= COOP_LANES) p2g_global_wave<B>(o, s, S, sm, vp, An, bn, fs, home);
                else if (slow) p2g_global<B>(o, s, S, vp, An, bn, fs, home);
            }
            if (act && !slow) scatter_packed<B>(t64 + tile_index<T>(fb, org), fn, ts, vp, An);
        }
    }
    const GridOut go = grid_out(a.substep + 1);   // on its way while the wave finishes
    bnd = wave_max(bnd);
    if ((t & 63) == 0 && bnd > 0.0f) atomicMax((int *)(a.L.ibound + it), __float_as_int(bnd));
    if (PEN && a.wrench) {
        // the colliders receive minus what the penalty gave the particles: one wave sum and
        // one atomic per component, for the colliders a lane of the wave touched
#pragma unroll
        for (int c = 0; c < (PEN ? MAX_COLLIDERS_PER_SCENE : 1); c++) {
            if (c >= pen_ncol) break;
            if (!__any((pen_hit >> c) & 1u)) continue;
            float tot[6];
#pragma unroll
            for (int j = 0; j < 6; j++) tot[j] = wave_total(pacc[c][j]);
            if ((t & 63) == 0)
#pragma unroll
                for (int j = 0; j < 6; j++) atomicAdd(a.wrench + 6 * (long long)(S.col_off + c) + j, -tot[j]);
        }
    }
    if (bad_any) atomicOr(a.flags + s, (int)FLAG_NONFINITE);
    if (cl_any) atomicOr(a.flags + s, (int)FLAG_CLAMPED);
    __syncthreads();
    if (FUSE) flush_packed<B, NT>(go, s, S, org, t64, ts);
    int mx = 0;
    for (int n = t; n < NC; n += NT) mx = max(mx, cells[n]);
    mx = wave_max_i(mx);
    if ((t & 63) == 0) atomicMax(cells + NC, mx);
    __syncthreads();
    if (t == 0) a.L.icell[it] = cells[NC];
}

template <int B, bool PEN, int NT>
__global__ __launch_bounds__(NT, 4) void k_g2p(StepArgs a)
{
    constexpr int T = tile_edge<B>(), T3 = T * T * T;
    __shared__ float vt[3 * T3];
    __shared__ float pf[(NT / 64) * PF_COMPS * 64];
    __shared__ int cells[p2g_cells<B>() + 1];
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicExch(ovf_count(a, a.substep), 0);   // consumed by the grid update
    const int n_items = *a.L.n_items;
    const int G = active_wgs(n_items);
    if ((int)blockIdx.x >= G) return;
    for (int r = blockIdx.x; r < n_items; r += G) {   // most particles first (L.order)
        const int it = a.L.order[r];
        Item item = a.L.items[it];
        if (!a.active[item.scene]) continue;
        g2p_item<B, true, PEN, NT>(a, it, item, vt, pf, cells);
    }
}

// G2P of substep a.substep fused with the P2G of substep a.substep + 1 (one
// pass over the particles; the grid update sits between two such launches).
// LDS: the velocity tile, the fixed-point tile and the base-cell counts (40 KB
// at block edge 8: four workgroups of 256 threads per CU).  x and G go straight
// into registers: the LDS prefetch slices of k_g2p would cost a workgroup per
// CU (measured 2.5 % slower on the 256-scene workload, 1.6 % on the heap).
// With penalty contact the kernel needs more registers than four workgroups
// leave, and keeps the prefetch.
// Bound by vector instructions (83 to 87 % of the cycles issue one at 256
// scenes): what it gained came from fewer of them, the strain series in scalar
// invariants and the wave-wide slow paths (100 substeps of 256 scenes, 7.7
// million particles, 44.1 -> 40.5 ms; 50 of 23 scenes 2.84 -> 2.52 ms).
template <int B, bool PEN, int NT>
__global__ __launch_bounds__(NT, 4) void k_g2p2g(StepArgs a)
{
    constexpr int T = tile_edge<B>(), T3 = T * T * T;
    __shared__ float vt[3 * T3];
    __shared__ float pf[PEN ? (NT / 64) * PF_COMPS * 64 : 1];
    __shared__ __align__(16) long long t64[2 * T3];
    __shared__ int cells[p2g_cells<B>() + 1];
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicExch(ovf_count(a, a.substep), 0);   // consumed by the grid update
    const int n_items = *a.L.n_items;
    const int G = active_wgs(n_items);
    if ((int)blockIdx.x >= G) return;
    for (int r = blockIdx.x; r < n_items; r += G) {   // most particles first (L.order)
        const int it = a.L.order[r];
        Item item = a.L.items[it];
        if (!a.active[item.scene]) continue;
        g2p_item<B, PEN, PEN, NT, true>(a, it, item, vt, pf, cells, t64);
    }
}

template <int NT>
static void launch_g2p2g_nt(const StepArgs &a, int n_wg, hipStream_t st)
{
    const bool pen = a.contact != 0;
    if (a.B == 4) {
        if (pen) launch_timed(k_g2p2g<4, true, NT>, n_wg, NT, st, a);
        else launch_timed(k_g2p2g<4, false, NT>, n_wg, NT, st, a);
    } else {
        if (pen) launch_timed(k_g2p2g<8, true, NT>, n_wg, NT, st, a);
        else launch_timed(k_g2p2g<8, false, NT>, n_wg, NT, st, a);
    }
}

hipError_t launch_g2p2g(const StepArgs &a, int n_wg, hipStream_t st)
{
    if (a.nt == 512) n_wg /= 2;
    n_wg = (n_wg + 7) & ~7;
    if (a.nt == 512) launch_g2p2g_nt<512>(a, n_wg, st);
    else launch_g2p2g_nt<WG>(a, n_wg, st);
    return hipGetLastError();
}

hipError_t launch_p2g(const StepArgs &a, int chunk, int n_wg, hipStream_t st)
{
    (void)chunk;
    if (a.nt == 512) n_wg /= 2;   // the same threads in workgroups of twice the size
    n_wg = (n_wg + 7) & ~7;
    if (a.nt == 512) {
        if (a.B == 4) launch_timed(k_p2g<4, 512>, n_wg, 512, st, a);
        else launch_timed(k_p2g<8, 512>, n_wg, 512, st, a);
    } else {
        if (a.B == 4) launch_timed(k_p2g<4, WG>, n_wg, WG, st, a);
        else launch_timed(k_p2g<8, WG>, n_wg, WG, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_grid(const StepArgs &a, int n_wg, hipStream_t st)
{
    n_wg = (n_wg + 7) & ~7;
    const bool extra = a.cap || a.dense;
    if (a.B == 4) {
        if (extra) launch_timed(k_grid<4, true>, n_wg, WG, st, a);
        else launch_timed(k_grid<4, false>, n_wg, WG, st, a);
    } else {
        if (extra) launch_timed(k_grid<8, true>, n_wg, WG, st, a);
        else launch_timed(k_grid<8, false>, n_wg, WG, st, a);
    }
    return hipGetLastError();
}

template <int NT>
static void launch_g2p_nt(const StepArgs &a, int n_wg, hipStream_t st)
{
    const bool pen = a.contact != 0;
    if (a.B == 4) {
        if (pen) launch_timed(k_g2p<4, true, NT>, n_wg, NT, st, a);
        else launch_timed(k_g2p<4, false, NT>, n_wg, NT, st, a);
    } else {
        if (pen) launch_timed(k_g2p<8, true, NT>, n_wg, NT, st, a);
        else launch_timed(k_g2p<8, false, NT>, n_wg, NT, st, a);
    }
}

hipError_t launch_g2p(const StepArgs &a, int n_wg, hipStream_t st)
{
    if (a.nt == 512) n_wg /= 2;   // the same threads in workgroups of twice the size
    n_wg = (n_wg + 7) & ~7;
    if (a.nt == 512) launch_g2p_nt<512>(a, n_wg, st);
    else launch_g2p_nt<WG>(a, n_wg, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------- one-launch substep
// One cooperative launch per substep over all scenes: every workgroup is
// resident at once (the launch is sized from the kernel's occupancy and the
// runtime refuses a larger one), and the three phases of the substep are
// separated by grid-wide barriers: P2G over all work items, the grid update
// over every listed block (one wave per block), G2P over all work items.
// Within a phase the workgroups stride over the work as the separate kernels
// do.  The phases share one LDS allocation (the P2G tile, or the G2P
// velocity tile and prefetch slices).
template <int B, bool PEN>
__global__ __launch_bounds__(WG, 4) void k_substep_coop(StepArgs a)
{
    constexpr int T = tile_edge<B>(), T3 = T * T * T;
    constexpr int P2G_WORDS = 4 * T3;
    constexpr int G2P_WORDS = 3 * T3 + (WG / 64) * PF_COMPS * 64;
    __shared__ __align__(16) int smem[P2G_WORDS > G2P_WORDS ? P2G_WORDS : G2P_WORDS];
    __shared__ int cells[p2g_cells<B>() + 1];
    __shared__ ColliderNow cls[WG / 64][MAX_COLLIDERS_PER_SCENE];
    cooperative_groups::grid_group grid = cooperative_groups::this_grid();
    const int G = gridDim.x;   // a multiple of 8: every workgroup takes part in every phase
    const int n_items = *a.L.n_items;
    // P2G, items in reverse order: the G2P of the previous substep walked them forward, so the
    // particles it wrote last are still in the memory-side cache
    for (int r = xcd_remap(blockIdx.x, G); r < n_items; r += G) {
        const int it = n_items - 1 - r;
        const Item item = a.L.items[it];
        if (!a.active[item.scene]) continue;
        p2g_item<B, WG>(a, it, item, smem, cells);
    }
    grid.sync();
    {
        const int lane = threadIdx.x & 63;
        const int ng = *a.L.n_gitems;
        const int no = min(*ovf_count(a, a.substep), a.L.ovf_cap);
        const int nw = G * (WG / 64);
        const int w0 = xcd_remap(blockIdx.x, G) * (WG / 64) + (threadIdx.x >> 6);
        for (int w = w0; w < ng + no; w += nw) {
            const int2 e = w < ng ? a.L.gitems[w] : a.L.ovf[w - ng];
            if (w < ng) publish_colliders(a, w, e.x, lane);
            grid_block<B, false>(a, e.x, e.y, lane, cls[threadIdx.x >> 6]);
            if (w >= ng && lane == 0) a.L.bflag[a.scenes[e.x].bin_off + e.y] = 0;
        }
    }
    grid.sync();
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicExch(ovf_count(a, a.substep), 0);   // consumed by the grid update
    float *vt = (float *)smem;
    for (int it = xcd_remap(blockIdx.x, G); it < n_items; it += G) {
        const Item item = a.L.items[it];
        if (!a.active[item.scene]) continue;
        g2p_item<B, true, PEN, WG>(a, it, item, vt, vt + 3 * T3, cells);
    }
}

// Workgroups of the cooperative substep (a multiple of 8): at most what can
// be resident at once (the kernel's occupancy), and no more per CU than
// per_cu_cap.  Each grid-wide barrier costs about 0.1 us per workgroup on
// MI355X (cfg2, one 65,536-particle scene: 94 / 146 / 260 us per substep
// at 1 / 2 / 4 workgroups per CU), so small problems take fewer; 0 on error.
template <int B, bool PEN>
static int coop_workgroups(int cus, int per_cu_cap)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_substep_coop<B, PEN>, WG, 0) != hipSuccess) return 0;
    per_cu = min(per_cu, max(per_cu_cap, 1));
    return (per_cu * cus) & ~7;
}

hipError_t launch_persistent(const StepArgs &a, int cus, int per_cu_cap, hipStream_t st)
{
    const bool pen = a.contact != 0;
    const void *fn;
    int G;
    if (a.B == 4) {
        fn = pen ? (const void *)k_substep_coop<4, true> : (const void *)k_substep_coop<4, false>;
        G = pen ? coop_workgroups<4, true>(cus, per_cu_cap) : coop_workgroups<4, false>(cus, per_cu_cap);
    } else {
        fn = pen ? (const void *)k_substep_coop<8, true> : (const void *)k_substep_coop<8, false>;
        G = pen ? coop_workgroups<8, true>(cus, per_cu_cap) : coop_workgroups<8, false>(cus, per_cu_cap);
    }
    if (G <= 0) return hipErrorInvalidConfiguration;
    StepArgs args = a;
    void *params[] = {(void *)&args};
    return hipLaunchCooperativeKernel(fn, dim3(G), dim3(WG), params, 0, st);
}

// ====================================================================== colliders
__global__ void k_collider_advance(ColliderDev *cols, int n, const int *col_scene, const SceneDev *scenes, int steps)
{
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    ColliderDev &cd = cols[c];
    float tk = (float)steps * scenes[col_scene[c]].dt;
    float q[4];
    quat_advance(cd.quat, cd.omega, tk, q);
    for (int d = 0; d < 3; d++) cd.pos[d] = fmaf(tk, cd.vlin[d], cd.pos[d]);
    for (int d = 0; d < 4; d++) cd.quat[d] = q[d];
}

hipError_t launch_collider_advance(ColliderDev *cols, int n_cols, const int *col_scene, const SceneDev *scenes,
                                   int n_substeps, hipStream_t st)
{
    if (n_cols > 0) k_collider_advance<<<(n_cols + 63) / 64, 64, 0, st>>>(cols, n_cols, col_scene, scenes, n_substeps);
    return hipGetLastError();
}

// ====================================================================== boundary conversions
size_t collider_now_bytes() { return sizeof(ColliderNow); }

__global__ void k_wrench_out(const SceneDev *scenes, int n_scenes, int max_col, float *acc, float *out)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;   // (scene, slot, component)
    if (e >= n_scenes * max_col * 6) return;
    const int s = e / (max_col * 6), k = (e / 6) % max_col, j = e % 6;
    const SceneDev &S = scenes[s];
    float val = 0.0f;
    if (k < S.n_col) {
        float *p = acc + 6 * (long long)(S.col_off + k) + j;
        val = *p;
        *p = 0.0f;
    }
    out[e] = val;
}

hipError_t launch_wrench_out(const SceneDev *scenes, int n_scenes, int max_col, float *acc, float *out, hipStream_t st)
{
    const int n = n_scenes * max_col * 6;
    if (n > 0) k_wrench_out<<<(n + 255) / 256, 256, 0, st>>>(scenes, n_scenes, max_col, acc, out);
    return hipGetLastError();
}

// Copies n floats that a workgroup's particles hold in a row, coalesced whatever the base's alignment.
__device__ __forceinline__ void stage_rows(const float *src, float *lds, int n)
{
    for (int q = threadIdx.x; q < n; q += WG) lds[q] = src[q];
}

// Bound by memory (96 B in, 100 B out a particle).  The rows of 3 and 9 floats
// go through LDS (odd strides: no bank conflicts), so that each load instruction
// of a wave takes 256 bytes in a row instead of every 36th (7.7 million
// particles: 590 -> 460 us, at a copy's rate 290).
__global__ __launch_bounds__(WG) void k_init_particles(const SceneDev *scenes, const int *psc, float *P,
                                                       long long ps, const float *x, const float *v, const float *C,
                                                       const float *F, int begin, int end, int *flags)
{
    __shared__ float lx[3 * WG], lv[3 * WG], lC[9 * WG], lF[9 * WG];
    const int i0 = begin + blockIdx.x * WG, n = min(WG, end - i0);
    const long long k0 = i0 - begin;
    stage_rows(x + 3 * k0, lx, 3 * n);
    if (v) stage_rows(v + 3 * k0, lv, 3 * n);
    if (C) stage_rows(C + 9 * k0, lC, 9 * n);
    if (F) stage_rows(F + 9 * k0, lF, 9 * n);
    __syncthreads();
    const int t = threadIdx.x, i = i0 + t;
    if (t >= n) return;
    float xr[3], vr[3], Cr[9], Fr[9];
#pragma unroll
    for (int d = 0; d < 3; d++) {
        xr[d] = lx[3 * t + d];
        vr[d] = v ? lv[3 * t + d] : 0.0f;
    }
#pragma unroll
    for (int e = 0; e < 9; e++) {
        Cr[e] = C ? lC[9 * t + e] : 0.0f;
        Fr[e] = F ? lF[9 * t + e] : (e % 4 == 0 ? 1.0f : 0.0f);
    }
    init_particle(scenes, psc[i], xr, vr, Cr, Fr, P, ps, i, i, flags);
}

hipError_t launch_init_particles(const SceneDev *scenes, int n_scenes, const int *psc, float *P, long long pstride,
                                 const float *x, const float *v, const float *C, const float *F, int begin, int end,
                                 int *flags, hipStream_t st)
{
    (void)n_scenes;
    if (end > begin)
        k_init_particles<<<(end - begin + WG - 1) / WG, WG, 0, st>>>(scenes, psc, P, pstride, x, v, C, F, begin, end, flags);
    return hipGetLastError();
}

// A row of N floats in the widest stores that a 4-byte alignment allows.
template <int N>
__device__ __forceinline__ void store_row(float *dst, const float (&r)[N])
{
    __builtin_memcpy(dst, r, sizeof(r));
}

// Slot order to creation order.  Bound by memory (100 B in, 96 B out a
// particle): each particle's rows go to its own place in the caller's arrays, a
// part of a cache line, so a contiguous share of the slots per XCD keeps a
// scene's lines in one L2 until its other particles have filled them, and all
// loads come before the stores, which the compiler cannot tell apart from them
// (7.7 million particles: 2010 -> 740 us, at a copy's rate 290; taking the caller's
// arrays directly saves 890 us of copies more).
__global__ __launch_bounds__(WG) void k_get_state(const SceneDev *scenes, const int *psc, const float *P, long long ps,
                                                  int begin, int end, float *x, float *v, float *C, float *F)
{
    const int j = begin + xcd_remap(blockIdx.x, gridDim.x) * WG + threadIdx.x;
    if (j >= end) return;
    const long long k = __float_as_int(P[PID * ps + j]) - begin;
    const SceneDev &S = scenes[psc[j]];
    float xr[3], vr[3], G[9], A[9];
#pragma unroll
    for (int d = 0; d < 3; d++) xr[d] = P[(X0 + d) * ps + j];
    if (v)
#pragma unroll
        for (int d = 0; d < 3; d++) vr[d] = P[(V0 + d) * ps + j];
#pragma unroll
    for (int e = 0; e < 9; e++) G[e] = P[(G00 + e) * ps + j];
    if (C) {
#pragma unroll
        for (int e = 0; e < 9; e++) A[e] = P[(A00 + e) * ps + j];
        const Material mat = material_of(S);
        const float mass = S.mass, kstress = S.kstress;
        float tau[9];
        int bad = 0;
        state_stress(G, mat, tau, bad);
#pragma unroll
        for (int e = 0; e < 9; e++) A[e] = fmaf(kstress, tau[e], A[e]) / mass;
        store_row(C + 9 * k, A);
    }
    if (x) store_row(x + 3 * k, xr);
    if (v) store_row(v + 3 * k, vr);
    if (F) {
#pragma unroll
        for (int e = 0; e < 9; e++) G[e] += (e % 4 == 0 ? 1.0f : 0.0f);
        store_row(F + 9 * k, G);
    }
}

hipError_t launch_get_state(const SceneDev *scenes, const int *psc, const float *P, long long pstride, int begin,
                            int end, float *x, float *v, float *C, float *F, hipStream_t st)
{
    const int g = (((end - begin + WG - 1) / WG) + 7) & ~7;   // xcd_remap needs a multiple of 8 workgroups
    if (end > begin) k_get_state<<<g, WG, 0, st>>>(scenes, psc, P, pstride, begin, end, x, v, C, F);
    return hipGetLastError();
}

__global__ void k_clear_f(float *p, long long n)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long st = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += st) p[i] = 0.0f;
}

hipError_t launch_clear_f(float *p, long long n, hipStream_t st)
{
    if (n > 0) {
        long long nb = (n + WG - 1) / WG;
        k_clear_f<<<(unsigned)(nb < 8192 ? nb : 8192), WG, 0, st>>>(p, n);
    }
    return hipGetLastError();
}

__global__ void k_fill_i(int *p, long long n, int v)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t launch_fill_i(int *p, long long n, int v, hipStream_t st)
{
    if (n > 0) {
        long long nb = (n + WG - 1) / WG;
        k_fill_i<<<(unsigned)(nb < 4096 ? nb : 4096), WG, 0, st>>>(p, n, v);
    }
    return hipGetLastError();
}

}  // namespace mpm
