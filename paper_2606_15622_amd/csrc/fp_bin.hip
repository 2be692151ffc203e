// fp_bin.hip -- stable counting sort of particles by cell key.
//
// Particles arrive in the order of the previous sort, so a wave of 64 consecutive
// particles carries only a handful of distinct destination keys.  Each wave folds its
// lanes by key (ballot) into "contributions" (source wave, 64-bit lane mask), one
// integer atomic per distinct key.  A destination cell then orders its contributions
// by source wave, which reproduces the order of a stable counting sort exactly,
// expands them to source indices in LDS and gathers the particle records.  No float
// atomics, no global radix passes; the result is deterministic.
#include "fp_mom_dev.h"
#include "fp_sample_dev.h"

#include <type_traits>

namespace fpg {

constexpr int BIN_BLOCK = 256;

// PLACE = false: count particles and contributions per key: cpair[k] holds both counts
// (particles in its low word, contributions in its high word), so one 64-bit atomic adds
// a contribution.
// PLACE = true:  write the contribution records at their slots.
template <bool PLACE>
__global__ __launch_bounds__(BIN_BLOCK) void bin_wave_kernel(
    const int32_t* __restrict__ key, int64_t n, const int64_t* __restrict__ n_dev, int32_t ncell,
    unsigned long long* __restrict__ cpair, int32_t* __restrict__ ccur,
    const int32_t* __restrict__ coff, int32_t* __restrict__ cwave, uint64_t* __restrict__ cmask,
    unsigned long long* __restrict__ errcount) {
    if (n_dev) n = *n_dev;   // the count kept on the device (the grid covers the slots)
    const int64_t p = (int64_t)blockIdx.x * BIN_BLOCK + threadIdx.x;
    const int32_t wave = (int32_t)(p >> 6);
    const int lane = threadIdx.x & 63;
    const bool valid = p < n;
    int32_t k = -1;
    if (valid) {
        k = key[p];
        if (k < 0 || k > ncell) {
            if (!PLACE) atomicAdd(errcount, 1ull);
            k = ncell;  // dropped
        }                // k == ncell: deleted particle, dropped
    }
    // the lanes of each distinct key: its lowest lane leads and keeps the mask; the leaders'
    // atomics then go out together (one round trip per wave, not one per key in turn)
    uint64_t active = __ballot(valid), mine = 0;
    while (active) {
        const int leader = __builtin_ctzll(active);
        const int32_t kl = __builtin_amdgcn_readlane(k, leader);
        const uint64_t m = __ballot(valid && k == kl);
        if (lane == leader) mine = m;
        active &= ~m;
    }
    if (mine && k < ncell) {
        if (PLACE) {
            const int32_t slot = coff[k] + atomicAdd(&ccur[k], 1);
            cwave[slot] = wave;
            cmask[slot] = mine;
        } else {
            atomicAdd(&cpair[k], (1ull << 32) | (unsigned long long)__popcll(mine));
        }
    }
}

// ---- exclusive scan of two int arrays of length len (ends written at [len]) ------------
// Two kernels: the tiles' totals, then every workgroup adds up the totals before its own tile
// and scans the tile.  Tiles are small (four items a thread: 196 workgroups for 2e5 cells
// instead of 49 of 16 items) while the totals stay few enough to be added up by everyone:
// 4.7 + 4.9 us at 2e5 cells, where 16 items and a kernel between for the totals took
// 13.2 + 4.6 + 10.4.
constexpr int SCAN_BLOCK = 256, SCAN_MAX = 8191, SCAN_MAX_CELLS = SCAN_MAX * SCAN_BLOCK * 16;

template <int BLOCK, int N>
__device__ __forceinline__ void wg_excl_scan_n(int32_t (&v)[N], int32_t (*sh)[N], int32_t (&total)[N]);

// a[j st], b[j st]: two arrays, or (st = 2) the two words of interleaved pairs
template <int ITEMS>
__global__ __launch_bounds__(SCAN_BLOCK) void scan_reduce_kernel(
    const int32_t* __restrict__ a, const int32_t* __restrict__ b, int32_t st, int32_t len,
    int32_t* __restrict__ bsum) {
    __shared__ int32_t sh[2][SCAN_BLOCK / 64];
    const int64_t base = (int64_t)blockIdx.x * (SCAN_BLOCK * ITEMS);
    int32_t sa = 0, sb = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t j = base + (int64_t)i * SCAN_BLOCK + threadIdx.x;
        if (j < len) {
            sa += a[j * st];
            sb += b[j * st];
        }
    }
    sa = group_sum_i<64>(sa);
    sb = group_sum_i<64>(sb);
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = sa;
        sh[1][threadIdx.x >> 6] = sb;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        int32_t t = 0;
#pragma unroll
        for (int w = 0; w < SCAN_BLOCK / 64; ++w) t += sh[threadIdx.x][w];
        bsum[8192 * threadIdx.x + blockIdx.x] = t;
    }
}

// item-contiguous per thread: thread t owns ITEMS consecutive elements of the tile
template <int ITEMS>
__global__ __launch_bounds__(SCAN_BLOCK) void scan_final_kernel(
    const int32_t* __restrict__ a, const int32_t* __restrict__ b, int32_t st, int32_t len,
    const int32_t* __restrict__ bsum, int32_t* __restrict__ outa, int32_t* __restrict__ outb) {
    __shared__ int32_t sh[SCAN_BLOCK / 64][4];
    const int64_t base = (int64_t)blockIdx.x * (SCAN_BLOCK * ITEMS) + (int64_t)threadIdx.x * ITEMS;
    int32_t va[ITEMS], vb[ITEMS];
    int32_t s[4] = {0, 0, 0, 0}, t[4];   // own items; totals of the tiles before this one
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t j = base + i;
        va[i] = j < len ? a[j * st] : 0;
        vb[i] = j < len ? b[j * st] : 0;
        s[0] += va[i];
        s[1] += vb[i];
    }
    for (int32_t j = threadIdx.x; j < (int32_t)blockIdx.x; j += SCAN_BLOCK) {
        s[2] += bsum[j];
        s[3] += bsum[8192 + j];
    }
    wg_excl_scan_n<SCAN_BLOCK>(s, sh, t);
    int32_t ea = s[0] + t[2], eb = s[1] + t[3];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t j = base + i;
        if (j < len) {
            outa[j] = ea;
            outb[j] = eb;
        }
        ea += va[i];
        eb += vb[i];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        outa[len] = t[2] + t[0];
        outb[len] = t[3] + t[1];
    }
}

// both scans on stream s, len <= SCAN_MAX_CELLS
static void scan_pair(const int32_t* a, const int32_t* b, int32_t st, int32_t len, int32_t* bsum, int32_t* outa,
                      int32_t* outb, hipStream_t s) {
    auto run = [&](auto items) {
        constexpr int ITEMS = decltype(items)::value;
        const int32_t tile = SCAN_BLOCK * ITEMS, nblocks = (int32_t)(((int64_t)len + tile - 1) / tile);
        hipLaunchKernelGGL(scan_reduce_kernel<ITEMS>, dim3(nblocks), dim3(SCAN_BLOCK), 0, s, a, b, st, len, bsum);
        hipLaunchKernelGGL(scan_final_kernel<ITEMS>, dim3(nblocks), dim3(SCAN_BLOCK), 0, s, a, b, st, len,
                           (const int32_t*)bsum, outa, outb);
    };
    // up to 2048 tiles of four items (eight totals a thread), else tiles of sixteen
    if (len <= 2048 * SCAN_BLOCK * 4) run(std::integral_constant<int, 4>{});
    else run(std::integral_constant<int, 16>{});
}

// ---- per-cell ordering of contributions and gather --------------------------------------
// the general sort's gather runs one wave per workgroup (GBLK lanes; one cell of 64 lanes
// or 64 / G cells): its barriers wait for the wave itself, never for other cells
template <int G>
struct GatherShape {
    static constexpr int BLK = G > 64 ? G : 64;
    static constexpr int GROUPS = BLK / G;
    static constexpr int CAPC = 6 * G;   // contributions per cell held in LDS
};

// position of the r-th set bit (from 0) of a mask with more than r set bits: the half of
// the current window that holds it, by population counts, down to one bit
__device__ __forceinline__ int select_bit(uint64_t m, int r) {
    int pos = 0;
    uint32_t w = (uint32_t)m;
    const int c = __popc(w);
    if (r >= c) {
        r -= c;
        w = (uint32_t)(m >> 32);
        pos = 32;
    }
#pragma unroll
    for (int half = 16; half >= 1; half >>= 1) {
        const int cl = __popc(w & ((1u << half) - 1u));
        if (r >= cl) {
            r -= cl;
            w >>= half;
            pos += half;
        }
    }
    return pos;
}

template <typename T, int G>
__global__ __launch_bounds__(GatherShape<G>::BLK) void bin_gather_kernel(
    int32_t ncell, const int32_t* __restrict__ offsets, const int32_t* __restrict__ coff,
    const int32_t* __restrict__ cwave, const uint64_t* __restrict__ cmask,
    unsigned long long* __restrict__ cpair, int32_t* __restrict__ ccur, int32_t* __restrict__ gidx, const T* __restrict__ sx, const T* __restrict__ sy,
    const T* __restrict__ svx, const T* __restrict__ svy, const T* __restrict__ svz,
    const uint32_t* __restrict__ spid, T* __restrict__ dx, T* __restrict__ dy,
    T* __restrict__ dvx, T* __restrict__ dvy, T* __restrict__ dvz, uint32_t* __restrict__ dpid,
    int32_t* __restrict__ dkey, int32_t* __restrict__ perm, int64_t* __restrict__ kept) {
    if (kept && blockIdx.x == 0 && threadIdx.x == 0) *kept = offsets[ncell];
    using S = GatherShape<G>;
    __shared__ int32_t s_w[S::GROUPS][S::CAPC];
    __shared__ int32_t s_base[S::GROUPS][S::CAPC];
    __shared__ uint64_t s_m[S::GROUPS][S::CAPC];

    // counters of the count and place passes are spent: leave them zero for the next call
    for (int64_t i = (int64_t)blockIdx.x * S::BLK + threadIdx.x; i <= ncell;
         i += (int64_t)gridDim.x * S::BLK) {
        cpair[i] = 0ull;
        ccur[i] = 0;
    }
    const int grp = threadIdx.x / G;
    const int lg = threadIdx.x % G;
    const int32_t cell = blockIdx.x * S::GROUPS + grp;
    const bool in = cell < ncell;
    int32_t b = 0, np = 0, cb = 0, m = 0;
    if (in) {
        b = offsets[cell];
        np = offsets[cell + 1] - b;
        cb = coff[cell];
        m = coff[cell + 1] - cb;
    }
    const bool lds_c = m <= S::CAPC;

    // phase A: contributions of this cell into LDS
    if (lds_c)
        for (int32_t j = lg; j < m; j += G) {
            s_w[grp][j] = cwave[cb + j];
            s_m[grp][j] = cmask[cb + j];
        }
    __syncthreads();

    // phase B: slot base of every contribution = particles of contributions from earlier
    // source waves (source waves are unique within a cell).  Cells with more
    // contributions than LDS holds expand their masks into a slot list in gidx.
    for (int32_t j = lg; j < m; j += G) {
        const int32_t wj = lds_c ? s_w[grp][j] : cwave[cb + j];
        uint64_t mj = lds_c ? s_m[grp][j] : cmask[cb + j];
        int32_t base = 0;
        for (int32_t i = 0; i < m; ++i) {
            const int32_t wi = lds_c ? s_w[grp][i] : cwave[cb + i];
            const uint64_t mi = lds_c ? s_m[grp][i] : cmask[cb + i];
            base += wi < wj ? __popcll(mi) : 0;
        }
        if (lds_c) {
            s_base[grp][j] = base;
        } else {
            int32_t* idx = gidx + b;
            const int32_t src0 = wj << 6;
            while (mj) {
                const int t = __builtin_ctzll(mj);
                idx[base++] = src0 + t;
                mj &= mj - 1;
            }
        }
    }
    __syncthreads();

    // phase C: every lane takes slots, U per round (slots s0 + u G + lg); the source of slot
    // s is the r-th lane of the contribution whose range [base, base + count) holds s, found
    // for the round's U slots in one pass over the contributions; then all of the round's
    // loads, then its stores
    constexpr int U = 4;
    for (int32_t s0 = 0; s0 < np; s0 += G * U) {
        int32_t src[U];
        if (lds_c) {
            int32_t jj[U], rr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) jj[u] = rr[u] = 0;
            for (int32_t i = 0; i < m; ++i) {
                const int32_t bi = s_base[grp][i], ci = __popcll(s_m[grp][i]);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t sl = s0 + u * G + lg;
                    if (sl >= bi && sl < bi + ci) {
                        jj[u] = i;
                        rr[u] = sl - bi;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                src[u] = s0 + u * G + lg < np ? (s_w[grp][jj[u]] << 6) + select_bit(s_m[grp][jj[u]], rr[u]) : -1;
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t sl = s0 + u * G + lg;
                src[u] = sl < np ? gidx[b + sl] : -1;
            }
        }
        T rx[U], ry[U], rvx[U], rvy[U], rvz[U];
        uint32_t rp[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (src[u] < 0) continue;
            const int32_t q = src[u];
            rx[u] = sx[q];
            ry[u] = sy ? sy[q] : (T)0;
            rvx[u] = svx[q];
            rvy[u] = svy[q];
            rvz[u] = svz[q];
            rp[u] = spid[q];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (src[u] < 0) continue;
            const int32_t d = b + s0 + u * G + lg;
            dx[d] = rx[u];
            if (sy) dy[d] = ry[u];
            dvx[d] = rvx[u];
            dvy[d] = rvy[u];
            dvz[d] = rvz[u];
            dpid[d] = rp[u];
            dkey[d] = cell;
            if (perm) perm[d] = src[u];
        }
    }
}

template <typename T, int G>
static void gather_launch(fp_ctx* c, const fp_particles* src, fp_particles* dst,
                          const int32_t* offsets, int32_t* perm, hipStream_t s) {
    const int groups = GatherShape<G>::GROUPS;
    const int grid = (c->ncell + groups - 1) / groups;
    const bool two_d = c->cfg.geometry != FP_COUETTE1D;
    hipLaunchKernelGGL((bin_gather_kernel<T, G>), dim3(grid), dim3(GatherShape<G>::BLK), 0, s, c->ncell,
                       offsets, c->coff, c->cwave, c->cmask, (unsigned long long*)c->cpair, c->ccur, c->gidx,
                       (const T*)src->x,
                       two_d ? (const T*)src->y : (const T*)nullptr, (const T*)src->vx,
                       (const T*)src->vy, (const T*)src->vz, src->pid, (T*)dst->x,
                       two_d ? (T*)dst->y : (T*)nullptr, (T*)dst->vx, (T*)dst->vy,
                       (T*)dst->vz, dst->pid, dst->key, perm, dst->n_dev);
}

template <typename T>
static void gather_dispatch(fp_ctx* c, const fp_particles* src, fp_particles* dst,
                            const int32_t* offsets, int32_t* perm, hipStream_t s) {
    // about one particle per lane, at most 32: the per-cell work (ordering the
    // contributions, expanding their masks) shortens with wider groups (the quadtree
    // cylinder's loop on 7.6e5 leaves of 24 particles: 1.68 ms per step at 32 lanes, 1.70 at
    // 16, 1.91 at 8)
    int g = lanes_per_cell(c, src->n, FILL_8, 1);
    if (c->cfg.lanes <= 0 && g > 32) g = 32;
    switch (g) {
        case 4: gather_launch<T, 4>(c, src, dst, offsets, perm, s); break;
        case 8: gather_launch<T, 8>(c, src, dst, offsets, perm, s); break;
        case 16: gather_launch<T, 16>(c, src, dst, offsets, perm, s); break;
        case 32: gather_launch<T, 32>(c, src, dst, offsets, perm, s); break;
        default: gather_launch<T, 64>(c, src, dst, offsets, perm, s); break;
    }
}

// ---- re-sort of particles that were sorted by cell one step earlier ---------------------
// After a step almost every particle sits in one of the 3 x 3 cells around its old cell.
// Pass 1 (one group per OLD cell) counts the particles bound for each of those nine
// neighbours, and lists the source indices of each direction, in source order, inside
// the old cell's own index range ("buckets": bidx, bucket ends in bend[cell][9]); every
// other particle (moved farther, or after the grouped range) goes to a short far list.
// Every old cell adds its bucket lengths to the counts of the destinations (nine integer
// atomics), far arrivals add one each, and one scan gives the offsets.  Pass 2 (one group
// per DESTINATION cell) concatenates its nine buckets in the order of their old cells --
// which is the order of source indices, i.e. the stable order -- inserting each far arrival
// before the buckets whose old cell starts after it, and writes its slots contiguously
// (whole cache lines, each written once).

// inclusive prefix sum over the G consecutive lanes of a group (lane lg of it): steps
// inside rows of 16 lanes by DPP row shifts (lanes before the row start read 0, lanes
// before the group start are masked), then across rows by the row broadcasts
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, true);
}
template <int G>
__device__ __forceinline__ uint32_t group_incl_scan(uint32_t x, int lg) {
    if constexpr (G >= 2) { const uint32_t y = dpp_u<0x111>(x); x += (G >= 16 || lg >= 1) ? y : 0u; }
    if constexpr (G >= 4) { const uint32_t y = dpp_u<0x112>(x); x += (G >= 16 || lg >= 2) ? y : 0u; }
    if constexpr (G >= 8) { const uint32_t y = dpp_u<0x114>(x); x += (G >= 16 || lg >= 4) ? y : 0u; }
    if constexpr (G >= 16) x += dpp_u<0x118>(x);
    if constexpr (G >= 32) x += dpp_u<0x142, 0xA>(x);   // row_bcast:15 into rows 1 and 3
    if constexpr (G >= 64) x += dpp_u<0x143, 0xC>(x);   // row_bcast:31 into rows 2 and 3
    return x;
}

// exclusive prefix sums of N values over a workgroup of BLOCK <= 1024 threads, in place;
// total: the sums over the block.  One LDS round for all of them: every wave scans the wave
// totals in its own lanes.  (With one thread walking them while the others waited, and a round
// for each value, the scan of 100 cells took 5.5 us instead of 3.2; two steps of 1e6 particles
// on 1e4 cells 168 us instead of 162)
template <int BLOCK, int N>
__device__ __forceinline__ void wg_excl_scan_n(int32_t (&v)[N], int32_t (*sh)[N], int32_t (&total)[N]) {
    constexpr int WAVES = BLOCK / 64;
    static_assert(WAVES >= 1 && WAVES <= 16, "the wave totals fit one row of lanes");
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        x[i] = (int32_t)group_incl_scan<64>((uint32_t)v[i], lane);
        if (lane == 63) sh[wv][i] = x[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int32_t t = (int32_t)group_incl_scan<16>(lane < WAVES ? (uint32_t)sh[lane][i] : 0u, lane & 15);
        total[i] = __builtin_amdgcn_readlane(t, WAVES - 1);
        v[i] = (wv > 0 ? __builtin_amdgcn_readlane(t, max(wv - 1, 0)) : 0) + x[i] - v[i];
    }
    __syncthreads();
}

// one value; sh holds BLOCK / 64 ints
template <int BLOCK>
__device__ __forceinline__ int32_t wg_excl_scan(int32_t v, int32_t* sh, int32_t& total) {
    int32_t x[1] = {v}, t[1];
    wg_excl_scan_n<BLOCK>(x, reinterpret_cast<int32_t(*)[1]>(sh), t);
    total = t[0];
    return x[0];
}

__device__ __forceinline__ void far_put(int32_t k, int32_t j, int64_t slot, int64_t cap,
                                        uint64_t* flist, int32_t* cnt, int32_t* fcnt) {
    if (slot < cap) flist[slot] = ((uint64_t)(uint32_t)k << 32) | (uint32_t)j;
    atomicAdd(&cnt[k], 1);
    atomicAdd(&fcnt[k], 1);
}

// length of the bucket of old cell c for direction d
__device__ __forceinline__ int32_t bucket_len(const int32_t* __restrict__ bend, int32_t c, int d) {
    const int32_t* e = bend + (int64_t)c * 9;
    return e[d] - (d > 0 ? e[d - 1] : 0);
}

// grid: ncell*G lanes for the old cells, then FAR_BLOCKS blocks for the ungrouped tail.
// Far movers are appended to the list with one atomic per block (cells) or per wave
// (tail) on its length.  These atomics on one address are what bounds the kernel as soon as
// most blocks have a far mover: 10.6 ns each, whatever else runs, 66 us for the 6272 blocks of
// 256 threads that 2e7 particles on 200 704 cells make.  Hence blocks of 1024 threads from
// RC_WIDE lanes on (93 -> 67 us; 1e6 particles on 1e4 cells 14.5 -> 11; the grid of 100
// cells, 25 narrow blocks or 7 wide ones, 5.6 against 7.9 us the other way).  Persistent blocks
// that collect far movers in LDS over several tiles: 69 and 13 us.
// A lane takes a run of consecutive particles, and LDS counters of its own give a particle
// its place: against a prefix sum over the group for every round of particles, and all keys
// read again for the far movers, 113 -> 93 us.
constexpr int FAR_BLOCKS = 64;

// Order in which the gathers visit destination cells on a 2-D grid: column strips of
// STRIP cells, each strip row by row (a narrower last strip takes the rest).  A
// destination row reads the particles of the three source rows around it; in row-major
// order those rows are a whole grid row apart and their cache lines are evicted from L2
// between the reads, in strip order they are STRIP cells apart.  A bijection on
// [0, nx*ny); the identity for grids no wider than one strip.
constexpr int32_t STRIP = 32;
__device__ __forceinline__ int32_t strip_cell(int32_t t, int32_t nx, int32_t ny) {
    if (nx <= STRIP) return t;
    const int32_t full = nx / STRIP, per = STRIP * ny;
    const int32_t sidx = t / per;
    if (sidx < full) {
        const int32_t r = t - sidx * per;
        return (r / STRIP) * nx + sidx * STRIP + r % STRIP;
    }
    const int32_t w = nx - full * STRIP, r = t - full * per;
    return (r / w) * nx + full * STRIP + r % w;
}

// entries of bidx that a wave of the count kernel puts together in LDS
constexpr int RC_STAGE = 1024;
// lanes from which workgroups of 1024 are taken: enough of them for most CUs.  Whole re-sorts of
// 100 particles per cell, narrow against wide, FP32 (FP64): 10^2 cells 18.2 / 19.1 us, 46^2
// (135 424 lanes) 23.1 / 23.5 (24.5 / 25.2), 56^2 (200 704) 25.6 / 25.7 (28.6 / 28.9), 58^2 (215 296)
// 25.7 / 25.7 (30.0 / 29.4), 64^2 27.6 / 27.5 (32.1 / 31.7), 80^2 35.6 / 34.4, 110^2 50.2 / 45.5,
// 200^2 122.7 / 117.6
constexpr int64_t RC_WIDE = 200 * 1024;
// *p += 1 in LDS, old value returned
__device__ __forceinline__ int32_t lds_inc(int32_t* p) {
    return __hip_atomic_fetch_add(p, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

template <int G, int BLK>
__global__ __launch_bounds__(BLK) void rebin_count_kernel(
    int32_t ncell, int32_t nx, int64_t n, const int64_t* __restrict__ n_dev, int64_t cap,
    int32_t cell_blocks, const int32_t* __restrict__ src_off, const int32_t* __restrict__ key,
    int32_t* __restrict__ bend, int32_t* __restrict__ bidx, int32_t* __restrict__ cnt,
    int32_t* __restrict__ fcnt, int32_t* __restrict__ farn, uint64_t* __restrict__ flist,
    unsigned long long* __restrict__ errcount) {
    if (n_dev) n = *n_dev;
    __shared__ int32_t sh[BLK / 64];
    __shared__ int32_t s_base;
    __shared__ int32_t s_pos[BLK / 64][10][64];   // the last row: no direction
    __shared__ __attribute__((aligned(16))) uint16_t s_stage[BLK / 64][RC_STAGE + 8];   // (and a place for no bucket)
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    if ((int32_t)blockIdx.x >= cell_blocks) {
        // particles after the grouped range: all take the general path
        const int64_t t0 = max((int64_t)src_off[ncell], (int64_t)0);
        const int64_t stride = (int64_t)FAR_BLOCKS * BLK;
        for (int64_t jb = t0 + (int64_t)(blockIdx.x - cell_blocks) * BLK; jb < n;
             jb += stride) {
            const int64_t j = jb + threadIdx.x;
            int32_t k = ncell;
            if (j < n) {
                k = key[j];
                if (k < 0 || k > ncell) {
                    atomicAdd(errcount, 1ull);
                    k = ncell;
                }
            }
            const bool far = k < ncell;
            const uint64_t m = __ballot(far);
            int32_t wbase = 0;
            if (lane == 0 && m) wbase = atomicAdd(farn, (int32_t)__popcll(m));
            wbase = __shfl(wbase, 0, 64);
            if (far) far_put(k, (int32_t)j, (int64_t)wbase + __popcll(m & below), cap, flist, cnt, fcnt);
        }
        return;
    }
    const int64_t gt = (int64_t)blockIdx.x * BLK + threadIdx.x;
    const int32_t cell = (int32_t)(gt / G);
    const int lg = (int)(gt % G);
    int32_t nfar = 0, b = 0, e = 0, cx = 0, rs = 0;
    if (cell < ncell) {
        b = (int32_t)min((int64_t)max(src_off[cell], 0), n);
        e = (int32_t)min((int64_t)src_off[cell + 1], n);
        cx = cell % nx;
        rs = cell - cx;
    }
    // lane lg takes the lg-th run of the cell's particles, so that a particle's rank among
    // those of its direction is the count of the lanes before plus its lane's own so far
    const int32_t size = e > b ? e - b : 0;   // (a bad src_off may leave any e)
    const int32_t chunk = (size + G - 1) / G, j0 = b + lg * chunk;
    const int32_t mine = max(min(size - lg * chunk, chunk), 0);
    int32_t(&pos)[10][64] = s_pos[threadIdx.x >> 6];   // this lane's column only
    uint16_t* stage = s_stage[threadIdx.x >> 6];
    // the wave's cells follow each other, so do their ranges of bidx: they are put together in
    // LDS and written as one (else, only with crowded cells or a bad src_off, in place)
    const int64_t cells_left = (int64_t)ncell - (gt - lane) / G;
    const int32_t wb = __builtin_amdgcn_readfirstlane(b);
    const int32_t we = cells_left > 0 ? __builtin_amdgcn_readlane(e, (int)min(cells_left * G, (int64_t)64) - 1) : wb;
    const bool staged = we >= wb && we - wb <= RC_STAGE && __all(cell >= ncell || (b >= wb && b <= e && e <= we));
#pragma unroll
    for (int i = 0; i < 9; ++i) pos[i][lane] = 0;
    // all of the range is written out, also behind a cell's buckets, where no particle with a
    // direction puts anything; with a bad src_off the ranges of different waves overlap, and
    // what a gather reads there must be a particle's index: wb then
#pragma unroll
    for (int i = 0; i < RC_STAGE / 512; ++i) reinterpret_cast<uint4*>(stage)[i * 64 + lane] = make_uint4(0, 0, 0, 0);
    // four keys of the run from r on, ncell (no destination) beyond it.  Read as one, up to
    // three keys past the run, but for the last waves
    struct Keys { int32_t k[4]; };
    const bool wide = __all(j0 + (int64_t)mine + 4 <= n);
    auto load4 = [&](int32_t r) __attribute__((always_inline)) {
        Keys q = {{ncell, ncell, ncell, ncell}};
        if (wide) {
            const int32_t* p = key + (r < mine ? j0 + r : 0);
            q = {{p[0], p[1], p[2], p[3]}};
#pragma unroll
            for (int u = 0; u < 4; ++u) q.k[u] = r + u < mine ? q.k[u] : ncell;
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (r + u < mine) q.k[u] = key[j0 + r + u];
        }
        return q;
    };
    // direction 0..8 of key k among the 3 x 3 cells around the old cell (column cx, its row
    // starting at cell rs), NONE for any other, deleted or invalid one; no division: k's row is
    // told by comparing k - rs with 0 and nx, and no branch
    constexpr uint32_t NONE = 9;
    auto direction = [&](int32_t k) __attribute__((always_inline)) {
        const int32_t rel = (int32_t)((uint32_t)k - (uint32_t)rs);   // (an invalid key may be anything)
        const int32_t dy = (rel >= nx ? 1 : 0) - (rel < 0 ? 1 : 0);
        const int32_t dx = rel - dy * nx - cx;
        const bool near = (uint32_t)k < (uint32_t)ncell & rel >= -nx & rel < 2 * nx & (uint32_t)(dx + 1) < 3u;
        return near ? (uint32_t)(3 * dy + dx + 4) : NONE;
    };
    // first pass: counts per direction; the directions of a lane's first sixteen particles
    // are kept, four bits each
    uint64_t kept = 0;
    int32_t nbad = 0;
    {
        auto count4 = [&](const Keys& q, int32_t r) __attribute__((always_inline)) {
            uint32_t quad = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t k = q.k[u];
                const uint32_t d = direction(k);
                nbad += (uint32_t)k > (uint32_t)ncell ? 1 : 0;
                nfar += ((uint32_t)k < (uint32_t)ncell && d == NONE) ? 1 : 0;
                quad |= d << (4 * u);
                lds_inc(&pos[d][lane]);
            }
            if (r < 16) kept |= (uint64_t)quad << (4 * r);
        };
        Keys q[4];   // all of the first sixteen on their way at once
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (v == 0 || __any(4 * v < mine)) q[v] = load4(4 * v);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (__any(4 * v < mine)) count4(q[v], 4 * v);
        for (int32_t r = 16; __any(r < mine); r += 4) count4(load4(r), r);
    }
    if (nbad) atomicAdd(errcount, (unsigned long long)nbad);
    // the lane's next place in every bucket (from wb if staged): bucket starts inside the cell, then the
    // lanes before
    {
        const int last = lane - lg + G - 1;
        int32_t run = 0, t[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int32_t c = pos[i][lane];
            const int32_t incl = (int32_t)group_incl_scan<G>((uint32_t)c, lg);
            t[i] = __shfl(incl, last, 64);
            pos[i][lane] = (staged ? b - wb : b) + run + incl - c;
            run += t[i];
            if (cell < ncell && lg == i % G) bend[(int64_t)cell * 9 + i] = run;
        }
        // this cell's share of the destination counts (integer adds: order-free); lane lg
        // takes directions lg, lg + G, ... (groups may have fewer than 9 lanes)
        if (cell < ncell)
            for (int q = lg; q < 9; q += G) {
                int32_t cnt_d = 0;
#pragma unroll
                for (int i = 0; i < 9; ++i) cnt_d = q == i ? t[i] : cnt_d;
                if (cnt_d > 0) atomicAdd(&cnt[cell + (q / 3 - 1) * nx + (q % 3 - 1)], cnt_d);
            }
    }
    // second pass: source indices into the buckets, in source order
    auto place = [&](auto put) __attribute__((always_inline)) {
        for (int32_t r = 0; __any(r < mine); r += 4) {
            uint32_t quad = 0;
            if (r < 16) {
                quad = (uint32_t)(kept >> (4 * r));
            } else {
                const Keys q = load4(r);
#pragma unroll
                for (int u = 0; u < 4; ++u) quad |= direction(q.k[u]) << (4 * u);
            }
            int32_t p[4];
            uint32_t d[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                d[u] = (quad >> (4 * u)) & 15u;
                p[u] = lds_inc(&pos[d[u]][lane]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) put(d[u] != NONE, p[u], j0 + r + u);
        }
    };
    if (staged) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        place([&](bool near, int32_t p, int32_t j) { stage[near ? p : RC_STAGE] = (uint16_t)(j - wb); });
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int32_t i = lane; i < we - wb; i += 64) bidx[wb + i] = wb + stage[i];
    } else {
        place([&](bool near, int32_t p, int32_t j) {
            if (near) bidx[p] = j;
        });
    }
    if (!__syncthreads_or(nfar)) return;
    int32_t tot;
    const int32_t pre = wg_excl_scan<BLK>(nfar, sh, tot);
    if (threadIdx.x == 0) s_base = atomicAdd(farn, tot);
    __syncthreads();
    if (nfar == 0) return;
    int64_t slot = (int64_t)s_base + pre;
    // of the first sixteen only those without a direction are read again
    const uint64_t ones = 0x1111111111111111ull;
    uint64_t x = kept ^ (ones * NONE);
    x = ~(x | x >> 1 | x >> 2 | x >> 3) & ones;   // bit 4 u: no direction
    if (mine < 16) x &= (1ull << (4 * mine)) - 1;
    for (int32_t r = 16;;) {
        int32_t j;
        if (x) {
            j = j0 + (__ffsll((unsigned long long)x) - 1) / 4;
            x &= x - 1;
        } else {
            if (r >= mine) break;
            j = j0 + r++;
        }
        const int32_t k = key[j];
        if ((uint32_t)k < (uint32_t)ncell && direction(k) == NONE) far_put(k, j, slot++, cap, flist, cnt, fcnt);
    }
}

// both exclusive scans for grids of up to SMALL_SCAN_CELLS cells in one launch: each
// workgroup of SSB cells adds up all earlier counts itself (at most a few tens of KB,
// coalesced, one round of loads) instead of waiting for a second pass
constexpr int SSB = 1024, SS_UR = 16;
constexpr int SMALL_SCAN_CELLS = SSB * SS_UR;

// It also splits the far list into per-destination segments for its own cells (every
// workgroup reads the whole list and keeps the entries bound for its range; the slot
// inside a segment comes from an LDS counter, so the order inside a segment is
// arbitrary): no separate far-placement launch on small grids.
__global__ __launch_bounds__(SSB) void rebin_small_scan_kernel(
    int32_t ncell, int64_t cap, const int32_t* __restrict__ cnt, const int32_t* __restrict__ fcnt,
    int32_t* __restrict__ offsets, int32_t* __restrict__ foff, const int32_t* __restrict__ farn,
    const uint64_t* __restrict__ flist, int32_t* __restrict__ fkey, int32_t* __restrict__ fsrc) {
    __shared__ int32_t sh[SSB / 64][4];
    __shared__ int32_t s_foff[SSB], s_cur[SSB];
    const int32_t k0 = blockIdx.x * SSB, k = k0 + threadIdx.x;
    // own counts; the counts of the earlier ranges (one branch per range for the whole
    // workgroup, no wait between the loads)
    int32_t s[4] = {0, 0, 0, 0}, t[4];
    if (k < ncell) {
        s[0] = cnt[k];
        s[1] = fcnt[k];
    }
    int32_t la[SS_UR - 1], lb[SS_UR - 1];
#pragma unroll
    for (int u = 0; u < SS_UR - 1; ++u) {
        la[u] = lb[u] = 0;
        if (u < (int)blockIdx.x) {
            la[u] = cnt[u * SSB + threadIdx.x];
            lb[u] = fcnt[u * SSB + threadIdx.x];
        }
    }
#pragma unroll
    for (int u = 0; u < SS_UR - 1; ++u) {
        s[2] += la[u];
        s[3] += lb[u];
    }
    wg_excl_scan_n<SSB>(s, sh, t);
    const int32_t ea = s[0] + t[2], eb = s[1] + t[3], sb = t[1];
    if (k < ncell) {
        offsets[k] = ea;
        foff[k] = eb;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        offsets[ncell] = t[2] + t[0];
        foff[ncell] = t[3] + t[1];
    }
    if (sb == 0) return;    // no far arrivals in this range (block-uniform)
    s_foff[threadIdx.x] = eb;
    s_cur[threadIdx.x] = 0;
    __syncthreads();
    const int64_t nf = min((int64_t)farn[0], cap);
    for (int64_t i = threadIdx.x; i < nf; i += SSB) {
        const uint64_t v = flist[i];
        const int32_t kf = (int32_t)(v >> 32) - k0;
        if (kf < 0 || kf >= SSB) continue;
        const int32_t slot = s_foff[kf] + atomicAdd(&s_cur[kf], 1);
        if (slot < cap) {
            fkey[slot] = kf + k0;
            fsrc[slot] = (int32_t)(uint32_t)v;
        }
    }
}

// far list -> per-destination segments (order inside a segment is arbitrary)
__global__ __launch_bounds__(BIN_BLOCK) void rebin_far_place_kernel(
    int64_t cap, const int32_t* __restrict__ farn, const uint64_t* __restrict__ flist,
    const int32_t* __restrict__ foff, int32_t* __restrict__ fcur, int32_t* __restrict__ fkey,
    int32_t* __restrict__ fsrc) {
    const int64_t nf = min((int64_t)farn[0], cap);
    for (int64_t i = (int64_t)blockIdx.x * BIN_BLOCK + threadIdx.x; i < nf;
         i += (int64_t)gridDim.x * BIN_BLOCK) {
        const uint64_t v = flist[i];
        const int32_t k = (int32_t)(v >> 32), p = (int32_t)(uint32_t)v;
        const int32_t slot = foff[k] + atomicAdd(&fcur[k], 1);
        if (slot < cap) {
            fkey[slot] = k;
            fsrc[slot] = p;
        }
    }
}

template <typename T>
struct Rec {
    const T *sx, *sy, *svx, *svy, *svz;
    const uint32_t* spid;
    T *dx, *dy, *dvx, *dvy, *dvz;
    uint32_t* dpid;
    int32_t *dkey, *perm;
    __device__ __forceinline__ void copy(int32_t p, int32_t d, int32_t k) const {
        dx[d] = sx[p];
        if (sy) dy[d] = sy[p];
        dvx[d] = svx[p];
        dvy[d] = svy[p];
        dvz[d] = svz[p];
        dpid[d] = spid[p];
        dkey[d] = k;
        if (perm) perm[d] = p;
    }
};

// grid: cell blocks (one group of G lanes per destination cell), then FAR_BLOCKS blocks
// for the far arrivals.  Every block also clears a share of fcnt/fcur/farn for the next
// call.
template <typename T, int G>
__global__ __launch_bounds__(BIN_BLOCK) void rebin_gather_kernel(
    int32_t ncell, int32_t nx, int32_t ny, int64_t n, const int64_t* __restrict__ n_dev,
    int64_t* __restrict__ kept, int64_t cap, int32_t cell_blocks,
    const int32_t* __restrict__ src_off, const int32_t* __restrict__ bend,
    const int32_t* __restrict__ bidx, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ foff, const int32_t* __restrict__ fkey,
    const int32_t* __restrict__ fsrc, int32_t* __restrict__ cnt, int32_t* __restrict__ fcnt,
    int32_t* __restrict__ fcur, int32_t* __restrict__ farn, Rec<T> r) {
    if (n_dev) n = *n_dev;
    if (kept && blockIdx.x == 0 && threadIdx.x == 0) *kept = offsets[ncell];
    constexpr int GROUPS = BIN_BLOCK / G;
    __shared__ int32_t s_run[GROUPS][9][3];   // bucket start in bidx, length, far arrivals before
    for (int64_t i = (int64_t)blockIdx.x * BIN_BLOCK + threadIdx.x; i <= ncell;
         i += (int64_t)gridDim.x * BIN_BLOCK) {
        cnt[i] = 0;
        fcnt[i] = 0;
        fcur[i] = 0;
        if (i == 0) farn[0] = 0;
    }
    const int64_t lim = min((int64_t)offsets[ncell], n);   // slots that exist in dst
    const int32_t fend = (int32_t)min((int64_t)foff[ncell], cap);
    if ((int32_t)blockIdx.x >= cell_blocks) {
        for (int32_t i = (int32_t)(blockIdx.x - cell_blocks) * BIN_BLOCK + threadIdx.x; i < fend;
             i += FAR_BLOCKS * BIN_BLOCK) {
            const int32_t k = fkey[i], p = fsrc[i];
            if (k < 0 || k >= ncell || p < 0 || p >= n) continue;   // only with bad src_off
            const int32_t ky = k / nx, kx = k - ky * nx;
            int32_t slot = offsets[k];
            for (int ey = -1; ey <= 1; ++ey)
                for (int ex = -1; ex <= 1; ++ex) {
                    const int32_t sx = kx - ex, sy = ky - ey;
                    if (sx < 0 || sx >= nx || sy < 0 || sy >= ny) continue;
                    const int32_t c2 = sy * nx + sx;
                    if (src_off[c2] < p) slot += bucket_len(bend, c2, (ey + 1) * 3 + (ex + 1));
                }
            const int32_t f1 = min(foff[k + 1], fend);
            for (int32_t q = foff[k]; q < f1; ++q) slot += fsrc[q] < p ? 1 : 0;
            if (slot >= 0 && slot < lim) r.copy(p, slot, k);
        }
        return;
    }
    const int grp = threadIdx.x / G, lg = threadIdx.x % G;
    const int32_t ord = xcd_block((int32_t)blockIdx.x, cell_blocks) * GROUPS + grp;
    const bool in = ord < ncell;
    const int32_t k = in ? strip_cell(ord, nx, ny) : ord;
    int32_t kx = 0, ky = 0, base = 0;
    if (in) {
        ky = k / nx;
        kx = k - ky * nx;
        base = offsets[k];
    }
    // the nine buckets in the order of their old cells (rows ky-1, ky, ky+1; columns
    // kx-1, kx, kx+1): that is the order of source indices
    for (int q = lg; q < 9; q += G) {
        int32_t st = 0, len = 0, fb = 0;
        const int32_t sy = ky - 1 + q / 3, sx = kx - 1 + q % 3;
        if (in && sx >= 0 && sx < nx && sy >= 0 && sy < ny) {
            const int32_t c2 = sy * nx + sx;
            const int d = (ky - sy + 1) * 3 + (kx - sx + 1);
            const int32_t* e2 = bend + (int64_t)c2 * 9;
            const int32_t b0 = d > 0 ? e2[d - 1] : 0;
            const int32_t s0 = max(src_off[c2], 0);
            st = s0 + b0;
            len = e2[d] - b0;
            const int32_t f1 = min(foff[k + 1], fend);
            for (int32_t f = foff[k]; f < f1; ++f) fb += fsrc[f] < s0 ? 1 : 0;
        }
        s_run[grp][q][0] = st;
        s_run[grp][q][1] = len;
        s_run[grp][q][2] = fb;
    }
    __syncthreads();
    int32_t rs[10], rst[9], rfb[9];
    rs[0] = 0;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        rst[q] = s_run[grp][q][0];
        rs[q + 1] = rs[q] + s_run[grp][q][1];
        rfb[q] = s_run[grp][q][2];
    }
    const int32_t nk = rs[9];
    // position q of the concatenated buckets -> source index, U per lane per round
    constexpr int U = 4;
    for (int32_t q0 = 0; q0 < nk; q0 += G * U) {
        int32_t src[U], dst[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t q = q0 + u * G + lg;
            src[u] = -1;
            dst[u] = -1;
            if (q < nk) {
                int32_t st = rst[0] - rs[0], fb = rfb[0];
#pragma unroll
                for (int t = 1; t < 9; ++t)
                    if (q >= rs[t]) {
                        st = rst[t] - rs[t];
                        fb = rfb[t];
                    }
                src[u] = bidx[st + q];
                dst[u] = base + q + fb;
            }
        }
        T rx[U], ry[U], rvx[U], rvy[U], rvz[U];
        uint32_t rp[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (src[u] >= 0) {
                const int32_t j = src[u];
                rx[u] = r.sx[j];
                ry[u] = r.sy ? r.sy[j] : (T)0;
                rvx[u] = r.svx[j];
                rvy[u] = r.svy[j];
                rvz[u] = r.svz[j];
                rp[u] = r.spid[j];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t d = dst[u];
            if (src[u] >= 0 && d >= 0 && d < lim) {
                r.dx[d] = rx[u];
                if (r.dy) r.dy[d] = ry[u];
                r.dvx[d] = rvx[u];
                r.dvy[d] = rvy[u];
                r.dvz[d] = rvz[u];
                r.dpid[d] = rp[u];
                r.dkey[d] = k;
                if (r.perm) r.perm[d] = src[u];
            }
        }
    }
}

// The gather of one destination cell can also produce the cell's moments (the same
// quantities fp_moments computes from the sorted particles): the group has just written
// every particle of its cell.  In this form the group also places its own far arrivals
// (no separate far blocks) and then reads its fresh slots back (L1/L2-resident) for the
// two moment passes.  Its workgroups are one wave (GM_BLOCK lanes, 64 / G cells, or one
// cell of 64 lanes): the group's barriers (far staging, bucket prefix, slot read-back, the
// moment reduction in LDS) then wait for the wave itself and never for other cells.
constexpr int GM_BLOCK = 64;

// (in FP64 five positions a lane take 134 registers, one wave fewer per SIMD: bounded to 128, of
// which two are spilled)
template <typename T, int G, int NVX, int BLK = GM_BLOCK>
__global__ __launch_bounds__(BLK, sizeof(T) == 8 && G >= 32 ? 4 : 1) void rebin_gather_mom_kernel(
    int32_t ncell, int32_t nx, int32_t ny, int64_t n, const int64_t* __restrict__ n_dev,
    int64_t* __restrict__ kept, int64_t cap,
    const int32_t* __restrict__ src_off, const int32_t* __restrict__ bend,
    const int32_t* __restrict__ bidx, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ foff, const int32_t* __restrict__ fsrc,
    int32_t* __restrict__ cnt, int32_t* __restrict__ fcnt, int32_t* __restrict__ fcur,
    int32_t* __restrict__ farn, Rec<T> r, double* __restrict__ mom, double* __restrict__ samp) {
    if (n_dev) n = *n_dev;
    if (kept && blockIdx.x == 0 && threadIdx.x == 0) *kept = offsets[ncell];
    constexpr int GROUPS = BLK / G;
    // positions per lane and round: at 32 lanes one more, so that a cell of 100 particles and
    // the shift to an aligned slot (below) still take one round
    constexpr int GM_U = G >= 32 ? 5 : 4;
    __shared__ int32_t s_run[GROUPS][9][4];   // start in bidx, length, far before, range start
    __shared__ int32_t s_pre[GROUPS][10];     // bucket starts in the cell's concatenation
    __shared__ double s_samp[GROUPS][14];     // the cells' time-average sums
    __shared__ MomShared<BLK, G> sm;
    // far arrivals of a cell staged in LDS, up to FCAP of them (their ranks compare every
    // arrival with all others and with the nine source ranges), in the space of the
    // moment reduction, which is used only after the gather's last barrier: the
    // workgroup's LDS stays at 7 to 9 KB from 16 lanes on (15 KB at four), so that the 16
    // one-wave workgroups that a CU's registers allow fit into 160 KB
    constexpr int FCAP = (2048 / GROUPS) < (int)(sizeof(sm.red) / (sizeof(int32_t) * GROUPS))
                             ? (2048 / GROUPS) : (int)(sizeof(sm.red) / (sizeof(int32_t) * GROUPS));
    static_assert(sizeof(int32_t) * GROUPS * FCAP <= sizeof(sm.red), "far staging space");
    int32_t(*s_far)[FCAP] = reinterpret_cast<int32_t(*)[FCAP]>(&sm.red[0][0]);
    for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i <= ncell;
         i += (int64_t)gridDim.x * BLK) {
        cnt[i] = 0;
        fcnt[i] = 0;
        fcur[i] = 0;
        if (i == 0) farn[0] = 0;
    }
    const int64_t lim = min((int64_t)offsets[ncell], n);
    const int32_t fend = (int32_t)min((int64_t)foff[ncell], cap);
    const int grp = threadIdx.x / G, lg = threadIdx.x % G;
    const int32_t ord = xcd_block((int32_t)blockIdx.x, (int32_t)gridDim.x) * GROUPS + grp;
    const bool in = ord < ncell;
    const int32_t k = in ? strip_cell(ord, nx, ny) : ord;
    int32_t kx = 0, ky = 0, base = 0, f0 = 0, f1 = 0;
    if (in) {
        ky = k / nx;
        kx = k - ky * nx;
        base = offsets[k];
        f0 = min(foff[k], fend);
        f1 = min(foff[k + 1], fend);
    }
    // the cell's 14 time-average sums, sum e on lane e % G, loaded now (parked in LDS
    // across the gather and the moments) and updated at the end
    constexpr int SQ = (14 + G - 1) / G;
    const bool samp_cell = samp && in;
    double samp_ld[SQ];
#pragma unroll
    for (int u = 0; u < SQ; ++u) {
        const int e = lg + u * G;
        samp_ld[u] = samp_cell && e < 14 ? samp[(int64_t)k * SAMP + e] : 0.0;
    }
    // the nine buckets' descriptors (bucket start and length in the old cell's range, the
    // range start), loaded before the far staging's barrier
    constexpr int QN = (9 + G - 1) / G;
    int32_t q_st[QN], q_len[QN], q_s0[QN];
#pragma unroll
    for (int u = 0; u < QN; ++u) {
        const int q = lg + u * G;
        q_st[u] = 0;
        q_len[u] = 0;
        q_s0[u] = INT32_MAX;   // a neighbour outside the grid
        const int32_t sy = ky - 1 + q / 3, sx = kx - 1 + q % 3;
        if (q < 9 && in && sx >= 0 && sx < nx && sy >= 0 && sy < ny) {
            const int32_t c2 = sy * nx + sx;
            const int d = (ky - sy + 1) * 3 + (kx - sx + 1);
            const int32_t* e2 = bend + (int64_t)c2 * 9;
            const int32_t b0 = d > 0 ? e2[d - 1] : 0;
            q_s0[u] = max(src_off[c2], 0);
            q_st[u] = q_s0[u] + b0;
            q_len[u] = e2[d] - b0;
        }
    }
    const int32_t nf = f1 - f0;
    const bool far_lds = nf <= FCAP;   // group-uniform
    if (far_lds)
        for (int32_t t = lg; t < nf; t += G) s_far[grp][t] = fsrc[f0 + t];
#pragma unroll
    for (int u = 0; u < SQ; ++u)
        if (samp_cell && lg + u * G < 14) s_samp[grp][lg + u * G] = samp_ld[u];
    __syncthreads();
    auto far_at = [&](int32_t t) __attribute__((always_inline)) {
        return far_lds ? s_far[grp][t] : fsrc[f0 + t];
    };
#pragma unroll
    for (int u = 0; u < QN; ++u) {
        const int q = lg + u * G;
        if (q < 9) {
            int32_t fb = 0;
            if (q_s0[u] != INT32_MAX)
                for (int32_t f = 0; f < nf; ++f) fb += far_at(f) < q_s0[u] ? 1 : 0;
            s_run[grp][q][0] = q_st[u];
            s_run[grp][q][1] = q_len[u];
            s_run[grp][q][2] = fb;
            s_run[grp][q][3] = q_s0[u];
        }
    }
    __syncthreads();
    // bucket starts in the cell's concatenation: lane q adds up the lengths before bucket q
    // (ten lanes at once instead of one lane walking the nine buckets)
    for (int q = lg; q < 10; q += G) {
        int32_t acc = 0;
#pragma unroll
        for (int t = 0; t < 9; ++t) acc += t < q ? s_run[grp][t][1] : 0;
        s_pre[grp][q] = acc;
    }
    __syncthreads();
    int32_t rs[10];
#pragma unroll
    for (int q = 0; q < 10; ++q) rs[q] = s_pre[grp][q];
    const int32_t nk = rs[9];
    // bucket of position q: the number of bucket starts at or before q (the buckets are
    // in order; empty ones share their start), its descriptor read back from LDS
    auto lookup = [&](int32_t q, int32_t& j, int32_t& fb) __attribute__((always_inline)) {
        int t = 0;
#pragma unroll
        for (int tt = 1; tt < 9; ++tt) t += q >= rs[tt] ? 1 : 0;
        fb = s_run[grp][t][2];
        j = ld_off(bidx, s_run[grp][t][0] + q - s_pre[grp][t]);
    };
    // one round: V of the GM_U positions per lane, all loads first (without a branch between
    // them, so that they go out together: 626 -> 616 us), then the stores; velocities returned
    auto round = [&](auto positions, int32_t q0, T (&ox)[GM_U], T (&oy)[GM_U], T (&oz)[GM_U])
                     __attribute__((always_inline)) {
        constexpr int V = decltype(positions)::value;
        int32_t src[V], dst[V];
#pragma unroll
        for (int u = 0; u < V; ++u) {
            // positions beyond the last take the last one's loads and no stores
            const int32_t q = q0 + u * G + lg;
            int32_t fb;
            lookup(max(min(q, nk - 1), 0), src[u], fb);
            dst[u] = q >= 0 && q < nk ? base + q + fb : -1;
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            if (src[u] < 0) dst[u] = -1;
            src[u] = max(src[u], 0);
        }
        T rx[V], ry[V];
        uint32_t rp[V];
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int32_t j = src[u];
            rx[u] = ld_off(r.sx, j);
            ry[u] = r.sy ? ld_off(r.sy, j) : (T)0;
            ox[u] = ld_off(r.svx, j);
            oy[u] = ld_off(r.svy, j);
            oz[u] = ld_off(r.svz, j);
            rp[u] = ld_off(r.spid, j);
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int32_t d = dst[u];
            if (d >= 0 && d < lim) {
                st_off(r.dx, d, rx[u]);
                if (r.dy) st_off(r.dy, d, ry[u]);
                st_off(r.dvx, d, ox[u]);
                st_off(r.dvy, d, oy[u]);
                st_off(r.dvz, d, oz[u]);
                st_off(r.dpid, d, rp[u]);
                st_off(r.dkey, d, k);
                if (r.perm) st_off(r.perm, d, src[u]);
            }
        }
    };
    // velocities of the first round stay in registers: a cell that one round covers and
    // that has no far arrival takes its moments from them instead of reading its slots back
    T kvx[GM_U], kvy[GM_U], kvz[GM_U];
#pragma unroll
    for (int u = 0; u < GM_U; ++u) kvx[u] = kvy[u] = kvz[u] = (T)0;
    // without far arrivals the rounds start at the slot aligned to the group's lanes at or
    // before the cell's first: every store of a group then writes whole cache lines but for
    // the cell's ends, instead of two halves of lines each (stores are a third of the
    // kernel: 626 -> 600 us for the re-sort of 2e7 particles; with four positions a lane, one
    // round in six did not cover its cell and nothing was gained: 622).  Cells of at most one
    // position a lane have nothing to gain from it, and neither they nor those that two cover
    // take the loads of GM_U (decided for a wave's cells together): at 28 particles per cell
    // and 32 lanes (a loop of 14 000 FP64 cells) two steps take 156 us instead of 161
    const bool one = __all(nk <= G);
    const int32_t off = nf == 0 && !one ? base & (G - 1) : 0;
    if (one) {
        if (nk > 0) round(std::integral_constant<int, 1>{}, 0, kvx, kvy, kvz);
    } else if (__all(nk + off <= 2 * G)) {
        if (nk > 0) round(std::integral_constant<int, 2>{}, -off, kvx, kvy, kvz);
    } else {
        for (int32_t q0 = nk > 0 ? -off : 0; q0 < nk; q0 += G * GM_U) {   // an empty cell loads nothing
            T tx[GM_U], ty[GM_U], tz[GM_U];
            round(std::integral_constant<int, GM_U>{}, q0, tx, ty, tz);
            if (q0 == -off) {
#pragma unroll
                for (int u = 0; u < GM_U; ++u) {
                    kvx[u] = tx[u];
                    kvy[u] = ty[u];
                    kvz[u] = tz[u];
                }
            }
        }
    }
    // far arrivals of this cell, placed by counting: after every bucket whose old cell
    // starts before it and every arrival with a smaller source index
    for (int32_t i = lg; i < nf; i += G) {
        const int32_t p = far_at(i);
        if (p < 0 || p >= n) continue;   // only with bad src_off
        int32_t slot = base;
#pragma unroll
        for (int q = 0; q < 9; ++q)
            if (s_run[grp][q][3] < p) slot += rs[q + 1] - rs[q];
        for (int32_t f = 0; f < nf; ++f) slot += far_at(f) < p ? 1 : 0;
        if (slot >= 0 && slot < lim) r.copy(p, slot, k);
    }
    // moments of the cell from its sorted slots, in slot order per lane (deterministic:
    // the far arrivals sit in the segment in arbitrary order, their slots do not); the
    // barrier makes the group's writes visible to all of its lanes
    __syncthreads();
    const int32_t ncnt = in ? (int32_t)min((int64_t)nk + (f1 - f0), lim - base) : 0;
    // register path (group-uniform): slot q of the cell is position q, held by lane
    // (q + off) % G as round value (q + off) / G
    const bool regs = nf == 0 && ncnt == nk && nk + off <= G * GM_U;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if (regs) {
#pragma unroll
        for (int u = 0; u < GM_U; ++u)
            if (u * G + lg >= off && u * G + lg - off < ncnt) {
                s0 += (double)kvx[u];
                s1 += (double)kvy[u];
                s2 += (double)kvz[u];
            }
        // the partial sum of the slots q = lg modulo G back to lane lg: the reduction's order,
        // and so its bits, do not depend on the shift (here, and for the moments in mom_finish)
        const int from = (lg + off) & (G - 1);
        s0 = __shfl(s0, from, G);
        s1 = __shfl(s1, from, G);
        s2 = __shfl(s2, from, G);
    } else {
        for (int32_t q = lg; q < ncnt; q += G) {
            s0 += (double)r.dvx[base + q];
            s1 += (double)r.dvy[base + q];
            s2 += (double)r.dvz[base + q];
        }
    }
    s0 = group_sum<G>(s0);
    s1 = group_sum<G>(s1);
    s2 = group_sum<G>(s2);
    const double inv_n = ncnt > 0 ? 1.0 / (double)ncnt : 0.0;
    const double U0 = s0 * inv_n, U1 = s1 * inv_n, U2 = s2 * inv_n;
    double acc[NVX];
#pragma unroll
    for (int i = 0; i < NVX; ++i) acc[i] = 0.0;
    if (regs) {
#pragma unroll
        for (int u = 0; u < GM_U; ++u)
            if (u * G + lg >= off && u * G + lg - off < ncnt)
                mom_accum<NVX>((double)kvx[u] - U0, (double)kvy[u] - U1, (double)kvz[u] - U2, acc);
    } else {
        for (int32_t q = lg; q < ncnt; q += G)
            mom_accum<NVX>((double)ld_off(r.dvx, base + q) - U0, (double)ld_off(r.dvy, base + q) - U1,
                           (double)ld_off(r.dvz, base + q) - U2, acc);
    }
    mom_finish<BLK, G, NVX>(sm, acc, grp, lg, in, ncnt, U0, U1, U2,
                            mom + (int64_t)(in ? k : 0) * MOM,
                            grp * G + (regs ? (lg - off) & (G - 1) : lg));
    if (samp_cell && lg < 14) {
        // the lane's time-average sums from the record's entries, rebuilt from the final
        // sums in LDS (the values mom_finish stored) instead of reading the record back;
        // every term with a compile-time entry index (no indexed access to m), the lane's
        // own ones kept
        double m[M_T + 10];
#pragma unroll
        for (int e = 0; e < M_T + 10; ++e) m[e] = mom_entry<BLK, G, NVX>(sm, grp, ncnt, U0, U1, U2, e);
        double t[SQ];
#pragma unroll
        for (int u = 0; u < SQ; ++u) t[u] = 0.0;
#pragma unroll
        for (int e = 0; e < 14; ++e) {
            const double v = sample_term(m, e);
#pragma unroll
            for (int u = 0; u < SQ; ++u) t[u] = lg + u * G == e ? v : t[u];
        }
#pragma unroll
        for (int u = 0; u < SQ; ++u) {
            const int e = lg + u * G;
            if (e < 14) samp[(int64_t)k * SAMP + e] = s_samp[grp][e] + t[u];
        }
    }
}

// Grid of the re-sort's neighbourhoods: the uniform grid, or on the adaptive tree the
// leaves as one row (the leaves just before and after in depth-first order are the side
// buckets; a particle bound for any other leaf takes the far path)
static void rebin_grid(const fp_ctx* c, int32_t& nx, int32_t& ny) {
    nx = c->amr_L >= 0 ? c->ncell : c->cfg.nx;
    ny = c->amr_L >= 0 ? 1 : c->cfg.ny;
}

// pass 1 with G lanes per old cell
template <int G>
static void rebin_count_launch(fp_ctx* c, const fp_particles* src, const int32_t* src_off,
                               hipStream_t s) {
    const int32_t nc = c->ncell;
    int32_t nx, ny;
    rebin_grid(c, nx, ny);
    // cnt, ccnt (far counts), ccur and farn are zero on entry: the previous sort call left
    // them so
    auto launch = [&](auto block) {
        constexpr int BLK = decltype(block)::value;
        const int32_t cblocks = (int32_t)(((int64_t)nc * G + BLK - 1) / BLK);
        hipLaunchKernelGGL((rebin_count_kernel<G, BLK>), dim3(cblocks + FAR_BLOCKS), dim3(BLK), 0, s, nc,
                           nx, src->n, (const int64_t*)src->n_dev, c->cfg.capacity, cblocks, src_off,
                           (const int32_t*)src->key, c->ncnt, c->bidx, c->cnt, c->ccnt, c->farn, c->cmask,
                           c->errcount);
    };
    if ((int64_t)nc * G >= RC_WIDE) launch(std::integral_constant<int, 1024>{});
    else launch(std::integral_constant<int, 256>{});
}

// pass 2 with G lanes per destination cell
template <typename T, int G>
static void rebin_gather_launch(fp_ctx* c, const fp_particles* src, const int32_t* src_off,
                                fp_particles* dst, int32_t* offsets, int32_t* perm, double* mom,
                                double* samp, hipStream_t s) {
    const int32_t nc = c->ncell;
    int32_t nx, ny;
    rebin_grid(c, nx, ny);
    const int64_t n = src->n, cap = c->cfg.capacity;
    const bool two_d = c->cfg.geometry != FP_COUETTE1D;
    Rec<T> r{(const T*)src->x,  two_d ? (const T*)src->y : nullptr, (const T*)src->vx,
             (const T*)src->vy, (const T*)src->vz,                   src->pid,
             (T*)dst->x,        two_d ? (T*)dst->y : nullptr,        (T*)dst->vx,
             (T*)dst->vy,       (T*)dst->vz,                         dst->pid,
             dst->key,          perm};
    const int32_t cblocks = (nc + BIN_BLOCK / G - 1) / (BIN_BLOCK / G);
    if (mom) {
        constexpr int BLK = G > GM_BLOCK ? G : GM_BLOCK;
        const int32_t mblocks = (nc + BLK / G - 1) / (BLK / G);
        if (c->cfg.moment_order == 3)
            hipLaunchKernelGGL((rebin_gather_mom_kernel<T, G, NV_LOW, BLK>), dim3(mblocks), dim3(BLK), 0, s,
                               nc, nx, ny, n, (const int64_t*)src->n_dev, dst->n_dev, cap, src_off,
                               (const int32_t*)c->ncnt, (const int32_t*)c->bidx,
                               (const int32_t*)offsets, (const int32_t*)c->coff, (const int32_t*)c->gidx,
                               c->cnt, c->ccnt, c->ccur, c->farn, r, mom, samp);
        else
            hipLaunchKernelGGL((rebin_gather_mom_kernel<T, G, NV, BLK>), dim3(mblocks), dim3(BLK), 0, s,
                               nc, nx, ny, n, (const int64_t*)src->n_dev, dst->n_dev, cap, src_off,
                               (const int32_t*)c->ncnt, (const int32_t*)c->bidx,
                               (const int32_t*)offsets, (const int32_t*)c->coff, (const int32_t*)c->gidx,
                               c->cnt, c->ccnt, c->ccur, c->farn, r, mom, samp);
        return;
    }
    hipLaunchKernelGGL((rebin_gather_kernel<T, G>), dim3(cblocks + FAR_BLOCKS), dim3(BIN_BLOCK),
                       0, s, nc, nx, ny, n, (const int64_t*)src->n_dev, dst->n_dev, cap, cblocks, src_off,
                       (const int32_t*)c->ncnt,
                       (const int32_t*)c->bidx, (const int32_t*)offsets, (const int32_t*)c->coff,
                       (const int32_t*)c->cwave, (const int32_t*)c->gidx, c->cnt, c->ccnt, c->ccur,
                       c->farn, r);
}

template <typename T>
static void rebin_typed(fp_ctx* c, const fp_particles* src, const int32_t* src_off,
                        fp_particles* dst, int32_t* offsets, int32_t* perm, double* mom,
                        double* samp, hipStream_t s) {
    const int32_t nc = c->ncell;
    // count: about 16 particles per lane (its work per particle is a few loads and a key:
    // measured 4 % faster than 8 at 100 per cell); gather: about 4 (its dependent load
    // chains are short per lane), at most 32 (the moment reduction sums G partials per value)
    switch (lanes_per_cell(c, src->n, FILL_4, 16)) {
        case 4: rebin_count_launch<4>(c, src, src_off, s); break;
        case 8: rebin_count_launch<8>(c, src, src_off, s); break;
        case 16: rebin_count_launch<16>(c, src, src_off, s); break;
        case 32: rebin_count_launch<32>(c, src, src_off, s); break;
        default: rebin_count_launch<64>(c, src, src_off, s); break;
    }
    if (nc <= SMALL_SCAN_CELLS) {
        hipLaunchKernelGGL(rebin_small_scan_kernel, dim3((nc + SSB - 1) / SSB), dim3(SSB), 0, s, nc,
                           (int64_t)c->cfg.capacity, (const int32_t*)c->cnt, (const int32_t*)c->ccnt,
                           offsets, c->coff, (const int32_t*)c->farn, (const uint64_t*)c->cmask,
                           c->cwave, c->gidx);
    } else {
        scan_pair(c->cnt, c->ccnt, 1, nc, c->blocksum, offsets, c->coff, s);
        hipLaunchKernelGGL(rebin_far_place_kernel, dim3(FAR_BLOCKS), dim3(BIN_BLOCK), 0, s,
                           (int64_t)c->cfg.capacity, (const int32_t*)c->farn, (const uint64_t*)c->cmask,
                           (const int32_t*)c->coff, c->ccur, c->cwave, c->gidx);
    }
    int g = lanes_per_cell(c, src->n, FILL_4, 4);
    if (c->cfg.lanes <= 0 && g > 32) g = 32;
    switch (g) {
        case 4: rebin_gather_launch<T, 4>(c, src, src_off, dst, offsets, perm, mom, samp, s); break;
        case 8: rebin_gather_launch<T, 8>(c, src, src_off, dst, offsets, perm, mom, samp, s); break;
        case 16: rebin_gather_launch<T, 16>(c, src, src_off, dst, offsets, perm, mom, samp, s); break;
        case 32: rebin_gather_launch<T, 32>(c, src, src_off, dst, offsets, perm, mom, samp, s); break;
        default: rebin_gather_launch<T, 64>(c, src, src_off, dst, offsets, perm, mom, samp, s); break;
    }
}

int launch_rebin(fp_ctx* c, const fp_particles* src, const int32_t* src_off, fp_particles* dst,
                 int32_t* offsets, int32_t* perm, double* mom, double* samp, hipStream_t s) {
    if (c->ncell > SCAN_MAX_CELLS) return set_err(c, FP_EINVAL, "fp_rebin: too many cells for the scan");
    if (c->cfg.precision == FP_F32)
        rebin_typed<float>(c, src, src_off, dst, offsets, perm, mom, samp, s);
    else
        rebin_typed<double>(c, src, src_off, dst, offsets, perm, mom, samp, s);
    return check_launch(c, "fp_rebin");
}

int launch_bin(fp_ctx* c, const fp_particles* src, fp_particles* dst, int32_t* offsets,
               int32_t* perm, hipStream_t s) {
    // cpair and ccur are zero on entry (fp_init, and every fp_bin leaves them so)
    const int32_t nc = c->ncell;
    const int64_t n = src->n, slots = slots_of(src);
    const int64_t pgrid = (slots + BIN_BLOCK - 1) / BIN_BLOCK;
    if (slots > 0)
        hipLaunchKernelGGL(bin_wave_kernel<false>, dim3((unsigned)pgrid), dim3(BIN_BLOCK), 0, s,
                           src->key, n, (const int64_t*)src->n_dev, nc, (unsigned long long*)c->cpair,
                           c->ccur, (const int32_t*)c->coff, c->cwave, c->cmask, c->errcount);
    if (nc > SCAN_MAX_CELLS) return set_err(c, FP_EINVAL, "fp_bin: too many cells for the scan");
    scan_pair(c->cpair, c->cpair + 1, 2, nc, c->blocksum, offsets, c->coff, s);
    if (slots > 0)
        hipLaunchKernelGGL(bin_wave_kernel<true>, dim3((unsigned)pgrid), dim3(BIN_BLOCK), 0, s,
                           src->key, n, (const int64_t*)src->n_dev, nc, (unsigned long long*)c->cpair,
                           c->ccur, (const int32_t*)c->coff, c->cwave, c->cmask, c->errcount);
    if (c->cfg.precision == FP_F32)
        gather_dispatch<float>(c, src, dst, offsets, perm, s);
    else
        gather_dispatch<double>(c, src, dst, offsets, perm, s);
    return check_launch(c, "fp_bin");
}

}  // namespace fpg
