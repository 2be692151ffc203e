// The count pass of the re-sort (rebin_count_kernel) on the CPU, for src_offsets as the contract
// has them and for others: no access out of range, every source index that the gather can
// read is one of a particle, and for proper offsets the buckets, counts and far list are right.
#include "fp_bin.hip"

using namespace fpg;

int fpg::set_err(fp_ctx*, int code, const std::string&) { return code; }
int fpg::check_launch(fp_ctx*, const char*) { return FP_OK; }

static uint64_t rng_state = 1;
static uint32_t rnd(uint32_t n) {
    rng_state = rng_state * 6364136223846793005ull + 1442695040888963407ull;
    return (uint32_t)(rng_state >> 33) % n;
}
static int fail(const char* what, int G, int BLK, int kind, int64_t at, int64_t v) {
    fprintf(stderr, "%s: G %d, workgroups of %d, offsets %d: at %ld value %ld\n", what, G, BLK, kind, (long)at, (long)v);
    return 1;
}

enum { PROPER, DECREASING, BEYOND, NEGATIVE, EXTREME };

template <int G, int BLK>
static int run(int kind, int nx, int ny, int ppc) {
    const int nc = nx * ny;
    std::vector<int32_t> count(nc), start(nc + 1, 0);
    for (int c = 0; c < nc; ++c) {
        count[c] = rnd(8) == 0 ? 0 : (int)rnd(2 * ppc + 1);
        start[c + 1] = start[c] + count[c];
    }
    const int64_t n = start[nc] + 5;   // and a few ungrouped ones
    emu::Buffer<int32_t> off(nc + 1), key(n), bend(9 * nc), bidx(n), cnt(nc + 1, 0), fcnt(nc + 1, 0), farn(1, 0);
    emu::Buffer<uint64_t> flist(n);
    emu::Buffer<unsigned long long> err(1, 0);
    for (int c = 0; c <= nc; ++c) off[c] = start[c];
    for (int c = 0; c <= nc; ++c) {
        const bool hit = rnd(6) == 0;
        if (kind == DECREASING && hit) off[c] = (int32_t)rnd((uint32_t)n);
        if (kind == BEYOND && hit) off[c] = (int32_t)(n + rnd(1000));
        if (kind == NEGATIVE && hit) off[c] = -(int32_t)rnd(1000) - 1;
        if (kind == EXTREME && hit) off[c] = rnd(2) ? INT32_MAX - (int32_t)rnd(9) : INT32_MIN + (int32_t)rnd(9);
    }
    int bad = 0;
    for (int64_t j = 0, c = 0; j < n; ++j) {
        while (c < nc - 1 && j >= start[c + 1]) ++c;
        const int x = (int)c % nx + (int)rnd(3) - 1, y = (int)c / nx + (int)rnd(3) - 1, r = (int)rnd(20);
        key[j] = x >= 0 && x < nx && y >= 0 && y < ny ? y * nx + x : (int32_t)c;
        if (r == 0) key[j] = (int32_t)rnd(nc);     // anywhere
        if (r == 1) key[j] = nc;                   // deleted
        if (r == 2 && rnd(4) == 0) {
            const int32_t wrong[] = {-1, nc + 1, INT32_MIN, INT32_MAX};
            key[j] = wrong[rnd(4)];
            ++bad;
        }
    }
    const int blocks = (nc * G + BLK - 1) / BLK;
    emu::launch(blocks + FAR_BLOCKS, BLK, [&] {
        rebin_count_kernel<G, BLK>(nc, nx, n, nullptr, n, blocks, off, key, bend, bidx, cnt, fcnt, farn, flist, err);
    });
    // what the gather reads: bucket d of cell c at max(off[c], 0) + [bend[d - 1], bend[d])
    for (int c = 0; c < nc; ++c) {
        const int64_t s = max(off[c], 0);
        int32_t before = 0;
        for (int d = 0; d < 9; ++d) {
            const int32_t end = bend[9 * c + d];
            if (end < before || (end > before && s + end > n)) return fail("bucket end", G, BLK, kind, 9 * c + d, end);
            for (int64_t q = s + before; q < s + end; ++q)
                if (bidx[q] < 0 || bidx[q] >= n) return fail("source index", G, BLK, kind, q, bidx[q]);
            before = end;
        }
    }
    if (kind != PROPER) return 0;
    std::vector<int32_t> want_cnt(nc + 1, 0), want_far(nc + 1, 0);
    std::vector<uint64_t> far, got;
    for (int c = 0; c < nc; ++c) {
        std::vector<int32_t> b[9];
        for (int j = start[c]; j < start[c + 1]; ++j) {
            const int32_t k = key[j];
            if (k < 0 || k >= nc) continue;
            const int dx = k % nx - c % nx, dy = k / nx - c / nx;
            if (dx < -1 || dx > 1 || dy < -1 || dy > 1) {
                far.push_back((uint64_t)k << 32 | (uint32_t)j);
                ++want_far[k];
            } else {
                b[3 * dy + dx + 4].push_back(j);
            }
            ++want_cnt[k];
        }
        int32_t at = 0;
        for (int d = 0; d < 9; ++d) {
            for (int32_t j : b[d])
                if (bidx[start[c] + at++] != j) return fail("bucket", G, BLK, kind, start[c] + at - 1, bidx[start[c] + at - 1]);
            if (bend[9 * c + d] != at) return fail("bucket end", G, BLK, kind, 9 * c + d, bend[9 * c + d]);
        }
    }
    for (int64_t j = start[nc]; j < n; ++j)
        if (key[j] >= 0 && key[j] < nc) {
            far.push_back((uint64_t)key[j] << 32 | (uint32_t)j);
            ++want_cnt[key[j]];
            ++want_far[key[j]];
        }
    for (int k = 0; k <= nc; ++k)
        if (cnt[k] != want_cnt[k] || fcnt[k] != want_far[k]) return fail("count", G, BLK, kind, k, cnt[k]);
    got.assign(flist.p, flist.p + farn[0]);
    std::sort(got.begin(), got.end());
    std::sort(far.begin(), far.end());
    if (got != far) return fail("far list", G, BLK, kind, farn[0], (int64_t)far.size());
    if ((int)err[0] != bad) return fail("invalid keys", G, BLK, kind, 0, (int64_t)err[0]);
    return 0;
}

template <int G>
static int all(int kind) {
    // cells of a few and of many particles (more of them than a wave stages, RC_STAGE)
    for (int ppc : {3, 20, 300})
        if (run<G, 256>(kind, 7, 5, ppc)) return 1;
    return run<G, 1024>(kind, 9, 4, 12) || run<G, 256>(kind, 41, 1, 9) || run<G, 256>(kind, 1, 3, 2);
}

int main(int argc, char** argv) {
    const int kind = atoi(argv[1]);
    for (int rep = 0; rep < 2; ++rep)
        if (all<4>(kind) || all<8>(kind) || all<16>(kind) || all<32>(kind) || all<64>(kind)) return 1;
    return 0;
}
