// The chain kernel of the LITE training (lite_train_kernel) on the CPU against plain loops with the
// same bfloat16 roundings: the fragments it leaves for the weight gradients bit for bit, the
// loss and the bias gradients up to the order of their sums.  Tiles of 32 and of 64 samples, a
// ragged last one, workgroups that take several.
#include "fp_lite.hip"

int fpg::set_err(fp_ctx*, int code, const std::string&) { return code; }
int fpg::check_launch(fp_ctx*, const char*) { return FP_OK; }
int fpg::launch_closure_nn(fp_ctx*, const float*, const float*, double, double, double, const double*, double*, int32_t*,
                           hipStream_t) {
    return FP_OK;
}

static uint64_t rng_state = 7;
static float rnd() {   // (-1, 1)
    rng_state = rng_state * 6364136223846793005ull + 1442695040888963407ull;
    return (float)(int32_t)(rng_state >> 32) * 0x1p-31f;
}
static float bf(float v) { return (float)(__bf16)v; }

template <int CT>
static int run(int64_t B, int grid) {
    constexpr int NH = lite::NH, NF = lite::NF, NO = lite::NO, W[6] = {0, NF, NH, NH, NH, NH};
    const int64_t tiles = (B + 32 * CT - 1) / (32 * CT), groups = tiles * 2 * CT;
    emu::Buffer<float> p(lite::N_PARAMS), feats(B * NF), T(B * NO), bpart(grid * lite::BROW);
    emu::Buffer<__bf16> img(lite::FR_N * 512), sf(lite::SF_N * groups * 512);
    emu::Buffer<double> lpart(grid);
    for (int64_t i = 0; i < lite::N_PARAMS; ++i) p[i] = 0.12f * rnd();
    for (int64_t i = lite::OFF_W5 + 9 * NH; i < lite::OFF_B5; ++i) p[i] = 0.0f;
    for (int i = 0; i < 16; ++i) {
        p[lite::OFF_B5 + i] = i < 9 ? rnd() : 0.0f;
        p[lite::OFF_XM + i] = rnd();
        p[lite::OFF_XS + i] = 1.0f + 0.4f * rnd();
        p[lite::OFF_YM + i] = rnd();
        p[lite::OFF_YS + i] = 1.0f + 0.4f * rnd();
    }
    for (int64_t i = 0; i < B * NF; ++i) feats[i] = 2.0f * rnd();
    for (int64_t i = 0; i < B * NO; ++i) T[i] = 2.0f * rnd();
    emu::launch(lite::FR_N, 64, [&] { lite::lite_train_pack_kernel(p, img); });
    emu::launch(grid, 512, [&] { lite::lite_train_kernel<CT>(B, p, img, feats, T, groups, sf, bpart, lpart); });

    const int64_t offb[6] = {0, lite::OFF_B1, lite::OFF_B2, lite::OFF_B3, lite::OFF_B4, lite::OFF_B5};
    std::vector<double> bias(lite::BROW, 0.0), babs(lite::BROW, 0.0);
    double loss = 0.0, dev = 0.0;
    // fragment f (32 units of a 16-sample group): unit `unit`, sample n
    auto frag = [&](int f, int unit, int64_t n) {
        return (float)sf[(((int64_t)f * groups + n / 16) * 64 + unit % 32 + 32 * (n % 16 / 8)) * 8 + n % 8];
    };
    for (int64_t n = 0; n < tiles * 32 * CT; ++n) {
        const bool real = n < B;
        const int64_t m = real ? n : B - 1;   // padding repeats the last sample, without a gradient
        std::vector<float> h[5], dz(NO, 0.0f);
        std::vector<bool> on[5];
        for (int k = 0; k < NF; ++k) h[0].push_back(bf((feats[m * NF + k] - p[lite::OFF_XM + k]) / p[lite::OFF_XS + k]));
        auto product = [&](int layer, int unit) {
            float acc = 0.0f;
            for (int k = 0; k < W[layer]; ++k) acc += bf(p[lite::off_w(layer) + unit * W[layer] + k]) * h[layer - 1][k];
            return acc + p[offb[layer] + unit];
        };
        for (int l = 1; l < 5; ++l)
            for (int u = 0; u < NH; ++u) {
                const float z = product(l, u);
                on[l].push_back(z > 0.0f);
                h[l].push_back(bf(fmaxf(z, 0.0f)));
            }
        for (int o = 0; o < 9; ++o) {
            const double e = (double)product(5, o) - ((double)T[m * NO + o] - p[lite::OFF_YM + o]) / p[lite::OFF_YS + o];
            if (real) {
                loss += e * e;
                dz[o] = (float)(2.0 * e * (1.0 / (double)B));
                bias[4 * NH + o] += dz[o];
                babs[4 * NH + o] += fabs(dz[o]);
            }
        }
        auto differ = [&](const char* what, int l, int unit, float got, float want) {
            if (got == want) return false;
            fprintf(stderr, "%s of layer %d, unit %d, sample %ld of %ld (tiles of %d): %g, not %g\n", what, l, unit, (long)n,
                    (long)B, 32 * CT, got, want);
            return true;
        };
        for (int u = 0; u < NF; ++u)
            if (differ("input", 0, u, frag(lite::SF_H0, u, n), h[0][u])) return 1;
        for (int u = 0; u < NO; ++u)
            if (differ("output gradient", 5, u, frag(lite::SF_DY, u, n), bf(dz[u]))) return 1;
        for (int l = 4; l > 0; --l) {
            std::vector<float> prev(NH);
            const int K = l == 4 ? NO : NH;   // outputs of the layer behind
            for (int u = 0; u < NH; ++u) {
                float acc = 0.0f;
                for (int k = 0; k < K; ++k) acc += bf(p[lite::off_w(l + 1) + k * NH + u]) * bf(dz[k]);
                prev[u] = on[l][u] ? acc : 0.0f;
                bias[(l - 1) * NH + u] += real ? prev[u] : 0.0;
                babs[(l - 1) * NH + u] += real ? fabs(prev[u]) : 0.0;
                if (differ("activation", l, u, frag(lite::SF_H + (l - 1) * lite::NT + u / 32, u, n), h[l][u])) return 1;
                if (differ("gradient", l, u, frag(lite::SF_Z + (l - 1) * lite::NT + u / 32, u, n), bf(prev[u]))) return 1;
            }
            dz = prev;
        }
    }
    double got = 0.0;
    for (int w = 0; w < grid; ++w) got += lpart[w];
    if (!(fabs(got - loss) <= 1e-12 * loss)) return fprintf(stderr, "loss %g, not %g\n", got, loss), 1;
    for (int i = 0; i < lite::BROW; ++i) {
        double b = 0.0;
        for (int w = 0; w < grid; ++w) b += (double)bpart[(int64_t)w * lite::BROW + i];
        // FP32 sums of B terms
        if (!(fabs(b - bias[i]) <= B * 0x1p-24 * babs[i])) return fprintf(stderr, "bias gradient %d: %g, not %g\n", i, b, bias[i]), 1;
    }
    return 0;
}

int main() { return run<1>(5, 1) || run<1>(70, 2) || run<2>(64, 1) || run<2>(200, 3); }
