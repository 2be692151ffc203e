// The training kernel of the 27-feature network (nn_train_kernel and the reduction behind it) on
// the CPU against plain loops with the same bfloat16 roundings, both losses, tiles of 32 and of
// 64 samples, a ragged last one, workgroups that take several.  The loops take the exponential
// from libm: a last bit of an activation may differ and round to the next bfloat16 now and
// then, so the gradient is compared within 2^-7 of its tensor's rms (a bfloat16 ulp) and the
// loss within 2^-8.
#include "fp_nn.hip"

int fpg::set_err(fp_ctx*, int code, const std::string&) { return code; }
int fpg::check_launch(fp_ctx*, const char*) { return FP_OK; }
int fpg::launch_closure_nn(fp_ctx*, const float*, const float*, double, double, double, const double*, double*, int32_t*,
                           hipStream_t) {
    return FP_OK;
}

using namespace fpg;

static uint64_t rng_state = 11;
static float rnd() {   // (-1, 1)
    rng_state = rng_state * 6364136223846793005ull + 1442695040888963407ull;
    return (float)(int32_t)(rng_state >> 32) * 0x1p-31f;
}
static double bf(double v) { return (double)(float)(__bf16)(float)v; }

template <int CT, int KIND>
static int run(int64_t B, int grid) {
    const int W[5] = {0, NF, NH, NH, NH}, M[5] = {0, NH, NH, NH, NO};
    const int ow[5] = {0, OFF_W1, OFF_W2, OFF_W3, OFF_W4}, ob[5] = {0, OFF_B1, OFF_B2, OFF_B3, OFF_B4};
    emu::Buffer<float> p(N_PARAMS), feats(B * NF), T(B * NO), part((int64_t)grid * GROW), grad(N_PARAMS, 0), loss(1);
    emu::Buffer<double> sys(B * 90), lpart(grid);
    emu::Buffer<__bf16> img(FR_N * 512);
    for (int64_t i = 0; i < N_PARAMS; ++i) p[i] = 0.2f * rnd();
    for (int i = OFF_W4 + 9 * NH; i < OFF_B4; ++i) p[i] = 0.0f;
    for (int i = 0; i < NO; ++i) {
        p[OFF_B4 + i] = i < 9 ? rnd() : 0.0f;
        p[OFF_YM + i] = rnd();
        p[OFF_YS + i] = 1.0f + 0.4f * rnd();
    }
    for (int i = 0; i < NF; ++i) p[OFF_XS + i] = 1.0f + 0.4f * rnd();
    for (int64_t i = 0; i < B * NF; ++i) feats[i] = 2.0f * rnd();
    for (int64_t i = 0; i < B * NO; ++i) T[i] = 2.0f * rnd();
    for (int64_t i = 0; i < B * 90; ++i) sys[i] = rnd();
    emu::launch(FR_N, 64, [&] { nn_train_pack_kernel(p, img); });
    emu::launch(grid, 256 * CT, [&] { nn_train_kernel<CT, KIND>(B, p, img, feats, T, sys, part, lpart); });
    emu::launch((GROW / 4 + 63) / 64 + 1, RED_BLOCK, [&] { nn_reduce_kernel<false>(grid, part, lpart, B, grad, loss, AdamArgs{}); });

    std::vector<double> g(N_PARAMS, 0.0);
    double want = 0.0;
    for (int64_t n = 0; n < B; ++n) {
        std::vector<double> h[5], d[5], dz(NO, 0.0);
        for (int k = 0; k < NF; ++k) h[0].push_back(bf((feats[n * NF + k] - p[OFF_XM + k]) / p[OFF_XS + k]));
        for (int l = 1; l < 5; ++l)
            for (int u = 0; u < M[l]; ++u) {
                double z = p[ob[l] + u];
                for (int k = 0; k < W[l]; ++k) z += bf(p[ow[l] + u * W[l] + k]) * h[l - 1][k];
                const double s = 1.0 / (1.0 + exp(-z));
                h[l].push_back(l < 4 ? bf(z * s) : z);
                d[l].push_back(s * (1.0 + z * (1.0 - s)));
            }
        if (KIND == 0) {
            for (int o = 0; o < 9; ++o) {
                const double e = h[4][o] - ((double)T[n * NO + o] - p[OFF_YM + o]) / p[OFF_YS + o];
                want += e * e / (double)B;
                dz[o] = 2.0 * e / (double)B;
            }
        } else {
            double y[9], r[9];
            for (int o = 0; o < 9; ++o)
                y[o] = h[4][o] * p[OFF_YS + o] + p[OFF_YM + o] + (o == 0 || o == 3 || o == 5 ? 5.0 * feats[n * NF + 25] : 0.0);
            for (int i = 0; i < 9; ++i) {
                r[i] = -sys[n * 90 + 81 + i];
                for (int k = 0; k < 9; ++k) r[i] += sys[n * 90 + 9 * i + k] * y[k];
                want += r[i] * r[i] / (double)B;
            }
            for (int o = 0; o < 9; ++o)
                for (int i = 0; i < 9; ++i) dz[o] += 2.0 * sys[n * 90 + 9 * i + o] * r[i] / (double)B * p[OFF_YS + o];
        }
        for (int l = 4; l > 0; --l) {
            std::vector<double> prev(W[l], 0.0);
            for (int u = 0; u < M[l]; ++u) {
                g[ob[l] + u] += dz[u];
                for (int k = 0; k < W[l]; ++k) {
                    g[ow[l] + u * W[l] + k] += bf(dz[u]) * h[l - 1][k];
                    prev[k] += bf(dz[u]) * bf(p[ow[l] + u * W[l] + k]);
                }
            }
            if (l > 1)
                for (int k = 0; k < W[l]; ++k) prev[k] *= d[l - 1][k];
            dz = prev;
        }
    }
    if (!(fabs((double)loss[0] - want) <= 0x1p-8 * want)) return fprintf(stderr, "loss %g, not %g\n", loss[0], want), 1;
    for (int l = 1; l < 5; ++l)
        for (int part_of = 0; part_of < 2; ++part_of) {   // weights, biases
            const int o = part_of ? ob[l] : ow[l], n = part_of ? M[l] : M[l] * W[l];
            double rms = 0.0;
            for (int i = 0; i < n; ++i) rms += g[o + i] * g[o + i] / n;
            for (int i = 0; i < n; ++i)
                if (!(fabs(grad[o + i] - g[o + i]) <= 0x1p-7 * sqrt(rms)))
                    return fprintf(stderr, "%s %d, entry %d: %g, not %g (rms %g; tiles of %d, loss %d)\n",
                                   part_of ? "bias" : "weights", l, i, grad[o + i], g[o + i], sqrt(rms), 32 * CT, KIND), 1;
        }
    return 0;
}

int main() {
    return run<1, 0>(5, 1) || run<1, 1>(70, 2) || run<1, 0>(100, 2) || run<2, 0>(200, 3) || run<2, 1>(150, 1) ||
           run<2, 1>(200, 3);
}
