// fp_lite.hip -- the paper's LITE surrogate on MFMA: 16 low-order inputs -> 256 -> 256 ->
// 256 -> 256 (ReLU) -> 9 (Secs. "Phase 1-2", "Neural Network Architecture", "Phase 3").
//
// Inference is one persistent kernel: every wave keeps 32 cells (the MFMA columns) in
// registers through all five layers, from the moment record to the update record, and the
// workgroup streams the BF16 weights through LDS (the 408 KB do not fit in LDS together; a
// 256 x 256 layer is 128 KB).  The activations never leave the registers: the columns of
// every next-layer weight matrix are permuted so that the rows a lane holds after one layer
// are exactly the k-slots it feeds into the next (the permutation of fp_nn.hip, over 16
// k-steps).  Training is a kernel for the chain of a batch tile (forward, loss and backward,
// activations kept on the CU), one for the weight gradients (split-K MFMA) and one that
// reduces them in a fixed order (bitwise reproducible) and takes the Adam step on FP32
// master weights.
//
// Inputs (solver units, then standardised): rho, T, U (3), Pi (11 12 13 22 23 33), q (3),
// DM2 = <|c|^2>, nu = 1/tau; targets Ct (6) and Gamma (3) of the update record, in solver
// units, standardised.
#include "fp_closure_dev.h"
#include "fp_mlp_dev.h"

#include <algorithm>
#include <cmath>
#include <new>
#include <string>

namespace fpg {
namespace lite {

constexpr int NF = 16, NH = 256, NO = 16;
constexpr int NT = NH / 32;   // 32-row output tiles of a hidden layer
constexpr int KS = NH / 16;   // 16-row k-steps of a hidden layer's input
// flat FP32 parameters (include/fp.h)
constexpr int64_t OFF_W1 = 0, OFF_B1 = 4096, OFF_W2 = 4352, OFF_B2 = 69888, OFF_W3 = 70144,
                  OFF_B3 = 135680, OFF_W4 = 135936, OFF_B4 = 201472, OFF_W5 = 201728,
                  OFF_B5 = 205824, OFF_XM = 205840, OFF_XS = 205856, OFF_YM = 205872,
                  OFF_YS = 205888, N_PARAMS = 205904, N_TRAIN = 205840;
// BF16 fragment image: layer 1 NT tiles x 1 k-step, layers 2-4 NT x KS, layer 5 1 x KS
constexpr int IMG_L1 = 0, IMG_L2 = 4096, IMG_L3 = 69632, IMG_L4 = 135168, IMG_L5 = 200704,
              IMG_BF = 208896;
// FP32 section: biases, scalers, and an identity output scaler (16 zeros, 16 ones) for the
// check kernel, which receives normalised coefficients
constexpr int SEC_B1 = 0, SEC_B2 = 256, SEC_B3 = 512, SEC_B4 = 768, SEC_B5 = 1024, SEC_XM = 1040,
              SEC_XS = 1056, SEC_YM = 1072, SEC_YS = 1088, SEC_ID = 1104, SEC_N = 1136;
constexpr int LDS_BF = NT * KS * 512;           // one hidden layer: 65536 BF16 (128 KB)

static_assert(IMG_L2 - IMG_L1 == NT * 512 && IMG_L3 - IMG_L2 == LDS_BF && IMG_L5 - IMG_L4 == LDS_BF &&
                  IMG_BF - IMG_L5 == KS * 512,
              "image layout");
static_assert(OFF_B3 - OFF_B2 == OFF_B2 - OFF_B1 && OFF_B4 - OFF_B3 == OFF_B2 - OFF_B1, "parameter layout");
static_assert(OFF_B5 + NO == N_TRAIN && OFF_YS + NO == N_PARAMS, "parameter layout");

// k-slot K of a hidden layer's input holds activation row perm_k(K) of the previous layer
__device__ __forceinline__ int perm_k(int K) {
    const int s = K >> 4, h = (K >> 3) & 1, i = K & 7;
    return 16 * s + 8 * (i >> 2) + 4 * h + (i & 3);
}

// ---------------------------------------------------------------------------------------
// FP32 parameters -> permuted BF16 fragment image ([tile][k-step][lane][8]) + FP32 section
__global__ void lite_pack_kernel(const float* __restrict__ p, __bf16* __restrict__ img,
                                 float* __restrict__ sec) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < IMG_BF) {
        int base, ks_n, layer;
        if (t < IMG_L2) { layer = 1; base = IMG_L1; ks_n = 1; }
        else if (t < IMG_L3) { layer = 2; base = IMG_L2; ks_n = KS; }
        else if (t < IMG_L4) { layer = 3; base = IMG_L3; ks_n = KS; }
        else if (t < IMG_L5) { layer = 4; base = IMG_L4; ks_n = KS; }
        else { layer = 5; base = IMG_L5; ks_n = KS; }
        const int e = t - base;
        const int i = e & 7, lane = (e >> 3) & 63, frag = e >> 9;
        const int ks = frag % ks_n, mt = frag / ks_n;
        const int m = mt * 32 + (lane & 31), h = lane >> 5;
        const int K = ks * 16 + 8 * h + i;
        float v;
        if (layer == 1) v = p[OFF_W1 + m * NF + K];
        else if (layer == 2) v = p[OFF_W2 + m * NH + perm_k(K)];
        else if (layer == 3) v = p[OFF_W3 + m * NH + perm_k(K)];
        else if (layer == 4) v = p[OFF_W4 + m * NH + perm_k(K)];
        else v = m < NO ? p[OFF_W5 + m * NH + perm_k(K)] : 0.0f;
        img[t] = (__bf16)v;
    }
    if (t < SEC_N) {
        float v;
        if (t < SEC_B5) v = p[OFF_B1 + (t / NH) * (OFF_B2 - OFF_B1) + t % NH];
        else if (t < SEC_XM) v = p[OFF_B5 + t - SEC_B5];
        else if (t < SEC_XS) v = p[OFF_XM + t - SEC_XM];
        else if (t < SEC_YM) v = p[OFF_XS + t - SEC_XS];
        else if (t < SEC_YS) v = p[OFF_YM + t - SEC_YM];
        else if (t < SEC_ID) v = p[OFF_YS + t - SEC_YS];
        else v = t < SEC_ID + 16 ? 0.0f : 1.0f;
        sec[t] = v;
    }
}

// the 16 inputs of one cell (FP64 arithmetic, FP32 result) and its tau (eq. tau):
// rho, T, U, Pi_ij = rho (P_ij - theta delta_ij), q_i = rho S_i / 2, DM2 = 3 theta, nu = 1/tau
__device__ __forceinline__ void cell_inputs(const fp_config& g, const double* __restrict__ m, double nv,
                                            float f[NF], double& tau) {
    const double N = m[M_N], th = m[M_TH];
    const double ndens = N * nv;
    const double rho = ndens * g.mass;
    tau = cell_tau(g, ndens, th);
    f[0] = (float)rho;
    f[1] = (float)(th * g.mass / g.kB);
#pragma unroll
    for (int q = 0; q < 3; ++q) f[2 + q] = (float)m[M_U + q];
    const double d6[6] = {1, 0, 0, 1, 0, 1};
#pragma unroll
    for (int q = 0; q < 6; ++q) f[5 + q] = (float)(rho * (m[M_P + q] - th * d6[q]));
    // S_i = T_ikk: T111 T112 T113 T122 T123 T133 T222 T223 T233 T333
    const double S1 = m[M_T + 0] + m[M_T + 3] + m[M_T + 5];
    const double S2 = m[M_T + 1] + m[M_T + 6] + m[M_T + 8];
    const double S3 = m[M_T + 2] + m[M_T + 7] + m[M_T + 9];
    f[11] = (float)(0.5 * rho * S1);
    f[12] = (float)(0.5 * rho * S2);
    f[13] = (float)(0.5 * rho * S3);
    f[14] = (float)(3.0 * th);
    f[15] = (float)(1.0 / tau);
}

// ---------------------------------------------------------------------------------------
// fused inference.  MODE 0: y[cell][16] = standardised network outputs (rows 9..15 zero);
// MODE 1: y[cell][16] = normalised coefficients [tau Ct - 5 eps_hat I (6), tau sqrt(theta)
// Gamma (3), 0...] from the de-standardised outputs, for the check kernel with the identity
// scaler; MODE 2 (records through third order, unchecked): the update records themselves.
// Cells without inputs (N <= 1 or theta <= 0) are evaluated on zero inputs in mode 0 and get
// zeros in mode 1.
//
// A workgroup of W waves takes 32 cells per wave through the five layers in registers and goes
// on to its next cells (a workgroup per CU).  The weights come in 26 chunks (layer 1, eight
// 32-row tiles of each hidden layer, layer 5) through two LDS slots: chunk k + 1 is written and
// chunk k + 3 loaded while chunk k multiplies, a barrier per chunk.  The next cells' moment
// records trickle into LDS meanwhile, a 1 KB piece per chunk, and each tile's ReLU runs
// between the next tile's MFMAs.  1e6 cells: 472 us in mode 2; a workgroup per 256 cells that
// staged whole 128 KB layers between barriers and left the records to the check kernel took
// 655 us.  Of a pass of 23 us at full clock the hidden layers take 16 (two thirds of their
// MFMA rate), the FP64 inputs and records 5, the first layer 1.4.  Four waves of 64 cells
// (half the LDS reads, twice the registers) were slower (490 to 600 us), and without any
// fragment reads it would take 445: the LDS is not the bound.  The eight waves fill their 256
// registers; in mode 2 two of a lane's and 123 scalar ones (to lanes) are spilled.
constexpr int CH_N = 26, CH_BF = KS * 512;   // chunks of a pass, bfloat16 of a chunk (layer 1: half)
constexpr int MROW = MOM + 1;   // LDS row of a record: rows start on different banks

template <int W>
struct InferShared {
    __attribute__((aligned(16))) __bf16 w[2][CH_BF];
    double mom[W][32 * MROW];
    __attribute__((aligned(16))) float sec[SEC_N];
};

template <int W>
struct InferPass {
    InferShared<W>& sm;
    const __bf16* gimg;
    const double* mom;
    int32_t ncell, next;      // first cell of the wave's next pass
    int tid, lane, wave, h, c;
    static constexpr int BLOCK = 64 * W, SQ = 16 / W;   // 16-byte loads of a chunk per thread
    bf16x8 st[2][SQ];         // chunks on their way to LDS
    double2 piece;            // a piece of the next records on its way to LDS

    // chunk k (mod CH_N) into the register set s
    __device__ __forceinline__ void load(int k, int s) {
        const int kk = k % CH_N;
        const __bf16* src = gimg + (kk == 0 ? IMG_L1 : IMG_L2 + (kk - 1) * CH_BF);
#pragma unroll
        for (int q = 0; q < SQ; ++q)
            if (kk != 0 || 2 * q < SQ) st[s][q] = *(const bf16x8*)(src + (q * BLOCK + tid) * 8);
    }
    __device__ __forceinline__ void store(int k, int s) {
        const int kk = k % CH_N;
#pragma unroll
        for (int q = 0; q < SQ; ++q)
            if (kk != 0 || 2 * q < SQ) *(bf16x8*)(sm.w[kk & 1] + (q * BLOCK + tid) * 8) = st[s][q];
    }
    // piece q of the next records (four of them, 16 bytes a lane), to registers and to LDS
    __device__ __forceinline__ void load_piece(int q) {
        const int64_t cell = min(next + 4 * q + (lane >> 4), ncell - 1);
        const double* p = mom + cell * MOM + (lane & 15) * 2;
        piece = make_double2(p[0], p[1]);
    }
    __device__ __forceinline__ void store_piece(int q) {
        double* d = sm.mom[wave] + (4 * q + (lane >> 4)) * MROW + (lane & 15) * 2;
        d[0] = piece.x;
        d[1] = piece.y;
    }
    // the traffic behind chunk K, once it is in LDS for everyone (lds_barrier)
    template <int K>
    __device__ __forceinline__ void move() {
        store(K + 1, (K + 1) & 1);
        load(K + 3, (K + 1) & 1);
        // pieces 0 .. 7 in chunks 2, 3, ...
        if constexpr (K >= 3 && K - 3 < 8) store_piece(K - 3);
        if constexpr (K >= 2 && K - 2 < 8) load_piece(K - 2);
    }
    // chunk K times bin into acc (16 k-steps); every fragment is read AHEAD k-steps before its
    // products (one wave per SIMD: nothing else hides the LDS latency), between(s) runs
    // between the products of step s and those of step s + 1
    template <int K, typename F>
    __device__ __forceinline__ void products(const bf16x8 (&bin)[KS], f32x16& acc, F between) {
        constexpr int AHEAD = 4;
        const __bf16* w = sm.w[K & 1] + lane * 8;
        bf16x8 a[AHEAD];
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) a[s] = *(const bf16x8*)(w + s * 512);
        move<K>();
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            acc = mfma32(a[s % AHEAD], bin[s], acc);
            if (s + AHEAD < KS) a[s % AHEAD] = *(const bf16x8*)(w + (s + AHEAD) * 512);
            between(s);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __device__ __forceinline__ f32x16 bias_of(const float* b, int mt) const {
        f32x16 v;
#pragma unroll
        for (int jq = 0; jq < 4; ++jq) {
            const float4 q = *(const float4*)(b + mt * 32 + 8 * jq + 4 * h);
            v[4 * jq + 0] = q.x;
            v[4 * jq + 1] = q.y;
            v[4 * jq + 2] = q.z;
            v[4 * jq + 3] = q.w;
        }
        return v;
    }
};

// rows 2 i, 2 i + 1 of the lane's tile mt through the ReLU
__device__ __forceinline__ void relu_pair(const f32x16& acc, bf16x8 (&bout)[KS], int mt, int i) {
#pragma unroll
    for (int j = 2 * i; j < 2 * i + 2; ++j) bout[2 * mt + (j >> 3)][j & 7] = (__bf16)fmaxf(acc[j], 0.0f);
}

// tiles MT .. of a hidden layer whose first tile is chunk K0; prev: the tile before this one
template <int W, int K0, int MT>
__device__ __forceinline__ void hidden_tiles(InferPass<W>& P, const float* bias, const bf16x8 (&bin)[KS],
                                             bf16x8 (&bout)[KS], const f32x16& prev) {
    if constexpr (MT < NT) {
        f32x16 acc = P.bias_of(bias, MT);
        lds_barrier();
        P.template products<K0 + MT>(bin, acc, [&](int s) {
            if (MT > 0 && (s & 1)) relu_pair(prev, bout, MT - 1, s >> 1);
        });
        hidden_tiles<W, K0, MT + 1>(P, bias, bin, bout, acc);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) relu_pair(prev, bout, NT - 1, i);
    }
}

template <int W, int MODE>
__global__ __launch_bounds__(64 * W) void lite_infer_kernel(fp_config g, int32_t ncell,
                                                               const double* __restrict__ mom,
                                                               const double* __restrict__ nvol,
                                                               const __bf16* __restrict__ gimg,
                                                               const float* __restrict__ gsec,
                                                               float* __restrict__ yout, double* __restrict__ rec,
                                                               int32_t* __restrict__ status, double relax) {
    __shared__ InferShared<W> sm;
    constexpr int BLOCK = 64 * W, CELLS = 32;   // cells of a wave and pass
    InferPass<W> P{sm, gimg, mom, ncell};
    P.tid = threadIdx.x;
    P.lane = threadIdx.x & 63;
    P.wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    P.h = P.lane >> 5;
    P.c = P.lane & 31;
    for (int t = threadIdx.x; t < SEC_N; t += BLOCK) sm.sec[t] = gsec[t];
    P.next = (blockIdx.x * W + P.wave) * CELLS;
    P.load(0, 0);
    P.load(1, 1);
    {
        double2 all[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            P.load_piece(q);
            all[q] = P.piece;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            P.piece = all[q];
            P.store_piece(q);
        }
    }
    P.store(0, 0);
    P.load(2, 0);
    // st[1] holds chunk 1, st[0] chunk 2: chunk k waits in set k & 1
    for (int32_t first = blockIdx.x * W * CELLS; first < ncell; first += gridDim.x * W * CELLS) {
        // no address is kept in registers over the loop (spilled, each would be reloaded behind
        // the weights in flight)
        __asm__ volatile("" : "+v"(P.tid), "+v"(P.lane), "+v"(P.h), "+v"(P.c)::"memory");
        const int lane = P.lane, h = P.h, c = P.c;
        // lane = cell (the upper half repeats the lower): its inputs
        const int32_t cell = P.next + (lane & (CELLS - 1));
        const bool valid = cell < ncell && lane < CELLS;
        P.next += gridDim.x * W * CELLS;
        double* mine = sm.mom[P.wave] + (lane & (CELLS - 1)) * MROW;
        const double N = mine[M_N], th = mine[M_TH];
        const bool feat = N > 1.0 && th > 0.0;
        bool finite = true;
        if constexpr (MODE == 2) {
#pragma unroll
            for (int i = 0; i < 31; ++i) finite = finite && isfinite(mine[i]);
        }
        double tau = 1.0;
        float f[NF];
#pragma unroll
        for (int q = 0; q < NF; ++q) f[q] = 0.0f;
        if (feat) cell_inputs(g, mine, nvol && cell < ncell ? nvol[cell] : g.fnum_over_vol, f, tau);
        // to LDS and back in the layout of the first product, in place of the records read
        lds_barrier();
        __bf16* xin = (__bf16*)sm.mom[P.wave];
        bf16x8 x[2];
#pragma unroll
        for (int k = 0; k < NF; ++k) x[k >> 3][k & 7] = (__bf16)((f[k] - sm.sec[SEC_XM + k]) / sm.sec[SEC_XS + k]);
        if (lane < CELLS) {
            *(bf16x8*)(xin + lane * 24) = x[0];
            *(bf16x8*)(xin + lane * 24 + 8) = x[1];
        }
        bf16x8 act0[KS], act1[KS];
        lds_barrier();
        P.template move<0>();
        const bf16x8 b0 = *(const bf16x8*)(xin + c * 24 + 8 * h);
#pragma unroll
        for (int mt = 0; mt < NT; ++mt) {
            const f32x16 acc =
                mfma32(*(const bf16x8*)(sm.w[0] + (mt * 64 + lane) * 8), b0, P.bias_of(sm.sec + SEC_B1, mt));
#pragma unroll
            for (int i = 0; i < 8; ++i) relu_pair(acc, act0, mt, i);
        }
        f32x16 acc = f32x16{};
        hidden_tiles<W, 1, 0>(P, sm.sec + SEC_B2, act0, act1, acc);
        hidden_tiles<W, 9, 0>(P, sm.sec + SEC_B3, act1, act0, acc);
        hidden_tiles<W, 17, 0>(P, sm.sec + SEC_B4, act0, act1, acc);
        lds_barrier();
        P.template products<25>(act1, acc, [](int) {});
        // lane = cell again: rows 0..3 and 8 live in half 0 (j = 0..3, 4), rows 4..7 in half 1
        float o[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) o[q] = __shfl(acc[q < 8 ? q & 3 : 4], c + (q >= 4 && q < 8 ? 32 : 0), 64);
        if (valid) {
            float y[9];
            const double d6[6] = {1, 0, 0, 1, 0, 1};
            const double sth = feat ? sqrt(th) : 0.0;
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                y[q] = o[q] + sm.sec[SEC_B5 + q];
                if constexpr (MODE != 0) {
                    const double d = (double)y[q] * (double)sm.sec[SEC_YS + q] + (double)sm.sec[SEC_YM + q];
                    const double v = q < 6 ? tau * d - 5.0 * g.eps_hat * d6[q] : tau * sth * d;
                    y[q] = feat ? (float)v : 0.0f;
                }
            }
            if constexpr (MODE == 2) {
                double yd[9];
#pragma unroll
                for (int q = 0; q < 9; ++q) yd[q] = (double)y[q];
                yd[0] += 5.0 * g.eps_hat;
                yd[3] += 5.0 * g.eps_hat;
                yd[5] += 5.0 * g.eps_hat;
                int st = cell_class(N, th, finite);
                double out[16];
                if (st == FP_CELL_OK) {
                    if (N < (double)g.n_min) {
                        st = FP_CELL_FEW;
                    } else {
                        st = FP_CELL_NN;
#pragma unroll
                        for (int q = 0; q < 9; ++q) st = isfinite(yd[q]) ? st : FP_CELL_SINGULAR;
                    }
                }
                update_record(g, st, th, finite, tau, yd, rec + (int64_t)cell * REC, relax, out);
#pragma unroll
                for (int i = 0; i < 16; ++i) rec[(int64_t)cell * REC + i] = out[i];
                status[cell] = st;
            } else {
                float* dst = yout + (int64_t)cell * NO;
#pragma unroll
                for (int q = 0; q < NO; ++q) dst[q] = q < 9 ? y[q] : 0.0f;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// training: the weights are packed to bfloat16 fragments (forward and transposed); one kernel
// takes tiles of samples through the forward pass, the loss and the backward pass, and leaves
// every layer's activations and pre-activation gradients as bfloat16 fragments whose inner
// dimension is the sample; one kernel multiplies those into the weight gradients, split over
// the samples; one adds the splits (and applies Adam).
//
// fragments of 64 lanes x 8 values: F1..F5 the forward A operands (rows = output units),
// T5..T2 the backward ones (rows = input units, inner dimension = output units)
constexpr int FR_F1 = 0, FR_F2 = NT, FR_F5 = FR_F2 + 3 * NT * KS, FR_T5 = FR_F5 + KS, FR_T2 = FR_T5 + NT,
              FR_N = FR_T2 + 3 * NT * KS;
// fragments of one 16-sample group: H1..H4 and dZ1..dZ4 (NT each), H0, dY (units 16..31 are
// copies of 0..15, their products are not used)
constexpr int SF_H = 0, SF_Z = 4 * NT, SF_H0 = 8 * NT, SF_DY = 8 * NT + 1, SF_N = 8 * NT + 2;
// one split's weight gradient: tiles of 32 x 32 in accumulator order, W2 W3 W4 (NT x NT each),
// W1 (by unit tile), W5 (by input tile, its rows 16..31 unused)
constexpr int GT_W1 = 3 * NT * NT, GT_W5 = GT_W1 + NT, GT_N = GT_W5 + NT;
constexpr int BROW = 4 * NH + NO;         // bias gradients of one workgroup: b1 .. b5
constexpr int TRAIN_MAX_WG = 256;         // one workgroup per CU
// splits of the weight gradients: 16 sample groups (256 samples) each while that gives at
// most 32
constexpr int SPLIT_GROUPS = 16, MAX_SPLITS = 32;

__host__ __device__ constexpr int64_t off_w(int layer) {   // layer 1..5
    return layer == 1 ? OFF_W1 : (layer == 5 ? OFF_W5 : OFF_W2 + (layer - 2) * (OFF_W3 - OFF_W2));
}

__global__ __launch_bounds__(64) void lite_train_pack_kernel(const float* __restrict__ p, __bf16* __restrict__ img) {
    const int f = blockIdx.x, lane = threadIdx.x, c = lane & 31, h = lane >> 5;
    bf16x8 v;
    if (f < FR_T5) {
        const bool first = f < FR_F2, last = f >= FR_F5;
        const int e = first ? f : (last ? f - FR_F5 : (f - FR_F2) % (NT * KS)), ks = first ? 1 : KS;
        const int layer = first ? 1 : (last ? 5 : 2 + (f - FR_F2) / (NT * KS));
        const int K = first ? NF : NH, m = (e / ks) * 32 + c, k0 = (e % ks) * 16 + 8 * h;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (__bf16)(last && m >= NO ? 0.0f : p[off_w(layer) + m * K + k0 + i]);
    } else {
        const bool last = f < FR_T2;
        const int e = last ? f - FR_T5 : (f - FR_T2) % (NT * KS), ks = last ? 1 : KS;
        const int layer = last ? 5 : 2 + (f - FR_T2) / (NT * KS);
        const int k = (e / ks) * 32 + c, m0 = (e % ks) * 16 + 8 * h;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (__bf16)p[off_w(layer) + (m0 + i) * NH + k];
    }
    *(bf16x8*)(img + (f * 64 + lane) * 8) = v;
}

template <int CT>
struct TrainShared {
    static constexpr int NS = 32 * CT;   // samples of a tile
    // row strides (bfloat16): 16-byte rows that start on different banks
    static constexpr int SH = NH + 8, SI = NF + 8, ST = NS + 8, SP = 40;
    __attribute__((aligned(16))) __bf16 hn[2][NS * SH];     // sample-major: H1..H4, then dZ4..dZ2
    __attribute__((aligned(16))) __bf16 tr[NT][32 * SP];    // a wave's tile, unit-major, on its way out
    __attribute__((aligned(16))) __bf16 h0n[NS * SI];
    __attribute__((aligned(16))) __bf16 h0t[NF * ST];
    __attribute__((aligned(16))) __bf16 dyn[NS * SI];
    __attribute__((aligned(16))) __bf16 dyt[NO * ST];       // rows 9..15 zero
    __attribute__((aligned(16))) float bias[BROW];
    float yf[NS * 17];                                      // Y, then dY in columns 0..8
    float xm[NF], xs[NF], ym[NO], ys[NO];
    double ll[512];
};

// Forward, loss (mean over samples of sum_o<9 (y_o - t_o)^2 on standardised targets) and
// backward of B samples, tile by tile; wave rt computes units 32 rt .. of every layer for the
// tile's 32 CT samples.  sf: fragments of every 16-sample group, [fragment][group][512].
// The weights (800 KB of fragments, two directions) stream from L2 once per tile.  Bound by the
// chain of twelve dependent phases of 1.2 to 2 us (products, activations, LDS both ways):
// 20 us for one tile per workgroup.  An Adam step at batch 4096 takes 35.9 us (this kernel
// 20, the weight gradients 7, the reduction 5, the packing 3); a kernel per layer with
// activations in memory, per-lane weight conversions and one thread per bias took 2113 us.
template <int CT>
__global__ __launch_bounds__(512) void lite_train_kernel(int64_t B, const float* __restrict__ p,
                                                         const __bf16* __restrict__ img,
                                                         const float* __restrict__ feats,
                                                         const float* __restrict__ T, int64_t groups,
                                                         __bf16* __restrict__ sf, float* __restrict__ bpart,
                                                         double* __restrict__ lpart) {
    using S = TrainShared<CT>;
    constexpr int NS = S::NS, BLOCK = 512, ITEMS = (NS * 9 + BLOCK - 1) / BLOCK;
    __shared__ S sm;
    int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
    const int rt = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: fragment bases in SGPRs
    const double invB = 1.0 / (double)B;
    for (int t = tid; t < NO * S::ST; t += BLOCK) sm.dyt[t] = (__bf16)0.0f;
    for (int t = tid; t < NS * S::SI; t += BLOCK) sm.dyn[t] = (__bf16)0.0f;
    for (int t = tid; t < 4 * NH; t += BLOCK)
        sm.bias[t] = p[OFF_B1 + (t / NH) * (OFF_B2 - OFF_B1) + t % NH];   // b1 .. b4, equally spaced
    if (tid < 16) {
        sm.bias[4 * NH + tid] = p[OFF_B5 + tid];
        sm.xm[tid] = p[OFF_XM + tid];
        sm.xs[tid] = p[OFF_XS + tid];
        sm.ym[tid] = p[OFF_YM + tid];
        sm.ys[tid] = p[OFF_YS + tid];
    }
    // the inputs of a tile: thread -> sample tid / 16 (and 32 further), feature tid % 16
    // (samples from B on read the last one's; their output gradients are zero)
    float fx[CT];
    auto load_inputs = [&](int64_t n0) {
#pragma unroll
        for (int u = 0; u < CT; ++u) fx[u] = feats[min(n0 + (tid >> 4) + 32 * u, B - 1) * NF + (tid & 15)];
    };
    float bs[4] = {0.0f, 0.0f, 0.0f, 0.0f}, b5 = 0.0f;   // bias gradients, units as row_sums() leaves them
    double loss = 0.0;
    load_inputs((int64_t)blockIdx.x * NS);
    lds_barrier();

    const int64_t tiles = (B + NS - 1) / NS;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t n0 = tile * NS, g0 = tile * 2 * CT;
        // nothing that a tile reads or addresses is kept in registers over the loop
        __asm__ volatile("" ::: "memory");
        __asm__ volatile("" : "+v"(tid), "+v"(lane), "+v"(h), "+v"(c));
        // the wave's tile of fragment f, samples 32 ct ..: v to LDS (for the next layer) and out
        auto put_out = [&](auto inner, const float (&v)[16], __bf16* hs, int ct, int f) {
            put_tile<decltype(inner)::value>(hs, S::SH, sm.tr[rt] - rt * 32 * S::SP - ct * 32, S::SP, ct * 32 + c, rt * 32, h,
                                             v);
            lds_wave_barrier();   // other lanes' values come back
#pragma unroll
            for (int s = 0; s < 2; ++s)
                *(bf16x8*)(sf + (((int64_t)(f + rt) * groups + g0 + 2 * ct + s) * 64 + lane) * 8) =
                    *(const bf16x8*)(sm.tr[rt] + c * S::SP + 16 * s + 8 * h);
            lds_wave_barrier();   // before the next tile takes their place
        };
        // products of the wave's units with the tile's samples; M fragments from nf on (a later
        // layer's weights) are loaded into nw in between, one per k-step: issued together, 128
        // KB over the workgroup at 64 B per cycle, they hold the waves up for as long as the
        // products take (0.7 of a 2.0 us layer)
        auto products = [&](auto ks, const bf16x8* a, const __bf16* hin, int stride, f32x16 (&acc)[CT], auto more, int nf,
                            bf16x8* nw) {
            constexpr int K = decltype(ks)::value, M = decltype(more)::value;
#pragma unroll
            for (int t = 0; t < CT; ++t) acc[t] = f32x16{};
            bf16x8 b[2][CT];
            auto read = [&](int s) {
#pragma unroll
                for (int t = 0; t < CT; ++t) b[s & 1][t] = *(const bf16x8*)(hin + (t * 32 + c) * stride + 16 * s + 8 * h);
            };
            read(0);
#pragma unroll
            for (int s = 0; s < (K > M ? K : M); ++s) {
                if (s + 1 < K) read(s + 1);
                if (s < K)
#pragma unroll
                    for (int t = 0; t < CT; ++t) acc[t] = mfma32(a[s], b[s & 1][t], acc[t]);
                if (s < M) nw[s] = *(const bf16x8*)(img + ((nf + s) * 64 + lane) * 8);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        using K0 = std::integral_constant<int, 0>;
        using K1 = std::integral_constant<int, 1>;
        using KH = std::integral_constant<int, KS>;
        uint32_t mask[4][CT];   // bit j: z > 0 in row j
        auto activate = [&](const f32x16 (&acc)[CT], int l, __bf16* hs) {
#pragma unroll
            for (int t = 0; t < CT; ++t) {
                float a[16];
                uint32_t m = 0;
#pragma unroll
                for (int jq = 0; jq < 4; ++jq) {
                    const float4 b = *(const float4*)(sm.bias + l * NH + rt * 32 + 8 * jq + 4 * h);
                    const float bb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float z = acc[t][4 * jq + e] + bb[e];
                        a[4 * jq + e] = fmaxf(z, 0.0f);
                        m |= z > 0.0f ? 1u << (4 * jq + e) : 0u;
                    }
                }
                __asm__ volatile("" : "+v"(m));   // the bits, not the 16 values behind them
                mask[l][t] = m;
                put_out(std::true_type{}, a, hs, t, SF_H + l * NT);
            }
        };
        auto backward = [&](auto inner, const f32x16 (&acc)[CT], int l, __bf16* zs) {
#pragma unroll
            for (int t = 0; t < CT; ++t) {
                float dz[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) dz[j] = (mask[l][t] >> j) & 1u ? acc[t][j] : 0.0f;
                bs[l] += row_sums(dz, lane);
                put_out(inner, dz, zs, t, SF_Z + l * NT);
            }
        };
        bf16x8 w1[1], wa[KS], wb[KS];
        load_frags<1>(img, FR_F1 + rt, lane, w1);
        load_frags<KS>(img, FR_F2 + rt * KS, lane, wa);
#pragma unroll
        for (int u = 0; u < CT; ++u) {
            const int n = (tid >> 4) + 32 * u, k = tid & 15;
            const __bf16 q = (__bf16)((fx[u] - sm.xm[k]) / sm.xs[k]);
            sm.h0n[n * S::SI + k] = q;
            sm.h0t[k * S::ST + n] = q;
        }
        // item it of the loss: sample it / 9 of the tile, output it % 9
        float tv[ITEMS];
#pragma unroll
        for (int u = 0; u < ITEMS; ++u) {
            const int it = min(tid + u * BLOCK, NS * 9 - 1), i = it / 9;
            tv[u] = T[min(n0 + i, B - 1) * NO + (it - 9 * i)];
        }
        lds_barrier();
        f32x16 acc[CT];
        products(K1{}, w1, sm.h0n, S::SI, acc, KH{}, FR_F2 + (NT + rt) * KS, wb);
        activate(acc, 0, sm.hn[0]);
        if (rt < 2 * CT)
            *(bf16x8*)(sf + (((int64_t)SF_H0 * groups + g0 + rt) * 64 + lane) * 8) =
                *(const bf16x8*)(sm.h0t + (c & 15) * S::ST + 16 * rt + 8 * h);
        lds_barrier();
        products(KH{}, wa, sm.hn[0], S::SH, acc, KH{}, FR_F2 + (2 * NT + rt) * KS, wa);
        activate(acc, 1, sm.hn[1]);
        lds_barrier();
        products(KH{}, wb, sm.hn[1], S::SH, acc, K0{}, 0, wb);
        if (rt < CT) load_frags<KS>(img, FR_F5, lane, wb);
        activate(acc, 2, sm.hn[0]);
        lds_barrier();
        load_frags<1>(img, FR_T5 + rt, lane, w1);
        products(KH{}, wa, sm.hn[0], S::SH, acc, KH{}, FR_T2 + (2 * NT + rt) * KS, wa);
        activate(acc, 3, sm.hn[1]);
        lds_barrier();
        if (rt < CT) {
            f32x16 y = f32x16{};
#pragma unroll
            for (int s = 0; s < KS; ++s)
                y = mfma32(wb[s], *(const bf16x8*)(sm.hn[1] + (rt * 32 + c) * S::SH + 16 * s + 8 * h), y);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int o = 8 * (j >> 2) + 4 * h + (j & 3);
                sm.yf[(rt * 32 + c) * 17 + o] = y[j] + sm.bias[4 * NH + o];
            }
        }
        load_frags<KS>(img, FR_T2 + (NT + rt) * KS, lane, wb);
        lds_barrier();
#pragma unroll
        for (int u = 0; u < ITEMS; ++u) {
            const int it = tid + u * BLOCK, i = it / 9, o = it - 9 * i;
            if (it >= NS * 9) continue;
            float d = 0.0f;
            if (n0 + i < B) {
                const double t = ((double)tv[u] - sm.ym[o]) / sm.ys[o];
                const double e = (double)sm.yf[i * 17 + o] - t;
                loss += e * e;
                d = (float)(2.0 * e * invB);
            }
            sm.yf[i * 17 + o] = d;
            sm.dyn[i * S::SI + o] = (__bf16)d;
            sm.dyt[o * S::ST + i] = (__bf16)d;
        }
        lds_barrier();
        products(K1{}, w1, sm.dyn, S::SI, acc, K0{}, 0, w1);
        backward(std::true_type{}, acc, 3, sm.hn[0]);
        if (rt < 2 * CT)
            *(bf16x8*)(sf + (((int64_t)SF_DY * groups + g0 + rt) * 64 + lane) * 8) =
                *(const bf16x8*)(sm.dyt + (c & 15) * S::ST + 16 * rt + 8 * h);
        if (rt == 7) {
            // the output bias: lane = output + 16 x quarter of the tile's samples
#pragma unroll
            for (int i = 0; i < NS / 4; ++i) b5 += sm.yf[((lane >> 4) * (NS / 4) + i) * 17 + (lane & 15)];
        }
        load_inputs((tile + gridDim.x) * NS);
        lds_barrier();
        products(KH{}, wa, sm.hn[0], S::SH, acc, KH{}, FR_T2 + rt * KS, wa);
        backward(std::true_type{}, acc, 2, sm.hn[1]);
        lds_barrier();
        products(KH{}, wb, sm.hn[1], S::SH, acc, K0{}, 0, wb);
        backward(std::true_type{}, acc, 1, sm.hn[0]);
        lds_barrier();
        products(KH{}, wa, sm.hn[0], S::SH, acc, K0{}, 0, wa);
        backward(std::false_type{}, acc, 0, sm.hn[1]);
    }

    float* out = bpart + (int64_t)blockIdx.x * BROW;
    if (!(lane & 16)) {
        const int j = lane & 15;
#pragma unroll
        for (int l = 0; l < 4; ++l) out[l * NH + rt * 32 + 8 * (j >> 2) + 4 * h + (j & 3)] = bs[l];
    }
    b5 += __shfl_xor(b5, 16, 64);
    b5 += __shfl_xor(b5, 32, 64);
    if (rt == 7 && lane < NO) out[4 * NH + lane] = lane < 9 ? b5 : 0.0f;
    sm.ll[tid] = loss;
    lds_barrier();
    for (int s = BLOCK / 2; s > 0; s >>= 1) {
        if (tid < s) sm.ll[tid] += sm.ll[tid + s];
        lds_barrier();
    }
    if (tid == 0) lpart[blockIdx.x] = sm.ll[0];
}

// weight gradients dZ^T H of one split of the sample groups: a wave takes 2 x 2 tiles of a
// hidden layer (or four tiles of the first or the last), both operands straight from the
// fragments (1 KB a load), four waves of a workgroup the four 64 x 64 quarters of 128 x 128
constexpr int JOBS = 3 * 16 + 4, WG_BLOCK = 256;
__global__ __launch_bounds__(WG_BLOCK) __attribute__((amdgpu_waves_per_eu(2, 2))) void lite_wgrad_kernel(int64_t groups, int splits, const __bf16* __restrict__ sf,
                                                              float* __restrict__ part) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // the workgroups of one split share its fragments: on one XCD
    const int lb = xcd_block(blockIdx.x, JOBS / 4 * splits), split = lb / (JOBS / 4);
    const int job = (lb % (JOBS / 4)) * 4 + wave;
    const int64_t g0 = groups * split / splits, g1 = groups * (split + 1) / splits;
    float* out = part + (int64_t)split * GT_N * 1024;
    auto run = [&](auto na, auto nb, int fa, int fb, int t0, int dt) {
        constexpr int NA = decltype(na)::value, NB = decltype(nb)::value;
        f32x16 acc[NA][NB];
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int k = 0; k < NB; ++k) acc[i][k] = f32x16{};
        const __bf16* a0 = sf + ((int64_t)fa * groups * 64 + lane) * 8;
        const __bf16* b0 = sf + ((int64_t)fb * groups * 64 + lane) * 8;
        // rounds of U groups, the next round's fragments in flight during this one's products
        // (left to itself the compiler waits for each load in turn: 14 against 8.5 us at 4096)
        constexpr int U = 4;
        struct Round {
            bf16x8 a[U][NA], b[U][NB];
        } r0, r1;
        auto load = [&](Round& r, int64_t g) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t at = min(g + u, g1 - 1);
#pragma unroll
                for (int i = 0; i < NA; ++i) r.a[u][i] = *(const bf16x8*)(a0 + (i * groups + at) * 512);
#pragma unroll
                for (int k = 0; k < NB; ++k) r.b[u][k] = *(const bf16x8*)(b0 + (k * groups + at) * 512);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto products = [&](const Round& r, int64_t g) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (g + u < g1)
#pragma unroll
                    for (int i = 0; i < NA; ++i)
#pragma unroll
                        for (int k = 0; k < NB; ++k) acc[i][k] = mfma32(r.a[u][i], r.b[u][k], acc[i][k]);
        };
        load(r0, g0);
        for (int64_t g = g0; g < g1; g += 2 * U) {
            if (g + U < g1) load(r1, g + U);
            products(r0, g);
            if (g + 2 * U < g1) load(r0, g + 2 * U);
            products(r1, g + U);
        }
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int k = 0; k < NB; ++k)
#pragma unroll
                for (int jq = 0; jq < 4; ++jq)
                    *(float4*)(out + (int64_t)(t0 + i * dt + k) * 1024 + jq * 256 + lane * 4) =
                        make_float4(acc[i][k][4 * jq], acc[i][k][4 * jq + 1], acc[i][k][4 * jq + 2], acc[i][k][4 * jq + 3]);
    };
    using N1 = std::integral_constant<int, 1>;
    using N2 = std::integral_constant<int, 2>;
    using N4 = std::integral_constant<int, 4>;
    if (job < 48) {
        // layer l + 2 (W2 W3 W4): dZ of layer l + 2, H of layer l + 1
        const int l = job / 16, q = (job % 16) / 4, w = job % 4;
        const int mt = 4 * (q >> 1) + 2 * (w >> 1), kt = 4 * (q & 1) + 2 * (w & 1);
        run(N2{}, N2{}, SF_Z + (l + 1) * NT + mt, SF_H + l * NT + kt, l * NT * NT + mt * NT + kt, NT);
    } else if (job < 50) {
        const int mt = 4 * (job - 48);
        run(N4{}, N1{}, SF_Z + mt, SF_H0, GT_W1 + mt, 1);
    } else {
        const int kt = 4 * (job - 50);
        run(N1{}, N4{}, SF_DY, SF_H + 3 * NT + kt, GT_W5 + kt, 0);
    }
}

// grad = the splits' (weights) and the workgroups' (biases) partial sums added in order: ranges
// of rows by the four waves, then the ranges, a float4 of four values per lane; with ADAM the
// parameters are updated as well.  The last workgroup adds the loss.
constexpr int RED_R = 4, RED_BLOCK = 64 * RED_R, RED_W = GT_N * 4, RED_B = (BROW / 4 + 63) / 64;
template <bool ADAM>
__global__ __launch_bounds__(RED_BLOCK) void lite_reduce_kernel(int splits, const float* __restrict__ part, int rows,
                                                                const float* __restrict__ bpart,
                                                                const double* __restrict__ lpart, int64_t B,
                                                                float* __restrict__ grad, float* __restrict__ loss,
                                                                AdamArgs ad) {
    const int lane = threadIdx.x & 63, r = threadIdx.x >> 6;
    if (blockIdx.x == RED_W + RED_B) {
        if (threadIdx.x >= 64) return;
        double s = 0.0;
        for (int i = lane; i < rows; i += 64) s += lpart[i];
        s = group_sum<64>(s);
        if (lane == 0) *loss = (float)(s / (double)B);
        return;
    }
    __shared__ float4 red[RED_R][64];
    // parameter of the lane's first value, the stride to the next ones, and whether they exist
    const float* src;
    int64_t q, row_len;
    int st = 1, n;
    bool live = true;
    if (blockIdx.x < RED_W) {
        const int t = blockIdx.x >> 2, row = 8 * (blockIdx.x & 3) + 4 * (lane >> 5), col = lane & 31;
        src = part + ((int64_t)blockIdx.x * 64 + lane) * 4;
        row_len = GT_N * 1024;
        n = splits;
        st = NH;
        if (t < GT_W1)
            q = OFF_W2 + (t / (NT * NT)) * (OFF_W3 - OFF_W2) + ((t / NT % NT) * 32 + row) * NH + (t % NT) * 32 + col;
        else if (t < GT_W5) {
            st = NF;
            q = OFF_W1 + ((t - GT_W1) * 32 + row) * NF + col;
            live = col < NF;
        } else {
            q = OFF_W5 + row * NH + (t - GT_W5) * 32 + col;
            live = row < NO;
        }
    } else {
        const int i = ((blockIdx.x - RED_W) * 64 + lane) * 4;
        src = bpart + i;
        row_len = BROW;
        n = rows;
        live = i < BROW;
        const int l = min(i / NH, 4);
        q = (l == 0 ? OFF_B1 : l == 1 ? OFF_B2 : l == 2 ? OFF_B3 : l == 3 ? OFF_B4 : OFF_B5) + i - l * NH;
    }
    float pq[4], mq[4], vq[4];
    if (ADAM && r == 0 && live) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pq[e] = ad.p[q + e * st];
            mq[e] = ad.m[q + e * st];
            vq[e] = ad.v[q + e * st];
        }
    }
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (live) {
        const int r1 = (r + 1) * n / RED_R;
#pragma unroll 8
        for (int i = r * n / RED_R; i < r1; ++i) {
            const float4 v = *(const float4*)(src + i * row_len);
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
    }
    red[r][lane] = s;
    __syncthreads();
    if (r != 0 || !live) return;
#pragma unroll
    for (int i = 1; i < RED_R; ++i) {
        const float4 v = red[i][lane];
        s.x += v.x;
        s.y += v.y;
        s.z += v.z;
        s.w += v.w;
    }
    const float g[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        grad[q + e * st] = g[e];
        if (ADAM) adam_one(ad, q + e * st, g[e], mq[e], vq[e], pq[e]);
    }
}

__global__ void lite_adam_kernel(AdamArgs a, const float* __restrict__ g) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < N_TRAIN) adam_one(a, q, g[q], a.m[q], a.v[q], a.p[q]);
}

// raw inputs of a batch of moment records (nvol per record, or the configuration's)
__global__ void lite_features_kernel(fp_config g, int64_t n, const double* __restrict__ mom,
                                     const double* __restrict__ nvol, float* __restrict__ feats) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    double m[M_R];
#pragma unroll
    for (int i = 0; i < M_R; ++i) m[i] = mom[c * MOM + i];
    float f[NF];
    double tau;
    cell_inputs(g, m, nvol ? nvol[c] : g.fnum_over_vol, f, tau);
#pragma unroll
    for (int q = 0; q < NF; ++q) feats[c * NF + q] = f[q];
}

// targets (Ct (6), Gamma (3), zeros) of a batch of update records
__global__ void lite_targets_kernel(int64_t n, const double* __restrict__ rec, float* __restrict__ tg) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
#pragma unroll
    for (int q = 0; q < NO; ++q) tg[c * NO + q] = q < 9 ? (float)rec[c * REC + q] : 0.0f;
}

}  // namespace lite

int launch_closure_nn(fp_ctx* c, const float* ynn, const float* ysec, double tol_abs, double tol_rel,
                      double relax, const double* mom, double* rec, int32_t* status, hipStream_t s);

}  // namespace fpg

// =========================================================================================
using namespace fpg;
using namespace fpg::lite;

struct fp_lite {
    fp_ctx* ctx = nullptr;
    int64_t max_batch = 0;
    __bf16* img = nullptr;
    float* sec = nullptr;
    float* ybuf = nullptr;   // [ncell][16] normalised coefficients of the last closure
    // training scratch: weight fragments, sample fragments, partial gradients and losses
    __bf16 *timg = nullptr, *sf = nullptr;
    float *part = nullptr, *bpart = nullptr, *grad = nullptr;
    double* lpart = nullptr;
};

template <typename T>
static bool lalloc(T** p, size_t count) {
    return hipMalloc((void**)p, sizeof(T) * (count ? count : 1)) == hipSuccess;
}

extern "C" void fp_lite_destroy(fp_lite* n) {
    if (!n) return;
    (void)hipDeviceSynchronize();
    for (void* q : {(void*)n->img, (void*)n->sec, (void*)n->ybuf, (void*)n->timg, (void*)n->sf, (void*)n->part,
                    (void*)n->bpart, (void*)n->grad, (void*)n->lpart})
        (void)hipFree(q);
    delete n;
}

// 16-sample groups of a batch (whole 64-sample tiles) and the splits of its weight gradients
static int64_t groups_of(int64_t B) { return (B + 63) / 64 * 4; }
static int splits_of(int64_t B) {
    return (int)std::min<int64_t>(MAX_SPLITS, (groups_of(B) + SPLIT_GROUPS - 1) / SPLIT_GROUPS);
}

extern "C" int fp_lite_create(fp_ctx* c, int64_t max_batch, fp_lite** out) {
    if (!c || !out || max_batch < 0 || max_batch > ((int64_t)1 << 24)) return FP_EINVAL;
    *out = nullptr;
    fp_lite* n = new (std::nothrow) fp_lite();
    if (!n) return FP_ENOMEM;
    n->ctx = c;
    n->max_batch = max_batch;
    bool ok = lalloc(&n->img, IMG_BF) && lalloc(&n->sec, SEC_N) && lalloc(&n->ybuf, (size_t)c->ncell * NO);
    if (ok && max_batch > 0) {
        // enough for every batch up to max_batch
        const size_t rows = (size_t)std::min<int64_t>(TRAIN_MAX_WG, (max_batch + 31) / 32);
        ok = lalloc(&n->timg, FR_N * 512) && lalloc(&n->sf, (size_t)SF_N * groups_of(max_batch) * 512) &&
             lalloc(&n->part, (size_t)splits_of(max_batch) * GT_N * 1024) && lalloc(&n->bpart, rows * BROW) &&
             lalloc(&n->grad, N_PARAMS) && lalloc(&n->lpart, rows);
    }
    if (!ok) {
        fp_lite_destroy(n);
        return FP_ENOMEM;
    }
    *out = n;
    return FP_OK;
}

extern "C" int fp_lite_load(fp_ctx* c, fp_lite* n, const float* params, hipStream_t s) {
    if (!c || !n || !params || n->ctx != c) return set_err(c, FP_EINVAL, "fp_lite_load: bad argument");
    hipLaunchKernelGGL(lite_pack_kernel, dim3((IMG_BF + 255) / 256), dim3(256), 0, s, params, n->img, n->sec);
    return check_launch(c, "fp_lite_load");
}

// a workgroup per CU: four waves while their workgroups reach all cells in one pass, else eight
// (two per SIMD, which hide each other's latencies), also where those leave CUs idle: mode 2 on
// 4096 / 32,768 / 32,769 / 65,536 / 131,072 cells takes 21.7 / 26.1 / 41.5 / 47.2 / 90.8 us with four and
// 28.3 / 31.4 / 31.2 / 38.3 / 70.5 us with eight
template <int MODE>
static void infer(fp_ctx* c, const fp_lite* n, const double* mom, float* y, double* rec, int32_t* status, double relax,
                  hipStream_t s) {
    const bool wide = c->ncell > 128 * 256;   // 256 workgroups of four waves, 32 cells a wave
    const int w = wide ? 8 : 4;
    const int grid = std::min(256, (c->ncell + 32 * w - 1) / (32 * w));
    hipLaunchKernelGGL((wide ? lite_infer_kernel<8, MODE> : lite_infer_kernel<4, MODE>), dim3(grid), dim3(64 * w), 0, s,
                       c->cfg, c->ncell, mom, (const double*)c->nvol, (const __bf16*)n->img, (const float*)n->sec, y, rec,
                       status, relax);
}

extern "C" int fp_lite_infer(fp_ctx* c, const fp_lite* n, const double* mom, float* y, hipStream_t s) {
    if (!c || !n || !mom || !y || n->ctx != c) return set_err(c, FP_EINVAL, "fp_lite_infer: bad argument");
    if (c->ncell == 0) return FP_OK;
    infer<0>(c, n, mom, y, nullptr, nullptr, 1.0, s);
    return check_launch(c, "fp_lite_infer");
}

extern "C" int fp_closure_lite(fp_ctx* c, const fp_lite* n, const double* mom, double* rec,
                               int32_t* status, double tol_abs, double tol_rel, double relax,
                               hipStream_t s) {
    if (!c || !n || !mom || !rec || !status || n->ctx != c || !(tol_abs >= 0) || !(tol_rel >= 0) ||
        !(relax > 0.0 && relax <= 1.0))
        return set_err(c, FP_EINVAL, "fp_closure_lite: bad argument");
    if (c->cfg.moment_order == 3 && tol_abs != INFINITY)
        return set_err(c, FP_EINVAL, "fp_closure_lite: the check needs moments through fifth order");
    if (c->ncell == 0) return FP_OK;
    // third-order records have no system to check or to fall back on: one kernel
    if (c->cfg.moment_order == 3) {
        infer<2>(c, n, mom, nullptr, rec, status, relax, s);
        return check_launch(c, "fp_closure_lite");
    }
    infer<1>(c, n, mom, n->ybuf, nullptr, nullptr, 1.0, s);
    const int rc = check_launch(c, "fp_closure_lite (network)");
    if (rc) return rc;
    return launch_closure_nn(c, n->ybuf, n->sec + SEC_ID, tol_abs, tol_rel, relax, mom, rec, status, s);
}

extern "C" int fp_lite_features(fp_ctx* c, const double* mom, const double* nvol, int64_t n, float* feats,
                                hipStream_t s) {
    if (!c || !mom || !feats || n < 0) return set_err(c, FP_EINVAL, "fp_lite_features: bad argument");
    if (n == 0) return FP_OK;
    hipLaunchKernelGGL(lite_features_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, c->cfg, n,
                       mom, nvol, feats);
    return check_launch(c, "fp_lite_features");
}

extern "C" int fp_lite_targets(fp_ctx* c, const double* rec, int64_t n, float* targets, hipStream_t s) {
    if (!c || !rec || !targets || n < 0) return set_err(c, FP_EINVAL, "fp_lite_targets: bad argument");
    if (n == 0) return FP_OK;
    hipLaunchKernelGGL(lite_targets_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, rec,
                       targets);
    return check_launch(c, "fp_lite_targets");
}

// gradient (and, with ad, the Adam step on it); the arguments are checked
static int train_launch(fp_ctx* c, fp_lite* n, const float* params, const float* feats, const float* targets,
                        int64_t B, float* grad, float* loss, const AdamArgs* ad, const char* what, hipStream_t s) {
    hipLaunchKernelGGL(lite_train_pack_kernel, dim3(FR_N), dim3(64), 0, s, params, n->timg);
    // tiles of 32 samples while they fit on the CUs at once, else of 64 (each weight read
    // serves twice the samples), a workgroup per CU: 47 us at 8192 samples, 53 us at 8193
    const bool small = B <= 32 * TRAIN_MAX_WG;
    const int rows = small ? (int)((B + 31) / 32) : (int)std::min<int64_t>(TRAIN_MAX_WG, (B + 63) / 64);
    const int64_t groups = small ? (int64_t)rows * 2 : groups_of(B);
    const int splits = splits_of(B);
    hipLaunchKernelGGL(small ? lite_train_kernel<1> : lite_train_kernel<2>, dim3(rows), dim3(512), 0, s, B, params,
                       (const __bf16*)n->timg, feats, targets, groups, n->sf, n->bpart, n->lpart);
    hipLaunchKernelGGL(lite_wgrad_kernel, dim3(JOBS / 4 * splits), dim3(WG_BLOCK), 0, s, groups, splits,
                       (const __bf16*)n->sf, n->part);
    const dim3 rgrid(RED_W + RED_B + 1);
    if (ad)
        hipLaunchKernelGGL(lite_reduce_kernel<true>, rgrid, dim3(RED_BLOCK), 0, s, splits, (const float*)n->part, rows,
                           (const float*)n->bpart, (const double*)n->lpart, B, grad, loss, *ad);
    else
        hipLaunchKernelGGL(lite_reduce_kernel<false>, rgrid, dim3(RED_BLOCK), 0, s, splits, (const float*)n->part, rows,
                           (const float*)n->bpart, (const double*)n->lpart, B, grad, loss, AdamArgs{});
    return check_launch(c, what);
}

static bool grad_args(const fp_ctx* c, const fp_lite* n, const float* params, const float* feats, const float* targets,
                      int64_t B, const float* grad, const float* loss) {
    return c && n && params && feats && targets && grad && loss && B > 0 && B <= n->max_batch && n->ctx == c;
}

extern "C" int fp_lite_grad(fp_ctx* c, fp_lite* n, const float* params, const float* feats,
                            const float* targets, int64_t B, float* grad, float* loss, hipStream_t s) {
    if (!grad_args(c, n, params, feats, targets, B, grad, loss))
        return set_err(c, FP_EINVAL, "fp_lite_grad: bad argument");
    return train_launch(c, n, params, feats, targets, B, grad, loss, nullptr, "fp_lite_grad", s);
}

extern "C" int fp_lite_adam(fp_ctx* c, float* params, const float* grad, float* m, float* v, int64_t t,
                            float lr, hipStream_t s) {
    if (!c || !params || !grad || !m || !v || t < 1 || !(lr >= 0.0f))
        return set_err(c, FP_EINVAL, "fp_lite_adam: bad argument");
    hipLaunchKernelGGL(lite_adam_kernel, dim3((unsigned)((N_TRAIN + 255) / 256)), dim3(256), 0, s,
                       adam_args(params, m, v, t, lr), grad);
    return check_launch(c, "fp_lite_adam");
}

extern "C" int fp_lite_train_step(fp_ctx* c, fp_lite* n, float* params, float* m, float* v, int64_t t,
                                  float lr, const float* feats, const float* targets, int64_t B, float* loss,
                                  hipStream_t s) {
    if (!n) return set_err(c, FP_EINVAL, "fp_lite_train_step: bad argument");
    if (!grad_args(c, n, params, feats, targets, B, n->grad, loss))
        return set_err(c, FP_EINVAL, "fp_lite_grad: bad argument");
    if (!m || !v || t < 1 || !(lr >= 0.0f)) {
        // as the two calls would: the gradient and the loss, then the refusal
        const int rc = train_launch(c, n, params, feats, targets, B, n->grad, loss, nullptr, "fp_lite_grad", s);
        return rc ? rc : set_err(c, FP_EINVAL, "fp_lite_adam: bad argument");
    }
    const AdamArgs ad = adam_args(params, m, v, t, lr);
    return train_launch(c, n, params, feats, targets, B, n->grad, loss, &ad, "fp_lite_train_step", s);
}

// ---- column statistics of a training matrix (the standardising scaler of Sec. "Phase 3":
// per-column mean and population standard deviation) ------------------------------------
namespace fpg {
namespace lite {
constexpr int STAT_BLOCK = 256;
// one workgroup per column: FP64 sums in a fixed order (strided per thread, then a tree in
// LDS), two passes (mean, then squared deviations): bitwise reproducible
__global__ __launch_bounds__(STAT_BLOCK) void column_stats_kernel(const float* __restrict__ x, int64_t n,
                                                                 int32_t k, double* __restrict__ mean,
                                                                 double* __restrict__ stdev) {
    __shared__ double sh[STAT_BLOCK];
    const int col = blockIdx.x;
    double s = 0.0;
    for (int64_t r = threadIdx.x; r < n; r += STAT_BLOCK) s += (double)x[r * k + col];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = STAT_BLOCK / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    const double mu = sh[0] / (double)n;
    __syncthreads();
    double q = 0.0;
    for (int64_t r = threadIdx.x; r < n; r += STAT_BLOCK) {
        const double d = (double)x[r * k + col] - mu;
        q += d * d;
    }
    sh[threadIdx.x] = q;
    __syncthreads();
    for (int w = STAT_BLOCK / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        mean[col] = mu;
        stdev[col] = sqrt(sh[0] / (double)n);
    }
}
}  // namespace lite
}  // namespace fpg

extern "C" int fp_column_stats(fp_ctx* c, const float* x, int64_t n, int32_t k, double* mean, double* stdev,
                               hipStream_t s) {
    if (!c || !x || !mean || !stdev || n < 1 || k < 1 || k > 4096)
        return set_err(c, FP_EINVAL, "fp_column_stats: bad argument");
    hipLaunchKernelGGL(fpg::lite::column_stats_kernel, dim3(k), dim3(fpg::lite::STAT_BLOCK), 0, s, x, n, k,
                       mean, stdev);
    return check_launch(c, "fp_column_stats");
}
