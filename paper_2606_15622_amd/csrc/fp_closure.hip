// fp_closure.hip -- batched exact closure: one lane per cell, FP64 in registers.
//
// Builds the theta-normalised 9x9 system of every cell (fp_closure_dev.h) and solves it
// by LU with partial pivoting, fully unrolled: the pivot row swap is a predicated select
// on every candidate row, so the 90 doubles of the augmented matrix stay in VGPRs.
#include "fp_closure_dev.h"

namespace fpg {

constexpr int CL_BLOCK = 64;

// NN = false: exact solve.  NN = true: the network's standardised outputs ynn[cell][16]
// are de-standardised (ysec = y_mean[16], y_std[16]) into normalised coefficients and
// accepted if the residual of the normalised system satisfies
// |A y - b| <= tol_abs + tol_rel |b|; otherwise the cell is solved exactly.  With
// tol_abs = +inf every finite output is accepted; a non-finite one is solved exactly, or,
// when the records hold moments through third order only (low), takes the Langevin drift
// (status SINGULAR).  relax < 1 blends the accepted coefficients with the cell's previous
// ones: C = relax C_net + (1 - relax) C_prev (the same for Gamma), where the previous
// record carries coefficients.
//
// One wave per workgroup, 64 cells, two waves per SIMD (the registers of the system).  A lane
// that read its own record, 16 bytes at a time, had every load touch 64 lines; the records
// come instead as 16-byte chunks straight into LDS, 1 KB (four cells) an instruction, and the
// results leave the same way.  Chunk c of row r lies in slot c ^ (r & 15) (of a result:
// c ^ (r / 2 & 7)), so the lanes of a row-per-lane access start on different banks.
// 1e6 cells (388 MB in and out): 99 -> 86 us, of which skipping rows that no lane pivots on
// (lu_solve) is 6; the traffic alone takes 75.  Bound by the FP64 and select instructions
// (about 60 us) that two waves cannot wholly hide behind memory.  Persistent waves that fetch
// the next 64 records during a solve: 116 us (the loop's hoisted constants spill).
constexpr int CL_PIECES = CL_BLOCK * MOM * 8 / 1024;

__device__ __forceinline__ void wait_loads() {
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    __asm__ volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lds() {
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __asm__ volatile("" ::: "memory");
}

// DIRECT: the records are 16-byte aligned; others pass through registers on their way to LDS
template <bool NN, bool DIRECT>
__global__ __launch_bounds__(CL_BLOCK, 2) void closure_kernel(fp_config g, int32_t ncell,
                                                               const double* __restrict__ mom,
                                                               double* __restrict__ rec,
                                                               int32_t* __restrict__ status,
                                                               const float* __restrict__ ynn,
                                                               const float* __restrict__ ysec,
                                                               double tol_abs, double tol_rel,
                                                               const double* __restrict__ nvol,
                                                               double relax) {
    __shared__ double2 rows[CL_BLOCK * MOM / 2];
    const int lane = threadIdx.x;
    const int64_t first = (int64_t)blockIdx.x * CL_BLOCK;
    const int64_t cell = min(first + lane, (int64_t)ncell - 1);
    {
        const double* base = mom + first * MOM;
        const int last = (int)min((int64_t)CL_BLOCK, ncell - first) - 1;   // repeated behind the end
#pragma unroll
        for (int q = 0; q < CL_PIECES; ++q) {
            const int r = 4 * q + (lane >> 4), chunk = (lane & 15) ^ (r & 15);
            const double* src = base + min(r, last) * MOM + chunk * 2;
            if (DIRECT)
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void*)src,
                    (__attribute__((address_space(3))) void*)(rows + q * 64), 16, 0, 0);
            else
                rows[q * 64 + lane] = make_double2(src[0], src[1]);
        }
    }
    const double nv = nvol ? nvol[cell] : g.fnum_over_vol;
    float yo[9] = {};
    if (NN)
#pragma unroll
        for (int i = 0; i < 9; ++i) yo[i] = ynn[cell * 16 + i];
    wait_loads();
    wait_lds();
    double m[MOM];
#pragma unroll
    for (int q = 0; q < MOM / 2; ++q) {
        const double2 v = rows[lane * (MOM / 2) + (q ^ (lane & 15))];
        m[2 * q] = v.x;
        m[2 * q + 1] = v.y;
    }
    bool finite = true;
#pragma unroll
    for (int i = 0; i < 31; ++i) finite = finite && isfinite(m[i]);
    const double N = m[M_N], theta = m[M_TH];
    int st = cell_class(N, theta, finite);
    double tau = 0.0, y[9];
    if (st == FP_CELL_OK) {
        tau = cell_tau(g, N * nv, theta);
        if (N < (double)g.n_min) {
            st = FP_CELL_FEW;
        } else {
            bool accepted = false;
            const bool unchecked = NN && tol_abs == INFINITY;   // accept any finite output
            if (NN) {
#pragma unroll
                for (int i = 0; i < 9; ++i) y[i] = (double)yo[i] * (double)ysec[16 + i] + (double)ysec[i];
                y[0] += 5.0 * g.eps_hat;
                y[3] += 5.0 * g.eps_hat;
                y[5] += 5.0 * g.eps_hat;
                if (unchecked) {
                    accepted = true;
#pragma unroll
                    for (int i = 0; i < 9; ++i) accepted = accepted && isfinite(y[i]);
                }
            }
            if (!accepted && NN && unchecked && g.moment_order == 3) {
                st = FP_CELL_SINGULAR;   // no system to fall back on: Langevin drift
            } else if (!accepted) {
                CellSystem s;
                build_system(m, g.eps_hat, s);
                if (NN && !unchecked) {
                    double rr = 0.0, bb = 0.0;
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        double t = -s.a[i][9];
#pragma unroll
                        for (int k = 0; k < 9; ++k) t = fma(s.a[i][k], y[k], t);
                        rr = fma(t, t, rr);
                        bb = fma(s.a[i][9], s.a[i][9], bb);
                    }
                    accepted = sqrt(rr) <= tol_abs + tol_rel * sqrt(bb);
#pragma unroll
                    for (int i = 0; i < 9; ++i) accepted = accepted && isfinite(y[i]);
                }
                if (!accepted) {
                    const bool ok = lu_solve(s, g.pivot_tol, y);
                    bool fin = true;
#pragma unroll
                    for (int i = 0; i < 9; ++i) fin = fin && isfinite(y[i]);
                    if (!ok || !fin) st = FP_CELL_SINGULAR;
                    else if (NN) st = FP_CELL_NN_FALLBACK;
                }
            }
            if (accepted) st = FP_CELL_NN;
        }
    }
    double out[16];
    update_record(g, st, theta, finite, tau, y, rec + cell * REC, relax, out);
    // the records leave through LDS the same way, eight cells an instruction
    wait_lds();
#pragma unroll
    for (int q = 0; q < REC / 2; ++q)
        rows[lane * (REC / 2) + (q ^ (lane >> 1 & 7))] = make_double2(out[2 * q], out[2 * q + 1]);
    wait_lds();
#pragma unroll
    for (int q = 0; q < REC / 2; ++q) {
        const int r = 8 * q + (lane >> 3), chunk = (lane & 7) ^ (r >> 1 & 7);
        const double2 v = rows[q * 64 + lane];
        if (first + r < ncell) {
            double* dst = rec + (first + r) * REC + chunk * 2;
            dst[0] = v.x;
            dst[1] = v.y;
        }
    }
    if (first + lane < ncell) status[cell] = st;
}

template <bool NN>
static void launch(fp_ctx* c, const double* mom, double* rec, int32_t* status, const float* ynn,
                   const float* ysec, double tol_abs, double tol_rel, double relax, hipStream_t s) {
    const auto kernel = (uintptr_t)mom & 15 ? closure_kernel<NN, false> : closure_kernel<NN, true>;
    const int grid = ((int64_t)c->ncell + CL_BLOCK - 1) / CL_BLOCK;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(CL_BLOCK), 0, s, c->cfg, c->ncell, mom, rec, status,
                       ynn, ysec, tol_abs, tol_rel, (const double*)c->nvol, relax);
}

int launch_closure(fp_ctx* c, const double* mom, double* rec, int32_t* status, hipStream_t s) {
    launch<false>(c, mom, rec, status, nullptr, nullptr, 0.0, 0.0, 1.0, s);
    return check_launch(c, "fp_closure_solve");
}

int launch_closure_nn(fp_ctx* c, const float* ynn, const float* ysec, double tol_abs,
                      double tol_rel, double relax, const double* mom, double* rec, int32_t* status,
                      hipStream_t s) {
    launch<true>(c, mom, rec, status, ynn, ysec, tol_abs, tol_rel, relax, s);
    return check_launch(c, "fp_closure_nn (check)");
}

}  // namespace fpg
