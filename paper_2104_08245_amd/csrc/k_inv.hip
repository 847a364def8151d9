// Inverse of T_J(S) by the coupled Newton-Schulz iteration (Sec. III-C.3,
// Eq. inv1-inv3) on the matrix cores, FP16 / BF16 operands with FP32
// accumulation, and the formation of A_J = T_J(S)^-1 T_J(K) - mu I and
// Y_J = T_J(S)^-1 E_cJ from it (Eq. purification_submatrix).
//
//   Y_0 = c S_J, Z_0 = I,  c = 1 / max row sum of |S_J| (spectrum of c S_J
//   inside (0, 1]); per iteration k:
//     R_k = I - Z_k Y_k                       (one GEMM; ||R_k||_F^2 partials)
//     Y_{k+1} = Y_k + Y_k R_k / 2,  Z_{k+1} = Z_k + R_k Z_k / 2
//   which equal Y_k (3I - V_k) / 2 and (3I - V_k) Z_k / 2 with V_k = Z_k Y_k;
//   R_k is small near convergence and keeps its relative precision in 16
//   bits. Z_k tends to (c S_J)^(-1/2), so S_J^-1 = c Z_K^2.
// The iteration stops like the 16-bit sign iteration (stagnation of
// ||R_k||_F below 0.5); a diverging one marks the molecule NOT_SPD. The
// outputs are exactly those of the Cholesky route: [A | Y] in the FP64 K
// buffer, |A| row / column sums and Frobenius partials per 64-column tile.
#include "dev_common.h"
#include "kernels.h"
#include "lp_gemm.h"

enum { IM_R = 1, IM_UPD = 2, IM_SQ = 3, IM_A = 4 };
enum { IACT_STOP = 0, IACT_UPDATE = 1 };

// c = 1 / max row sum of |S_J| over the padded np x np matrix (padding rows
// are identity), Y_0 = c S_J and Z_0 = I in 16 bits; one workgroup per slot.
// Bound by two reads of S_J and the writes of Y_0 and Z_0: sixteen waves a
// workgroup and 16-byte accesses keep enough of them in flight (600 slots of
// about 612 rows: 1105 us, 2250 with four waves and an element per access).
template <typename T>
__global__ __launch_bounds__(1024) void k_inv_init(ChunkDev cd, char *ws) {
    __shared__ double red[16];
    const int s = blockIdx.x;
    if (s >= cd.nsub) return;
    const SubMeta M = cd.meta[s];
    InvCtl *ic = cd.ictl + s;
    const int np = M.np, ldx = M.ldx, t = threadIdx.x, w = t >> 6, l = t & 63;
    const double *S = (const double *)(ws + M.offL);
    double mx = 0.0;
    for (int r = w; r < np; r += 16) {
        double rs = 0.0;
#pragma unroll 4
        for (int c = l; c < np; c += 64) rs += fabs(S[(int64_t)r * np + c]);
        mx = fmax(mx, wave_sum(rs));
    }
    if (l == 0) red[w] = mx;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) mx = fmax(mx, red[q]);
    const double c = 1.0 / mx;
    uint16_t *Y0 = (uint16_t *)(ws + M.offY0);
    uint16_t *Z0 = (uint16_t *)(ws + M.offZ0);
    const int n8 = np / 8;
    for (int f = t; f < np * n8; f += 1024) {
        const int r = f / n8, q = (f - r * n8) * 8;
        const double2 *src = (const double2 *)(S + (int64_t)r * np + q);
        uint32_t y[4], z[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double2 v = src[k];
            y[k] = Lp<T>::enc((float)(c * v.x)) | ((uint32_t)Lp<T>::enc((float)(c * v.y)) << 16);
            z[k] = Lp<T>::enc(r == q + 2 * k ? 1.0f : 0.0f) | ((uint32_t)Lp<T>::enc(r == q + 2 * k + 1 ? 1.0f : 0.0f) << 16);
        }
        *(uint4 *)(Y0 + (int64_t)r * ldx + q) = make_uint4(y[0], y[1], y[2], y[3]);
        *(uint4 *)(Z0 + (int64_t)r * ldx + q) = make_uint4(z[0], z[1], z[2], z[3]);
    }
    if (t == 0) {
        ic->done = 0;
        ic->iters = 0;
        ic->scale = c;
    }
    for (int i = t; i < NOLSM_MAX_ITER_CAP; i += 1024) ic->rhist[i] = 0.0;
}

// Decision at the update of iteration `it`, taken by wave 0 of every
// workgroup of the slot from the finished residual partials; the tile-0
// workgroup records it.
__device__ int inv_decide(const InvArgs &ia, const SubMeta &M, InvCtl *ic, SubCtl *ctl, const char *ws, int it,
                          int tile) {
    const double *res = (const double *)(ws + M.offRes) + (int64_t)it * M.ntile_ns;
    double ssum = 0.0;
    for (int i = threadIdx.x; i < M.ntile_ns; i += 64) ssum += res[i];
    const double r = sqrt(wave_sum(ssum));
    const double rprev = it > 0 ? ic->rhist[it - 1] : INFINITY;
    const bool stop = it >= 1 && r < ia.rmax && r > ia.theta * rprev;
    const bool diverge = !isfinite(r) || (it >= 1 && r > 2.0 * rprev && r > 1.0);
    const bool last = it + 1 >= ia.max_iter;
    if (tile == 0 && threadIdx.x == 0) {
        ic->rhist[it] = r;
        if (stop || diverge || last) {
            ic->done = 1;
            ic->iters = it;
            // no usable inverse (a diverging iteration, or none within the
            // slots): the molecule is reported NOT_SPD and the sign iteration,
            // finishing and extraction skip it, leaving its columns at zero
            if (diverge || !stop) {
                ctl->status = NOLSM_MOL_NOT_SPD;
                ctl->done = 1;
            }
        }
    }
    return (stop || diverge || last) ? IACT_STOP : IACT_UPDATE;
}

// One BM x BM tile of an inverse-route GEMM. `which` selects the product of
// the update (0: Y, 1: Z).
template <typename T, int BM>
__device__ __forceinline__ void inv_tile(const ChunkDev &cd, uint32_t task, char *ws, const InvArgs &ia, int it,
                                         int mode, int which, bool nt_out) {
    __shared__ double red[4];
    __shared__ int act_s;
    if (task == NOLSM_TASK_NONE) return;
    const int s = task_slot(task), ti = task_a(task), tj = task_b(task);
    const SubMeta M = cd.meta[s];
    SubCtl *ctl = cd.ctl + s;
    InvCtl *ic = cd.ictl + s;
    const int np = M.np, nt = (np + BM - 1) / BM, tile = ti * nt + tj, ldx = M.ldx;
    if (threadIdx.x < 64) {
        int act;
        if (ctl->status != NOLSM_MOL_OK) act = IACT_STOP;
        else if (mode == IM_R) act = ic->done ? IACT_STOP : IACT_UPDATE;
        else if (mode == IM_UPD) act = ic->done ? IACT_STOP : inv_decide(ia, M, ic, ctl, ws, it, tile);
        else act = IACT_UPDATE;   // after the loop: every OK slot
        if (threadIdx.x == 0) act_s = act;
    }
    __syncthreads();
    if (act_s == IACT_STOP) return;
    // buffers of iteration k: Y_k, Z_k in ping-pong slot k % 2
    const int K = (mode == IM_SQ || mode == IM_A) ? ic->iters : it;
    uint16_t *Yc = (uint16_t *)(ws + ((K & 1) ? M.offY1 : M.offY0));
    uint16_t *Yn = (uint16_t *)(ws + ((K & 1) ? M.offY0 : M.offY1));
    uint16_t *Zc = (uint16_t *)(ws + ((K & 1) ? M.offZ1 : M.offZ0));
    uint16_t *Zn = (uint16_t *)(ws + ((K & 1) ? M.offZ0 : M.offZ1));
    uint16_t *Rb = (uint16_t *)(ws + M.offB);
    // after the loop the Y buffers are free: S^-1 goes to Y0, K to Y1
    uint16_t *Sinv = (uint16_t *)(ws + M.offY0);
    uint16_t *K16 = (uint16_t *)(ws + M.offY1);
    const uint16_t *Ag, *Bg;
    switch (mode) {
        case IM_R: Ag = Zc; Bg = Yc; break;
        case IM_UPD: Ag = which ? Rb : Yc; Bg = which ? Zc : Rb; break;
        case IM_SQ: Ag = Zc; Bg = Zc; break;
        default: Ag = Sinv; Bg = K16; break;
    }
    constexpr int WT = BM / 2, NB = WT / 32;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w >> 1, wn = w & 1;
    uint16_t *st = lp_lds<BM>();
    const int rl = wm * WT + (l & 31), cl = wn * WT + (l >> 5) * 4, row0 = ti * BM, col0 = tj * BM;
    const double mu = ((const WsHeader *)ws)->mu, sc = (mode == IM_SQ) ? ic->scale : 0.0;
    double part = 0.0;
    auto finish = [&](v16f(&acc)[NB][NB]) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r = rl + i * 32, c = cl + j * 32 + q * 8, gr = row0 + r, gc = col0 + c;
                    uint2 *p = (uint2 *)(st + tile_idx<BM>(r, c));
                    uint16_t h[4];
                    if (mode == IM_A) {
                        // A_J = S^-1 K_J - mu I in FP64 (columns np.. of the
                        // K buffer hold Y_J)
                        double *Kb = (double *)(ws + M.offK) + (int64_t)gr * (np + 64) + gc;
                        double a[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) a[e] = (double)acc[i][j][4 * q + e] - (gr == gc + e ? mu : 0.0);
                        *(double2 *)Kb = make_double2(a[0], a[1]);
                        *(double2 *)(Kb + 2) = make_double2(a[2], a[3]);
                        continue;
                    }
                    if (mode == IM_R) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float v = (gr == gc + e ? 1.0f : 0.0f) - acc[i][j][4 * q + e];
                            part += (double)v * (double)v;
                            h[e] = Lp<T>::enc(v);
                        }
                    } else if (mode == IM_UPD) {
                        // Y_{k+1} = Y_k + Y_k R_k / 2 or Z_{k+1} = Z_k + R_k Z_k / 2
                        const uint2 x = *p;
                        const uint16_t y[4] = {(uint16_t)x.x, (uint16_t)(x.x >> 16), (uint16_t)x.y, (uint16_t)(x.y >> 16)};
#pragma unroll
                        for (int e = 0; e < 4; ++e) h[e] = enc_update<T>(y[e], acc[i][j][4 * q + e]);
                    } else {
                        // S^-1 = c Z_K^2 in 16 bits for the A GEMM; the columns
                        // of every owned molecule o (block position q_o) also
                        // go, from the FP32 accumulators, to its FP64 Y columns
                        // np + o bs .. of the K buffer
                        const int bs = ia.bs;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            h[e] = enc_scaled<T>((float)sc, acc[i][j][4 * q + e]);
                            const int qb = (gc + e) / bs;
                            for (int o = 0; o < M.nown; ++o)
                                if (ia.own_pos[M.own_off + o] == qb)
                                    ((double *)(ws + M.offK))[(int64_t)gr * (np + 64) + np + o * bs + (gc + e - qb * bs)] =
                                        sc * (double)acc[i][j][4 * q + e];
                        }
                    }
                    *p = pack4(h);
                }
    };
    lp_tile_product<T, BM, false>(Ag, Bg, mode == IM_UPD ? (which ? Zc : Yc) : nullptr, ldx, np, ti, tj, true,
                                  []() { return true; }, finish);
    if (mode == IM_A) return;
    if (mode == IM_R) {
        part = wave_sum(part);
        if (l == 0) red[w] = part;
    }
    __syncthreads();
    if (mode == IM_R && threadIdx.x == 0)
        ((double *)(ws + M.offRes))[(int64_t)it * M.ntile_ns + tile] = (red[0] + red[1]) + (red[2] + red[3]);
    tile_store<BM>(mode == IM_R ? Rb : mode == IM_SQ ? Sinv : which ? Zn : Yn, ldx, np, ti, tj, nt_out);
}

template <typename T, int BM>
__global__ __launch_bounds__(256, 3) void k_inv_lp(ChunkDev cd, const uint32_t *tasks, char *ws, InvArgs ia, int it,
                                                int mode) {
    inv_tile<T, BM>(cd, xcd_task(tasks), ws, ia, it, mode, blockIdx.y, lp_nt_out(gridDim.x, ia.pgrid));
}

// late iterations (scan_tasks): the tiles of the slots that still iterate
template <typename T, int BM>
__global__ __launch_bounds__(256, 2) void k_inv_tail(ChunkDev cd, const uint32_t *tasks, int ntask, char *ws, InvArgs ia,
                                                  int it, int mode) {
    scan_tasks(tasks, ntask, [&](int s) { return !cd.ictl[s].done && cd.ctl[s].status == NOLSM_MOL_OK; },
               [&](uint32_t task) {
                   inv_tile<T, BM>(cd, task, ws, ia, it, mode, blockIdx.y, lp_nt_out(ntask, ia.pgrid));
               });
}

// K_J (FP64, columns < np of the K buffer) to 16 bits in the Y1 buffer for
// the A GEMM; one workgroup per slot and 64 rows, eight values per thread.
template <typename T>
__global__ __launch_bounds__(256) void k_inv_k16(ChunkDev cd, char *ws) {
    const int s = blockIdx.x;
    if (s >= cd.nsub) return;
    const SubMeta M = cd.meta[s];
    if ((int)blockIdx.y >= M.P || cd.ctl[s].status != NOLSM_MOL_OK) return;
    const int np = M.np, ldx = M.ldx, r0 = blockIdx.y * 64, n8 = np / 8;
    const double *Kb = (const double *)(ws + M.offK);
    uint16_t *K16 = (uint16_t *)(ws + M.offY1);
#pragma unroll 2
    for (int f = threadIdx.x; f < 64 * n8; f += 256) {
        const int r = r0 + f / n8, q = (f % n8) * 8;
        const double2 *src = (const double2 *)(Kb + (int64_t)r * (np + 64) + q);
        uint32_t y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double2 v = src[k];
            y[k] = Lp<T>::enc((float)v.x) | ((uint32_t)Lp<T>::enc((float)v.y) << 16);
        }
        *(uint4 *)(K16 + (int64_t)r * ldx + q) = make_uint4(y[0], y[1], y[2], y[3]);
    }
}

// The bounds inputs the substitution would have written, from the FP64 A_J:
// for 64-column tile cc, partial |A| row sums (columns < n) per row, the
// complete |A| column sums (rows < n) and the tile's Frobenius share. Tasks
// (slot, cc) with cc <= P; cc = P (the Y tile) has nothing to add. Bound by
// the read of A_J: its 64 x 64 blocks pass through LDS (coalesced 16-byte
// loads, the next block's behind this one's sums), where wave 0 sums rows and
// wave 1 columns, in the order of the elements. With a row per thread read
// straight from memory 600 slots of about 612 rows took 2900 us; this, k_inv_init
// and k_inv_k16 together went from 6290 to 2050 us.
__global__ __launch_bounds__(256) void k_inv_sums(ChunkDev cd, char *ws) {
    __shared__ double tile[64][LDP];
    const uint32_t task = xcd_task(cd.t_subst);
    if (task == NOLSM_TASK_NONE) return;
    const int s = task_slot(task), cc = task_a(task);
    const SubMeta M = cd.meta[s];
    if (cd.ctl[s].status != NOLSM_MOL_OK || cc >= M.P) return;
    const int n = M.n, np = M.np, P = M.P, t = threadIdx.x;
    const int64_t ldk = np + 64;
    const double *A = (const double *)(ws + M.offK) + cc * 64;
    double *rowp = (double *)(ws + M.offRow);
    double *colp = (double *)(ws + M.offCol);
    const int nc = min(64, n - cc * 64);   // columns of this tile inside the matrix (may be none)
    double fs = 0.0, cs = 0.0;
    RegTile<double> pl;
    g2r_tile(pl, A, ldk);
    for (int b = 0; b < P; ++b) {
        r2s_tile(tile, pl);
        __syncthreads();
        if (b + 1 < P) g2r_tile(pl, A + (int64_t)(b + 1) * 64 * ldk, ldk);
        if (t < 64) {
            double rs = 0.0;
            if (b * 64 + t < n)
#pragma unroll 8
                for (int c = 0; c < nc; ++c) {
                    const double v = tile[t][c];
                    rs += fabs(v);
                    fs += v * v;
                }
            rowp[(int64_t)cc * np + b * 64 + t] = rs;
        } else if (t < 128) {
            const int nr = min(64, n - b * 64);
#pragma unroll 8
            for (int r = 0; r < nr; ++r) cs += fabs(tile[r][t - 64]);
        }
        __syncthreads();
    }
    if (t < 64) {
        fs = wave_sum(fs);
        if (t == 0) colp[np + cc] = fs;
    } else if (t < 128) {
        colp[cc * 64 + t - 64] = t - 64 < nc ? cs : 0.0;
    }
}

// Iterations from this one on take the scanning launch: with 600 slots of
// about 612 rows, converged after 10 of 40 iterations, a launch takes 4.5 us
// instead of 14 (R) and 25 (the update).
#define INV_TAIL_IT 16
template <typename T, int BM>
static void launch_inv_gemm(const ChunkDev &cd, const uint32_t *tasks, int ntask, char *ws, const InvArgs &ia, int it,
                            int mode, int nprod, hipStream_t st) {
    if (ntask <= 0) return;
    if (it < INV_TAIL_IT)
        hipLaunchKernelGGL((k_inv_lp<T, BM>), dim3(ntask, nprod), dim3(256), 0, st, cd, tasks, ws, ia, it, mode);
    else
        hipLaunchKernelGGL((k_inv_tail<T, BM>), dim3(scan_grid(ia.pgrid, ntask), nprod), dim3(256), 0, st, cd, tasks,
                           ntask, ws, ia, it, mode);
}
template <typename T>
static void launch_inv_gemm(const ChunkDev &cd, char *ws, const InvArgs &ia, int it, int mode, int nprod,
                            hipStream_t st) {
    launch_inv_gemm<T, 128>(cd, cd.t_ns, cd.n_ns, ws, ia, it, mode, nprod, st);
    launch_inv_gemm<T, 64>(cd, cd.t_ns64, cd.n_ns64, ws, ia, it, mode, nprod, st);
}

template <typename T>
static hipError_t run_inverse(const ChunkDev &cd, char *ws, const InvArgs &ia, hipStream_t st) {
    hipLaunchKernelGGL(k_inv_init<T>, dim3(cd.nsub), dim3(1024), 0, st, cd, ws);
    for (int it = 0; it < ia.max_iter; ++it) {
        launch_inv_gemm<T>(cd, ws, ia, it, IM_R, 1, st);
        launch_inv_gemm<T>(cd, ws, ia, it, IM_UPD, 2, st);
    }
    hipLaunchKernelGGL(k_inv_k16<T>, dim3(cd.nsub, cd.max_np / 64), dim3(256), 0, st, cd, ws);
    launch_inv_gemm<T>(cd, ws, ia, 0, IM_SQ, 1, st);
    launch_inv_gemm<T>(cd, ws, ia, 0, IM_A, 1, st);
    hipLaunchKernelGGL(k_inv_sums, dim3(cd.n_subst), dim3(256), 0, st, cd, ws);
    return hipGetLastError();
}

hipError_t launch_inverse(const ChunkDev &cd, char *ws, const InvArgs &ia, hipStream_t st) {
    if (!cd.ictl) return hipErrorInvalidValue;
    return ia.prec == NOLSM_FP16 ? run_inverse<_Float16>(cd, ws, ia, st) : run_inverse<__bf16>(cd, ws, ia, st);
}
