// Newton-Schulz sign iteration on the matrix cores (Sec. III-B.2, Eq. NS1-NS2;
// Sec. III-C.3: the iteration runs as GEMMs in mixed precision).
//
// One iteration is two batched GEMM launches over the tiles of every active
// submatrix of a chunk:
//   mode 1: T = X_k X_k; epilogue: partial sums of ||T - I||_F^2 per tile and
//           R = I - T stored in the iteration precision;
//   mode 2: every workgroup of a submatrix reads the finished residual
//           r_k = ||X_k^2 - I||_F, takes the same stop/continue/restart
//           decision, and if continuing writes X_{k+1} = X_k + X_k R / 2,
//           which equals X_k (3I - X_k^2) / 2 of Eq. NS1.
// X ping-pongs between two buffers (X_k in buffer k % 2). Precisions:
// FP64 / FP32 use 64x64 tiles on v_mfma_f64_16x16x4 / v_mfma_f32_16x16x4;
// FP16 / BF16 use 128x128 (or 64x64) tiles on v_mfma_f32_32x32x16_{f16,bf16}
// with FP32 accumulation.
#include "dev_common.h"
#include "kernels.h"
#include "lp_gemm.h"

enum { ACT_STOP = 0, ACT_UPDATE = 1, ACT_RESTART = 2 };

// Decision of mode 2 at iteration `it`. Computed by wave 0 of every
// workgroup of the submatrix from data that is final before this launch
// (the residual partials of mode 1 and rhist[0..it-1]); the tile-0
// workgroup records it. More than a few partials are read side by side: one
// thread's chain of 25 additions took about 1.5 us of a tile.
__device__ int ns_decide(const NsArgs &na, const SubMeta &M, SubCtl *ctl, const char *ws, int it, int tile,
                         bool done) {
    const double *res = (const double *)(ws + M.offRes) + (int64_t)it * M.ntile_ns;
    double ssum = 0.0;
    if (M.ntile_ns <= 9) {
        for (int i = 0; i < M.ntile_ns; ++i) ssum += res[i];
    } else {
        for (int i = threadIdx.x; i < M.ntile_ns; i += 64) ssum += res[i];
        ssum = wave_sum(ssum);
    }
    const double rprev = it > 0 ? ctl->rhist[it - 1] : INFINITY;
    const int ra = ctl->restart_at;
    // the reads above go out beside the one of `done`, not behind it
    asm volatile("" ::"v"(ssum), "v"(rprev), "v"(ra));
    if (done) return ACT_STOP;
    const double r = sqrt(ssum);
    bool stop;
    if (na.fixed_iters > 0)
        stop = it >= na.fixed_iters;
    else if (na.prec == NOLSM_FP64)
        stop = r < na.tol;
    else
        stop = (na.tol > 0.0 && r < na.tol) || (it >= 1 && r < na.rmax && r > na.theta * rprev);
    // a stall injected from the host for one molecule counts as divergence
    // at one iteration, so that the restart path can be checked (every
    // workgroup of the submatrix takes the same decision from `it` alone;
    // restart_at may already hold it + 1 from the tile-0 workgroup)
    const bool forced = na.force_stall >= 0 && M.J == na.force_stall && it == na.stall_it;
    const bool diverge = forced || !isfinite(r) || (it >= 1 && r > 2.0 * rprev && r > 1.0);
    int act;
    bool noconv = false;
    if (diverge && na.allow_restart && (ra < 0 || ra == it + 1)) {
        act = ACT_RESTART;
    } else if (diverge) {
        act = ACT_STOP;
        noconv = true;
    } else if (stop) {
        act = ACT_STOP;
    } else if (it + 1 >= na.max_iter) {
        act = ACT_STOP;
        noconv = na.fixed_iters <= 0;
    } else {
        act = ACT_UPDATE;
    }
    if (tile == 0 && threadIdx.x == 0) {
        ctl->rhist[it] = r;
        if (act == ACT_STOP) {
            ctl->iters = it;
            ctl->resid = r;
            // a status set earlier (NOT_SPD) is never overwritten
            if (noconv && ctl->status == NOLSM_MOL_OK) ctl->status = NOLSM_MOL_NOCONV;
            ctl->done = 1;
        } else if (act == ACT_RESTART) {
            ctl->fallback = 1;
            ctl->restart_at = it + 1;
            ctl->scale = ctl->scale_g;
        }
    }
    return act;
}

// X_{k+1} tile <- c_G A on [0,n)^2, identity on the padding (restart);
// sym: from the upper triangle of A, so that the restart is exactly symmetric
template <typename T, typename Cvt>
__device__ void restart_tile(const SubMeta &M, const SubCtl *ctl, const char *ws, T *Xn, int r0, int c0,
                             int rows, int cols, Cvt cvt, bool sym = false) {
    const int64_t ldk = M.np + 64;
    const double c = ctl->scale_g;
    for (int f = threadIdx.x; f < rows * cols; f += blockDim.x) {
        const int r = r0 + f / cols, q = c0 + f % cols;
        if (r >= M.np || q >= M.np) continue;
        const int ra = sym ? min(r, q) : r, qa = sym ? max(r, q) : q;
        const double v = (r < M.n && q < M.n) ? c * kbuf_get(M, ws, (int64_t)ra * ldk + qa) : (r == q ? 1.0 : 0.0);
        Xn[(int64_t)r * M.ldx + q] = cvt(v);
    }
}

// ------------------------------------------------------------ FP64 / FP32
template <typename T> struct Mma16;
// Output row of element e in lane group lk = l/16 (column is l%16 for both).
template <> struct Mma16<double> {
    typedef v4d acc_t;
    static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lk, int e) { return lk + 4 * e; }
};
template <> struct Mma16<float> {
    typedef v4f acc_t;
    static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lk, int e) { return 4 * lk + e; }
};

// LDS strides of the operand slices (64 x BK of A, BK x 32 NC of B), in
// values: an A operand read touches 16 rows and 4 (FP32) or 2 (FP64, per
// half-wave) neighbouring k, a B operand read 16 neighbouring columns of as
// many k rows, and each falls on distinct banks; rows start 16-byte aligned
template <typename T, int NC> struct Ns64Tile {
    static constexpr int BK = NC == 4 ? 32 : 64;
    static constexpr int LA = BK + (sizeof(T) == 8 ? 2 : 4), LB = 32 * NC + 16;
};

// One 64 x 32 NC output tile of one half-iteration (body shared by the
// one-workgroup-per-tile launch and the persistent queue launch): NC = 2, one
// 64-column tile, or NC = 4, two of them, tj and tj + 1 (the second may be
// past the matrix). The matrix cores bound it. With NC = 4 each wave holds
// 32 x 64 as 2 x 4 blocks, whose eight chains of products keep a SIMD's
// matrix core busy from two waves on (four chains a wave reached 125 of 155
// TF/s in FP32 with four waves): 512 submatrices of about 612 rows in FP64
// 4433 us a launch against 4834 with NC = 2 (5938 before the slices were
// fetched ahead), 777 in FP32 3296 against 3716 (3850). NC = 2 serves size
// ranges with too few of the wider tiles to fill the GPU. The next slice is
// fetched into registers while this one is multiplied from LDS. The
// contraction stops at n (X_k and R are identity and zero on the padding,
// whose products are exact zeros), and the padding of a result is set rather
// than computed.
template <typename T, int NC>
__device__ __forceinline__ void ns64_tile(const ChunkDev &cd, uint32_t task, char *ws, const NsArgs &na, int it,
                                          int mode) {
    typedef typename Mma16<T>::acc_t acc_t;
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    constexpr int BK = Ns64Tile<T, NC>::BK, LA = Ns64Tile<T, NC>::LA, LB = Ns64Tile<T, NC>::LB;
    constexpr int BN = 32 * NC, VE = 16 / sizeof(T);
    constexpr int AL = BK / VE, AR = 256 / AL, AP = 64 / AR;    // lanes per row, rows per pass, passes of A
    constexpr int BL = BN / VE, BR = 256 / BL, BP = BK / BR;   // and of B
    __shared__ __attribute__((aligned(16))) T sA[64 * LA];
    __shared__ __attribute__((aligned(16))) T sB[BK * LB];
    __shared__ double red[4];
    __shared__ int act_s;
    if (task == NOLSM_TASK_NONE) return;
    const int s = task_slot(task), ti = task_a(task), tj = task_b(task);
    const SubMeta M = cd.meta[s];
    SubCtl *ctl = cd.ctl + s;
    const int np = M.np, n = M.n, nt = np / 64, tile = ti * nt + tj;
    T *Xc = (T *)(ws + ((it & 1) ? M.offX1 : M.offX0));
    T *Xn = (T *)(ws + ((it & 1) ? M.offX0 : M.offX1));
    T *Bb = (T *)(ws + M.offB);
    // wave 0 reads the control state and decides for the whole workgroup
    if (threadIdx.x < 64) {
        const bool done = ctl->done != 0;
        const int act = mode == 2 ? ns_decide(na, M, ctl, ws, it, tile, done) : (done ? ACT_STOP : ACT_UPDATE);
        if (threadIdx.x == 0) act_s = act;
    }
    __syncthreads();
    {
        const int act = act_s;
        if (act == ACT_STOP) return;
        if (act == ACT_RESTART) {
            // columns past np are left alone
            restart_tile(M, ctl, ws, Xn, ti * 64, tj * 64, 64, BN, [](double v) { return (T)v; });
            return;
        }
    }
    const T *Bop = (mode == 1) ? Xc : Bb;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63;
    const int r0 = (w >> 1) * 32, c0 = (w & 1) * 16 * NC;
    const int li = l & 15, lk = l >> 4;
    const int ar = t / AL, ac = (t % AL) * VE, br = t / BL, bc = (t % BL) * VE;
    const T *Ag = Xc + (int64_t)(ti * 64 + ar) * np + ac, *Bg = Bop + (int64_t)br * np + tj * 64 + bc;
    const bool bin = tj * 64 + bc < np;
    const int nk = (n + BK - 1) / BK;
    vec pa[AP], pb[BP];
#pragma unroll
    for (int p = 0; p < BP; ++p) pb[p] = (vec)0;
    auto fetch = [&](int kt) {
#pragma unroll
        for (int p = 0; p < AP; ++p) pa[p] = *(const vec *)(Ag + (int64_t)p * AR * np + kt * BK);
        if (bin)
#pragma unroll
            for (int p = 0; p < BP; ++p) pb[p] = *(const vec *)(Bg + (int64_t)(kt * BK + p * BR) * np);
    };
    auto stash = [&]() {
#pragma unroll
        for (int p = 0; p < AP; ++p) *(vec *)(sA + (ar + p * AR) * LA + ac) = pa[p];
#pragma unroll
        for (int p = 0; p < BP; ++p) *(vec *)(sB + (br + p * BR) * LB + bc) = pb[p];
    };
    double part = 0.0;
    fetch(0);
    stash();
    __syncthreads();
    if (tj * 64 + c0 >= np) {
        // past the matrix: this wave only loads and stores for the others
        for (int kt = 0; kt + 1 < nk; ++kt) {
            fetch(kt + 1);
            __syncthreads();
            stash();
            __syncthreads();
        }
    } else {
        acc_t acc[2][NC];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NC; ++j) acc[i][j] = (acc_t){0, 0, 0, 0};
        const T *ra = sA + (r0 + li) * LA + lk, *rb = sB + lk * LB + c0 + li;
        auto step = [&](int k) {
            T a[2], b[NC];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = ra[i * 16 * LA + 4 * k];
#pragma unroll
            for (int j = 0; j < NC; ++j) b[j] = rb[4 * k * LB + j * 16];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NC; ++j) acc[i][j] = Mma16<T>::mma(a[i], b[j], acc[i][j]);
        };
        for (int kt = 0; kt + 1 < nk; ++kt) {
            fetch(kt + 1);
            __builtin_amdgcn_sched_barrier(0);   // ahead of the products, not next to their use
#pragma unroll
            for (int k = 0; k < BK / 4; ++k) step(k);
            __syncthreads();
            stash();
            __syncthreads();
        }
        const int ks = (n - (nk - 1) * BK + 3) / 4;   // the last slice, to n
        for (int k = 0; k < ks; ++k) step(k);
        const int gr0 = ti * 64 + r0, gc0 = tj * 64 + c0 + li;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            T x[NC][4];
            if (mode == 2)   // X_k of the block row, all loads before the stores
#pragma unroll
                for (int j = 0; j < NC; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        x[j][e] = Xc[(int64_t)(gr0 + i * 16 + Mma16<T>::row(lk, e)) * np + gc0 + j * 16];
#pragma unroll
            for (int j = 0; j < NC; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int gr = gr0 + i * 16 + Mma16<T>::row(lk, e);
                    const int gc = gc0 + j * 16;
                    const bool pad = gr >= n || gc >= n;
                    const T v = acc[i][j][e];
                    const int64_t o = (int64_t)gr * np + gc;
                    if (mode == 1) {
                        // R = I - X^2; the update below is X + X R / 2 = X (3I - X^2) / 2
                        const T rr = pad ? (T)0 : (gr == gc ? (T)1 : (T)0) - v;
                        part += (double)rr * (double)rr;
                        Bb[o] = rr;
                    } else {
                        Xn[o] = pad ? x[j][e] : x[j][e] + (T)0.5 * v;
                    }
                }
        }
    }
    if (mode == 1) {
        part = wave_sum(part);
        if (l == 0) red[w] = part;
        __syncthreads();
        if (t == 0) {
            double *res = (double *)(ws + M.offRes) + (int64_t)it * M.ntile_ns;
            res[tile] = (red[0] + red[1]) + (red[2] + red[3]);
            if (NC == 4 && tj + 1 < nt) res[tile + 1] = 0.0;
        }
    }
}

// Persistent launches: a fixed grid whose workgroups pop entries from the
// task-list segment of their XCD through an atomic counter (one counter per
// XCD, per launch, zeroed at chunk start). No workgroup ever waits for
// another one, so every wave exits once its segment is drained.
__device__ __forceinline__ int queue_pop(int *q, int *slot) {
    __syncthreads();
    if (threadIdx.x == 0) *slot = atomicAdd(q, 1);
    __syncthreads();
    return *slot;
}

template <typename T, int NC>
__global__ __launch_bounds__(256, sizeof(T) == 8 ? 2 : 3) void k_ns64(ChunkDev cd, const uint32_t *tasks, char *ws,
                                                                    NsArgs na, int it, int mode) {
    ns64_tile<T, NC>(cd, xcd_task(tasks), ws, na, it, mode);
}

// the slots that a scanning launch still has to work on
__device__ __forceinline__ auto iterating(const ChunkDev &cd) {
    return [&cd](int s) { return !cd.ctl[s].done; };
}

// The iterations from `it0` on of a small chunk as one launch: its workgroups
// scan their tasks (scan_tasks) and work on every submatrix that still iterates
// until it is done. What bounds the late launches of a small chunk is their
// number: 48 (FP16) or 60 (FP64) a chunk, 2.5 to 4.5 us each, when all is
// converged (64 submatrices of about 350 rows: 834 -> 583 us of iteration in
// FP16, 1402 -> 1166 us in FP64).
//
// A submatrix' tiles of both halves of every remaining iteration are handed
// out in order by a counter (rest_next); a tile of one half starts when all
// tiles of the half before are counted as complete (rest_fin). A workgroup
// holds one uncounted half at a time and counts it before it waits for the
// next, so it only ever waits for lower numbers, which running workgroups
// hold: the lowest open one never waits, and every wait ends whatever share
// of the grid is resident. tile(a, b, it, mode) runs one tile; the tiles of a
// submatrix are ncol columns of bstep per tile row, or (SYM) its upper tiles.
// Which workgroup runs a tile does not change its result.
template <bool SYM, typename Tile>
__device__ __forceinline__ void rest_of(SubCtl *ctl, int nt, int bstep, int it0, int max_iter, Tile tile) {
    __shared__ int next_s;
    const int ncol = (nt + bstep - 1) / bstep, ntile = SYM ? nt * (nt + 1) / 2 : nt * ncol;
    int mine = 0, last = -1;   // tiles run and not yet counted, their half
    for (;;) {
        // one block of thread 0 a turn, with a barrier on either side of it:
        // no branch on the thread leads from the end of a turn to the next,
        // so no wave goes round the loop without its first lane. Keep it so.
        // With a second block of thread 0 at the end of the turn (to count its
        // tile), and no barrier between that and this one, the compiler joined
        // the two: lanes 1 to 63 went on to the barriers of the next turn by
        // themselves, and the kernel hung. It does not move a branch across a
        // barrier.
        if (threadIdx.x == 0) {
            int k = __hip_atomic_fetch_add(&ctl->rest_next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int half = k / ntile;
            if (half != last) {
                // the tiles of the half before, written back once for all XCDs
                if (mine) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the write-back too
                    __hip_atomic_fetch_add(&ctl->rest_fin, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (half >= 2 * (max_iter - it0)) k = -1;
                while (k >= 0) {
                    // `done` after rest_fin: the half that set it then shows
                    // it. (No acquire here: every turn of the wait would
                    // empty the L2 that the other workgroups work from.)
                    const bool ready =
                        __hip_atomic_load(&ctl->rest_fin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= half * ntile;
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    if (__hip_atomic_load(&ctl->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) k = -1;
                    else if (ready) break;
                    else __builtin_amdgcn_s_sleep(8);
                }
            }
            next_s = k;
        }
        __syncthreads();
        const int k = __builtin_amdgcn_readfirstlane(next_s);
        if (k < 0) break;
        const int half = k / ntile, x = k - half * ntile;
        if (half != last) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // what other workgroups have written, on any XCD
            last = half;
            mine = 0;
        }
        ++mine;
        int a = 0, b = x;
        if (SYM) {
            while (b >= nt - a) b -= nt - a, ++a;
            b += a;
        } else {
            a = x / ncol;
            b = (x - a * ncol) * bstep;
        }
        tile(a, b, it0 + (half >> 1), 1 + (half & 1));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // each wave: its stores have reached L2
        __syncthreads();
    }
    __syncthreads();
}
template <typename T, int NC>
__global__ __launch_bounds__(256, 2) void k_ns64_tail(ChunkDev cd, const uint32_t *tasks, int ntask, char *ws, NsArgs na,
                                                    int it, int mode) {
    scan_tasks(tasks, ntask, iterating(cd), [&](uint32_t task) { ns64_tile<T, NC>(cd, task, ws, na, it, mode); });
}

template <typename T, int NC>
__global__ __launch_bounds__(256, 2) void k_ns64_rest(ChunkDev cd, const uint32_t *tasks, int ntask, char *ws, NsArgs na,
                                                    int it0) {
    scan_tasks(tasks, ntask, iterating(cd), [&](uint32_t task) {
        const int s = task_slot(task);
        rest_of<false>(cd.ctl + s, cd.meta[s].np / 64, NC / 2, it0, na.max_iter, [&](int a, int b, int it, int mode) {
            ns64_tile<T, NC>(cd, NOLSM_TASK(s, a, b), ws, na, it, mode);
        });
    });
}

template <typename T, int NC>
__global__ __launch_bounds__(256, sizeof(T) == 8 ? 2 : 3) void k_ns64_pq(ChunkDev cd, const uint32_t *tasks, int ntask,
                                                                       int *q, char *ws, NsArgs na, int it, int mode) {
    __shared__ int idx_s;
    const int x = blockIdx.x & 7, seg = ntask >> 3;
    for (;;) {
        const int i = queue_pop(q + x, &idx_s);
        if (i >= seg) break;
        ns64_tile<T, NC>(cd, tasks[x * seg + i], ws, na, it, mode);
    }
}

// ------------------------------------------------------------ FP16 / BF16
// Output tile (ti, tj) of the symmetric iteration from its LDS copy
// (tile_idx), 16-byte row stores of the rows and columns below np. A
// diagonal tile is written exactly symmetric, from its upper triangle: X R
// is symmetric only in exact arithmetic, and an iteration whose B operand is
// read as rows (X^T) doubles the skew part that anticommutes with the sign
// at every step.
template <int BM> __device__ __forceinline__ void sym_store(uint16_t *X, int ldx, int np, int ti, int tj, bool nt) {
    constexpr int NCH = BM / 8;
    const uint16_t *st = lp_lds<BM>();
    const int row0 = ti * BM, col0 = tj * BM;
    // eight values from a function of their position
    auto pack = [](auto at) {
        return make_uint4((uint32_t)at(0) | ((uint32_t)at(1) << 16), (uint32_t)at(2) | ((uint32_t)at(3) << 16),
                          (uint32_t)at(4) | ((uint32_t)at(5) << 16), (uint32_t)at(6) | ((uint32_t)at(7) << 16));
    };
#pragma unroll 4
    for (int f = threadIdx.x; f < BM * NCH; f += 256) {
        const int r = f / NCH, c0 = (f % NCH) * 8;
        if (row0 + r >= np || col0 + c0 >= np) continue;
        uint4 v;
        if (ti != tj || c0 >= r)
            v = *(const uint4 *)(st + tile_idx<BM>(r, c0));
        else
            v = pack([&](int k) { return st[tile_idx<BM>(min(r, c0 + k), max(r, c0 + k))]; });
        store16(X + (int64_t)(row0 + r) * ldx + col0 + c0, v, nt);
        if (BM == 64 && ti != tj)   // both triangles are stored: row r of the transpose
            store16(X + (int64_t)(col0 + r) * ldx + row0 + c0, pack([&](int k) { return st[tile_idx<BM>(c0 + k, r)]; }),
                    nt);
    }
}

// One BM x BM tile of a sign-iteration GEMM: mode 1 forms R = I - X_k^2 and
// the tile's share of ||R||_F^2, mode 2 decides stop / continue / restart and
// forms X_{k+1} = X_k + X_k R / 2. SYM: the upper tiles of the symmetric
// iteration; with 128-row tiles X_k and R are stored by their upper tiles,
// and so are the results, and what is left below the diagonal tiles is never
// read until it is filled in for the returned iterate.
template <typename T, int BM, bool SYM>
__device__ __forceinline__ void ns_tile(const ChunkDev &cd, uint32_t task, char *ws, const NsArgs &na, int it,
                                        int mode) {
    __shared__ double red[4];
    __shared__ int act_s;
    if (task == NOLSM_TASK_NONE) return;
    const int s = task_slot(task), ti = task_a(task), tj = task_b(task);
    const SubMeta M = cd.meta[s];
    SubCtl *ctl = cd.ctl + s;
    const int np = M.np, ldx = M.ldx, nt = (np + BM - 1) / BM, tile = ti * nt + tj;
    uint16_t *Xc = (uint16_t *)(ws + ((it & 1) ? M.offX1 : M.offX0));
    uint16_t *Xn = (uint16_t *)(ws + ((it & 1) ? M.offX0 : M.offX1));
    uint16_t *Bb = (uint16_t *)(ws + M.offB);
    // a converged submatrix costs one read. In mode 2 another workgroup may
    // record this iteration's stop meanwhile: whichever wave sees it loads
    // nothing, and `begin` comes to the same stop for all of them.
    const bool done = __builtin_amdgcn_readfirstlane(*(volatile int32_t *)&ctl->done) != 0;
    if (done && mode == 1) return;
    // wave 0 reads the control state and decides for the whole workgroup
    auto begin = [&]() {
        if (mode == 1) return true;
        if (threadIdx.x < 64) {
            const int act = ns_decide(na, M, ctl, ws, it, tile, done);
            if (threadIdx.x == 0) act_s = act;
        }
        __syncthreads();
        if (act_s == ACT_RESTART) {
            auto enc = [](double v) { return Lp<T>::enc((float)v); };
            restart_tile(M, ctl, ws, Xn, ti * BM, tj * BM, BM, BM, enc, SYM);
            if (SYM && BM == 64 && ti != tj) restart_tile(M, ctl, ws, Xn, tj * BM, ti * BM, BM, BM, enc, true);
        }
        return act_s == ACT_UPDATE;
    };
    constexpr int WT = BM / 2, NB = WT / 32;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w >> 1, wn = w & 1;
    uint16_t *st = lp_lds<BM>();
    const int rl = wm * WT + (l & 31), cl = wn * WT + (l >> 5) * 4;
    double part = 0.0;
    auto finish = [&](v16f(&acc)[NB][NB]) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r = rl + i * 32, c = cl + j * 32 + q * 8;
                    uint2 *p = (uint2 *)(st + tile_idx<BM>(r, c));
                    uint16_t o[4];
                    if (mode == 1) {
                        // R = I - X^2 is small near convergence and keeps full
                        // relative precision in 16 bits (3I - X^2 would not: its
                        // diagonal ~2 is quantised at 2^-9 in FP16)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float v = ((ti == tj && r == c + e) ? 1.0f : 0.0f) - acc[i][j][4 * q + e];
                            part += (double)v * (double)v;
                            o[e] = Lp<T>::enc(v);
                        }
                    } else {
                        // X_{k+1} = X_k + X_k R / 2 = X_k (3I - X_k^2) / 2, X_k
                        // from LDS, the result in its place
                        const uint2 x = *p;
                        const uint16_t h[4] = {(uint16_t)x.x, (uint16_t)(x.x >> 16), (uint16_t)x.y, (uint16_t)(x.y >> 16)};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if constexpr (SYM) {
                                // rounded to FP32 and then to 16 bits
                                float v = Lp<T>::dec(h[e]) + 0.5f * acc[i][j][4 * q + e];
                                asm volatile("" : "+v"(v));
                                o[e] = Lp<T>::enc(v);
                            } else {
                                o[e] = enc_update<T>(h[e], acc[i][j][4 * q + e]);
                            }
                        }
                    }
                    *p = pack4(o);
                }
    };
    if (!lp_tile_product<T, BM, SYM>(Xc, mode == 1 ? Xc : Bb, mode == 1 ? nullptr : Xc, ldx, np, ti, tj, !done,
                                     begin, finish))
        return;
    if (mode == 1) {
        // SYM: a value off the diagonal counts for its mirror too
        part = wave_sum(part) * ((SYM && (ti != tj || wm < wn)) ? 2.0 : 1.0);
        if (l == 0) red[w] = part;
    }
    __syncthreads();
    if (mode == 1 && threadIdx.x == 0) {
        double *res = (double *)(ws + M.offRes) + (int64_t)it * M.ntile_ns;
        res[tile] = (red[0] + red[1]) + (red[2] + red[3]);
        if (SYM && ti != tj) res[tj * nt + ti] = 0.0;   // the mirror tile is never launched
    }
    if constexpr (SYM) sym_store<BM>(mode == 1 ? Bb : Xn, ldx, np, ti, tj, na.nt_out);
    else tile_store<BM>(mode == 1 ? Bb : Xn, ldx, np, ti, tj, na.nt_out);
}

// Fills in the tiles below the diagonal of the returned iterate, which the
// finishing products read by rows: tile (tj, ti) is the transpose of the
// stored tile (ti, tj). One pass over the matrix, against one saved in every
// half-iteration by not storing them.
__global__ __launch_bounds__(256) void k_ns_mirror(ChunkDev cd, char *ws) {
    const uint32_t task = xcd_task(cd.t_ns);   // 128-row tiles
    if (task == NOLSM_TASK_NONE) return;
    const int s = task_slot(task), ti = task_a(task), tj = task_b(task);
    if (ti == tj) return;
    const SubMeta M = cd.meta[s];
    const SubCtl *ctl = cd.ctl + s;
    if (ctl->status == NOLSM_MOL_NOT_SPD) return;
    const int w = threadIdx.x >> 6, r0 = ti * 128 + (w >> 1) * 64, c0 = tj * 128 + (w & 1) * 64;
    if (c0 >= M.np) return;   // ti < tj: r0 is below np
    mirror_block((uint16_t *)(ws + ((ctl->iters & 1) ? M.offX1 : M.offX0)), M.ldx, r0, c0);
}

template <typename T, int BM, bool SYM>
__global__ __launch_bounds__(256, 3) void k_ns_lp(ChunkDev cd, const uint32_t *tasks, char *ws, NsArgs na, int it,
                                               int mode) {
    ns_tile<T, BM, SYM>(cd, xcd_task(tasks), ws, na, it, mode);
}

template <typename T, int BM, bool SYM>
__global__ __launch_bounds__(256, 3) void k_ns_lp_pq(ChunkDev cd, const uint32_t *tasks, int ntask, int *q, char *ws,
                                                  NsArgs na, int it, int mode) {
    __shared__ int idx_s;
    const int x = blockIdx.x & 7, seg = ntask >> 3;
    for (;;) {
        const int i = queue_pop(q + x, &idx_s);
        if (i >= seg) break;
        ns_tile<T, BM, SYM>(cd, tasks[x * seg + i], ws, na, it, mode);
    }
}

template <typename T, int BM, bool SYM>
__global__ __launch_bounds__(256, 2) void k_ns_lp_tail(ChunkDev cd, const uint32_t *tasks, int ntask, char *ws,
                                                    NsArgs na, int it, int mode) {
    scan_tasks(tasks, ntask, iterating(cd), [&](uint32_t task) { ns_tile<T, BM, SYM>(cd, task, ws, na, it, mode); });
}

template <typename T, int BM, bool SYM>
__global__ __launch_bounds__(256, 2) void k_ns_lp_rest(ChunkDev cd, const uint32_t *tasks, int ntask, char *ws,
                                                    NsArgs na, int it0) {
    scan_tasks(tasks, ntask, iterating(cd), [&](uint32_t task) {
        const int s = task_slot(task);
        rest_of<SYM>(cd.ctl + s, (cd.meta[s].np + BM - 1) / BM, 1, it0, na.max_iter,
                     [&](int a, int b, int it, int mode) {
                         ns_tile<T, BM, SYM>(cd, NOLSM_TASK(s, a, b), ws, na, it, mode);
                     });
    });
}
// iterations from this one on take the scanning launch (FP64 / FP32, which
// iterate longer: from the second one on; 64 launches after convergence then
// take 4 us each instead of 75 on 512 submatrices of about 612 rows)
#define NS_TAIL_IT 16
#define NS64_TAIL_IT 18
// and in a small chunk from these on one launch runs what is left. Where
// submatrices do still iterate, a tile behind a counter takes longer than in
// a launch of its own (every half writes back and empties the L2s), the more
// so the more of them: 216 submatrices of about 600 rows, all of them
// iterating, take 433 against 345 us an iteration (FP16), which the launches
// saved outweigh up to two such iterations, 64 of about 350 rows 61 against 32
// us, up to seven (FP64 127 against 63, up to four: so it starts later
// there); 1000 of about 600 rows 1940 against 1490 us, with 1% to gain. Hence
// chunks of at most eight tasks per workgroup of pgrid.
#define NS_REST_IT 16
#define NS64_REST_IT 22
static bool rest_chunk(const NsArgs &na, int ntask) { return ntask <= 8 * na.pgrid; }
// queue counters of one launch: [iteration][half][tile class][XCD]
static int *launch_queue(const ChunkDev &cd, int it, int mode, int cls) {
    return cd.queues + (((size_t)it * 2 + (mode - 1)) * 2 + cls) * 8;
}
static int persistent_grid(const NsArgs &na, int ntask) {
    int g = na.pgrid < ntask ? na.pgrid : ntask;
    g = (g + 7) / 8 * 8;
    return g < 8 ? 8 : g;
}

template <typename T, int BM, bool SYM>
static void launch_lp(const ChunkDev &cd, const uint32_t *tasks, int ntask, char *ws, const NsArgs &na, int it, int mode,
                      hipStream_t st) {
    if (ntask <= 0) return;
    if (na.persistent)
        hipLaunchKernelGGL((k_ns_lp_pq<T, BM, SYM>), dim3(persistent_grid(na, ntask)), dim3(256), 0, st, cd, tasks, ntask,
                           launch_queue(cd, it, mode, BM == 64), ws, na, it, mode);
    else if (it < NS_TAIL_IT)
        hipLaunchKernelGGL((k_ns_lp<T, BM, SYM>), dim3(ntask), dim3(256), 0, st, cd, tasks, ws, na, it, mode);
    else if (it < NS_REST_IT || !rest_chunk(na, ntask))
        hipLaunchKernelGGL((k_ns_lp_tail<T, BM, SYM>), dim3(scan_grid(na.pgrid, ntask)), dim3(256), 0, st, cd, tasks, ntask, ws,
                           na, it, mode);
    else if (it == NS_REST_IT && mode == 1)
        hipLaunchKernelGGL((k_ns_lp_rest<T, BM, SYM>), dim3(scan_grid(na.pgrid, ntask)), dim3(256), 0, st, cd, tasks, ntask, ws,
                           na, it);
}
template <typename T, bool SYM>
static void launch_lp(const ChunkDev &cd, char *ws, NsArgs na, int it, int mode, hipStream_t st) {
    na.nt_out = lp_nt_out(cd.n_ns, na.pgrid);
    launch_lp<T, 128, SYM>(cd, cd.t_ns, cd.n_ns, ws, na, it, mode, st);
    launch_lp<T, 64, SYM>(cd, cd.t_ns64, cd.n_ns64, ws, na, it, mode, st);
}

template <typename T, int NC>
static void launch_64(const ChunkDev &cd, const uint32_t *tasks, int ntask, char *ws, const NsArgs &na, int it, int mode,
                      hipStream_t st) {
    if (ntask <= 0) return;
    if (na.persistent)
        hipLaunchKernelGGL((k_ns64_pq<T, NC>), dim3(persistent_grid(na, ntask)), dim3(256), 0, st, cd, tasks, ntask,
                           launch_queue(cd, it, mode, NC == 2), ws, na, it, mode);
    else if (it < NS64_TAIL_IT)
        hipLaunchKernelGGL((k_ns64<T, NC>), dim3(ntask), dim3(256), 0, st, cd, tasks, ws, na, it, mode);
    else if (it < NS64_REST_IT || !rest_chunk(na, ntask))
        hipLaunchKernelGGL((k_ns64_tail<T, NC>), dim3(scan_grid(na.pgrid, ntask)), dim3(256), 0, st, cd, tasks, ntask, ws,
                           na, it, mode);
    else if (it == NS64_REST_IT && mode == 1)
        hipLaunchKernelGGL((k_ns64_rest<T, NC>), dim3(scan_grid(na.pgrid, ntask)), dim3(256), 0, st, cd, tasks, ntask, ws,
                           na, it);
}
template <typename T>
static void launch_64(const ChunkDev &cd, char *ws, const NsArgs &na, int it, int mode, hipStream_t st) {
    launch_64<T, 4>(cd, cd.t_ns, cd.n_ns, ws, na, it, mode, st);
    launch_64<T, 2>(cd, cd.t_ns64, cd.n_ns64, ws, na, it, mode, st);
}

hipError_t launch_ns_iter(const ChunkDev &cd, char *ws, const NsArgs &na, int it, hipStream_t st) {
    for (int mode = 1; mode <= 2; ++mode) {
        switch (na.prec) {
            case NOLSM_FP64: launch_64<double>(cd, ws, na, it, mode, st); break;
            case NOLSM_FP32: launch_64<float>(cd, ws, na, it, mode, st); break;
            case NOLSM_FP16:
                if (na.sym) launch_lp<_Float16, true>(cd, ws, na, it, mode, st);
                else launch_lp<_Float16, false>(cd, ws, na, it, mode, st);
                break;
            default:
                if (na.sym) launch_lp<__bf16, true>(cd, ws, na, it, mode, st);
                else launch_lp<__bf16, false>(cd, ws, na, it, mode, st);
                break;
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// launches that max_iter iterations of a chunk take (of each of its tile sizes)
int ns_launches(const ChunkDev &cd, const NsArgs &na) {
    const bool lp = na.prec == NOLSM_FP16 || na.prec == NOLSM_BF16;
    const int rest = lp ? NS_REST_IT : NS64_REST_IT;
    const bool one = !na.persistent && rest_chunk(na, cd.n_ns) && rest_chunk(na, cd.n_ns64);
    return one && na.max_iter > rest ? 2 * rest + 1 : 2 * na.max_iter;
}

// symmetric route, after the last iteration: the returned iterates whole
hipError_t launch_ns_mirror(const ChunkDev &cd, char *ws, hipStream_t st) {
    if (cd.n_ns > 0) hipLaunchKernelGGL(k_ns_mirror, dim3(cd.n_ns), dim3(256), 0, st, cd, ws);
    return hipGetLastError();
}
