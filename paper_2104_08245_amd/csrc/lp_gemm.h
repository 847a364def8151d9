// FP16 / BF16 tile products on v_mfma_f32_32x32x16_{f16,bf16} with FP32
// accumulation, shared by the Newton-Schulz sign iteration and the coupled
// Newton-Schulz inverse. Operands are row-major ldx x ldx 16-bit matrices in
// the workspace with ldx >= every tile extent (so loads need no masking) and
// the contraction runs over k < np (np a multiple of 64).
#pragma once
#include "dev_common.h"

template <typename T> struct Lp;
template <> struct Lp<_Float16> {
    typedef v8h vec;
    static __device__ __forceinline__ v16f mma(vec a, vec b, v16f c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint16_t enc(float x) {
        _Float16 h = (_Float16)x;
        return __builtin_bit_cast(uint16_t, h);
    }
    static __device__ __forceinline__ float dec(uint16_t x) { return (float)__builtin_bit_cast(_Float16, x); }
};
template <> struct Lp<__bf16> {
    typedef v8bf vec;
    static __device__ __forceinline__ v16f mma(vec a, vec b, v16f c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint16_t enc(float x) {
        __bf16 h = (__bf16)x;
        return __builtin_bit_cast(uint16_t, h);
    }
    static __device__ __forceinline__ float dec(uint16_t x) { return (float)__builtin_bit_cast(__bf16, x); }
};

// A product or sum rounded once to the 16-bit type (FP16: v_fma_mixlo_f16,
// without a rounding to FP32 in between). The value is kept to itself, or
// the compiler would round two of them to FP32 and convert the pair.
__device__ __forceinline__ uint16_t alone(uint16_t x) {
    asm volatile("" : "+v"(x));
    return x;
}
template <typename T> __device__ __forceinline__ uint16_t enc_update(uint16_t x, float acc) {   // x + acc / 2
    return alone(Lp<T>::enc(Lp<T>::dec(x) + 0.5f * acc));
}
template <typename T> __device__ __forceinline__ uint16_t enc_scaled(float c, float acc) {
    return alone(Lp<T>::enc(c * acc));
}
// four 16-bit values as two words
__device__ __forceinline__ uint2 pack4(const uint16_t (&h)[4]) {
    return make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
}

#define LBK 64

// LDS tiles hold 64 k per row (128 bytes, no padding). The 16-byte chunk c
// (8 consecutive k) of row n sits at chunk position c ^ ((n ^ n >> 3) & 7):
// an MFMA operand read (32 rows, one chunk) then touches 8 distinct chunk
// positions in every 8 consecutive rows, and the transposing B stores (one
// row per 8 columns) spread over all positions as well.
__device__ __forceinline__ int lds_swz(int n, int c) { return n * LBK + ((c ^ ((n ^ (n >> 3)) & 7)) << 3); }

// The two operand tiles of lp_tile_product (BM x LBK 16-bit values each),
// one allocation per kernel; free again when lp_tile_product returns, so an
// epilogue may stage through them.
template <int BM> __device__ __forceinline__ uint16_t *lp_lds() {
    __shared__ __attribute__((aligned(16))) uint16_t buf[2 * BM * LBK];
    return buf;
}

// ---------------------------------------------------------------------------
// BM x BM tile (ti, tj) of A B (BM = 128: each of the 4 waves 64x64 as 2x2
// 32x32 MFMA blocks; BM = 64: one 32x32 block per wave), K in slices of 64.
// Both operands sit in LDS as [row of A or column of B][k], so that an MFMA
// operand is one 16-byte read of 8 consecutive k.
//
// General matrices: A's rows come as they stand, B's k rows are read
// transposed: 4 (k) x 8 blocks per thread, turned on their way into LDS.
// SYM: A and B are symmetric and commute, and only tiles ti <= tj are formed.
// With 128-row tiles the operands are stored by their upper tiles (the
// diagonal tiles whole): row block ti of A at the k's of tile row kb is the
// stored tile (ti, kb) as it stands where kb >= ti, and the transpose of the
// stored tile (kb, ti) where kb < ti; row block tj of B (B[k][n] = B[n][k])
// likewise. Storing one triangle takes 0.6 of the memory traffic at 5 x 5
// tiles. 64-row tiles serve submatrices of one to three of them, which stay
// in the caches: there both triangles are stored and nothing is turned.
//
// acc[i][j] holds the transposed MFMA block (operands swapped, the same
// products in the same order): element e of the calling lane is tile row
// wm WT + i 32 + l % 32 and column wn WT + j 32 + (e / 4) 8 + (l / 32) 4 +
// e % 4 (w = wave = 2 wm + wn, l = lane, WT = BM / 2), so four elements in
// turn are consecutive columns of one row. Waves whose part of the tile is
// padding, or lies below the diagonal of a diagonal tile (SYM), load and
// store with the others but do not multiply.
// ---------------------------------------------------------------------------
// an output tile in LDS (the operand buffers, free after the product): rows
// of BM values, 16-byte chunks swizzled by row
template <int BM> __device__ __forceinline__ int tile_idx(int r, int c) {
    return r * BM + (((c >> 3) ^ (r & (BM / 8 - 1))) << 3) + (c & 7);
}

// 16 bytes, past the caches (nt) where an output is read again only a whole
// pass over a large chunk later: kept out of L2 it does not displace the
// operand tiles that the workgroups beside it share
__device__ __forceinline__ void store16(uint16_t *p, const uint4 &v, bool nt) {
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    const v4u x = {v.x, v.y, v.z, v.w};
    if (nt) __builtin_nontemporal_store(x, (v4u *)p);
    else *(v4u *)p = x;
}
// tile (ti, tj) from its LDS copy, the rows and columns below np
template <int BM> __device__ __forceinline__ void tile_store(uint16_t *X, int ldx, int np, int ti, int tj, bool nt) {
    constexpr int NCH = BM / 8;
    const uint16_t *st = lp_lds<BM>();
    const int row0 = ti * BM, col0 = tj * BM;
#pragma unroll 4
    for (int f = threadIdx.x; f < BM * NCH; f += 256) {
        const int r = f / NCH, c0 = (f % NCH) * 8;
        if (row0 + r >= np || col0 + c0 >= np) continue;
        store16(X + (int64_t)(row0 + r) * ldx + col0 + c0, *(const uint4 *)(st + tile_idx<BM>(r, c0)), nt);
    }
}
// every launch of more tiles than run at once (three workgroups per CU, pgrid
// being two): its outputs leave the caches before the next launch reads them
__host__ __device__ __forceinline__ bool lp_nt_out(int ntask, int pgrid) { return ntask > pgrid + pgrid / 2; }

template <int BM, bool SYM> __device__ __forceinline__ bool lp_live(int np, int ti, int tj) {
    constexpr int WT = BM / 2;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w >> 1, wn = w & 1;
    return ti * BM + wm * WT < np && tj * BM + wn * WT < np && !(SYM && ti == tj && wm > wn);
}

// `begin` runs between the issue of the first slice's loads and their use
// (all 256 threads; false: stop here). pre: issue them; a wave may clear it
// only if `begin` is going to stop. Eg: a matrix whose tile (ti, tj) is
// fetched behind the last slice and left in LDS in tile_idx order, or null.
// `finish` takes the accumulators of the waves that multiply (the others run
// a loop of their own, without products: a branch inside one loop would have
// the accumulators copied).
template <typename T, int BM, bool SYM, typename Begin, typename Finish>
__device__ __forceinline__ bool lp_tile_product(const uint16_t *Ag, const uint16_t *Bg, const uint16_t *Eg, int ldx,
                                               int np, int ti, int tj, bool pre, Begin begin, Finish finish) {
    typedef typename Lp<T>::vec vec;
    constexpr int WT = BM / 2, NB = WT / 32;
    constexpr bool UP = SYM && BM == 128;   // stored by upper tiles
    uint16_t *lds = lp_lds<BM>();
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63, wm = w >> 1, wn = w & 1;
    const bool same = SYM && Ag == Bg && ti == tj;   // one operand tile serves both sides
    const bool live = lp_live<BM, SYM>(np, ti, tj);
    const uint32_t none = 0x80000000u;        // beyond any buffer: zeros, no memory access
    const int nrec = ldx * ldx * 2, srow = 2 * ldx, nk = np / LBK;
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc((void *)Ag, (short)0, nrec, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc((void *)Bg, (short)0, nrec, 0x00020000);
    // as it stands: 16-byte chunk t % 8 of rows t / 8 + 32 q of the row block
    const int row0 = ti * BM, col0 = tj * BM;
    const uint32_t da = (uint32_t)((row0 + (t >> 3)) * srow + (t & 7) * 16);
    const uint32_t db = (uint32_t)((col0 + (t >> 3)) * srow + (t & 7) * 16);
    // transposed: k rows 4 kq + q, columns 8 nci .. + 7; each group of 16
    // lanes covers 8 column blocks and two k quads, so that its 8-byte LDS
    // stores land on 16 distinct 8-byte bank slots
    // (64-row tiles: half of the threads)
    const int nci = BM == 128 ? (t & 7) | (((t >> 4) & 1) << 3) : t & 7;
    const int kq = BM == 128 ? ((t >> 3) & 1) | ((t >> 5) << 1) : t >> 3;
    const int nc = nci * 8;
    const bool tl = BM == 128 || t < 128;
    const uint32_t ta = row0 + nc < np ? (uint32_t)(kq * 4 * srow + (row0 + nc) * 2) : none;
    const uint32_t tb = tl && col0 + nc < np ? (uint32_t)(kq * 4 * srow + (col0 + nc) * 2) : none;
    // the second half of a row block may be all padding (np is a multiple of 64)
    const bool a_hi = row0 + 64 < np, b_hi = col0 + 64 < np;
    constexpr int NQ = BM / 32, NB4 = SYM ? NQ : 4;   // 16-byte loads of A's and of B's slice per thread
    uint4 pf[NQ + NB4];                               // A's, then B's
    auto load = [](const __amdgpu_buffer_rsrc_t &rs, uint32_t vo, int so) {
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo, so, 0));
    };
    auto fetch = [&](int ks) {
        const int kb = ks * LBK / BM;
        const bool tra = UP && kb < ti, trb = !SYM || (UP && kb < tj);
        const int sa = tra ? srow : 32 * srow, sb = trb ? srow : 32 * srow;
        const uint32_t oa = tra ? (ta == none ? none : ta + (uint32_t)(ks * LBK * srow)) : da + (uint32_t)(ks * LBK * 2);
        const uint32_t ob = same ? none
                            : trb ? (tb == none ? none : tb + (uint32_t)(ks * LBK * srow))
                                  : db + (uint32_t)(ks * LBK * 2);
        const uint32_t oa2 = (tra || a_hi) ? oa : none, ob2 = (trb || b_hi) ? ob : none;
        pf[0] = load(rsA, oa, 0);
        pf[1] = load(rsA, oa, sa);
        if constexpr (NQ > 2) {
            pf[2] = load(rsA, oa2, 2 * sa);
            pf[3] = load(rsA, oa2, 3 * sa);
        }
        pf[NQ + 0] = load(rsB, ob, 0);
        pf[NQ + 1] = load(rsB, ob, sb);
        if constexpr (NB4 > 2) {
            pf[NQ + 2] = load(rsB, ob2, 2 * sb);
            pf[NQ + 3] = load(rsB, ob2, 3 * sb);
        }
    };
    // LDS byte offsets (the layout of lds_swz): the rows that a thread writes
    // or reads differ by multiples of 8, 32 or 64, which change its chunk
    // position only by an exclusive or with a constant
    const uint32_t wd = (uint32_t)lds_swz(t >> 3, t & 7) * 2, wt = (uint32_t)(lds_swz(nc, kq >> 1) + (kq & 1) * 4) * 2;
    const uint32_t ra = (uint32_t)lds_swz(wm * WT + (l & 31), l >> 5) * 2;
    const uint32_t rb = (uint32_t)(lds_swz(wn * WT + (l & 31), l >> 5) + (same ? 0 : BM * LBK)) * 2;
    char *const lb = (char *)lds;
    // one operand's slice into its LDS tile
    auto put = [&](char *s, const uint4 *p, bool tr) {
        if (!tr) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) *(uint4 *)(s + ((wd ^ ((q & 1) << 6)) + q * 32 * LBK * 2)) = p[q];
        } else if constexpr (UP || !SYM) {
            if (!tl) return;
            uint32_t o = wt;
            asm volatile("" : "+v"(o));   // the eight offsets are formed here, not kept through the loop
            auto col = [&](int j, uint32_t r0, uint32_t r1, uint32_t r2, uint32_t r3) {
                const uint32_t lo = (j & 1) ? (r0 >> 16) | (r1 & 0xFFFF0000u) : (r0 & 0xFFFFu) | (r1 << 16);
                const uint32_t hi = (j & 1) ? (r2 >> 16) | (r3 & 0xFFFF0000u) : (r2 & 0xFFFFu) | (r3 << 16);
                *(uint2 *)(s + ((o ^ (j << 4)) + j * LBK * 2)) = make_uint2(lo, hi);
            };
            col(0, p[0].x, p[1].x, p[2].x, p[3].x);
            col(1, p[0].x, p[1].x, p[2].x, p[3].x);
            col(2, p[0].y, p[1].y, p[2].y, p[3].y);
            col(3, p[0].y, p[1].y, p[2].y, p[3].y);
            col(4, p[0].z, p[1].z, p[2].z, p[3].z);
            col(5, p[0].z, p[1].z, p[2].z, p[3].z);
            col(6, p[0].w, p[1].w, p[2].w, p[3].w);
            col(7, p[0].w, p[1].w, p[2].w, p[3].w);
        }
    };
    auto stash = [&](int ks) {
        const int kb = ks * LBK / BM;
        put(lb, pf, UP && kb < ti);
        if (!same) put(lb + BM * LBK * 2, pf + NQ, !SYM || (UP && kb < tj));
    };
    // tile (ti, tj) of Eg: chunk f % (BM / 8) of row f / (BM / 8), f = t + 256 q
    const int er = t / (BM / 8), ec = t % (BM / 8);
    constexpr int EQ = BM * BM / 8 / 256, ES = 256 / (BM / 8);   // chunks per thread, rows between them
    // behind the products of slice kt: the loads of the next slice, or of Eg
    auto ahead = [&](int kt) {
        if (kt + 1 < nk) {
            fetch(kt + 1);
        } else if (Eg) {
            const __amdgpu_buffer_rsrc_t rsE = __builtin_amdgcn_make_buffer_rsrc((void *)Eg, (short)0, nrec, 0x00020000);
            const uint32_t oe = (uint32_t)((row0 + er) * srow + (col0 + ec * 8) * 2);
#pragma unroll
            for (int q = 0; q < EQ; ++q) pf[q] = load(rsE, oe, q * ES * srow);
        }
    };
    auto settle = [&](int kt) {
        __syncthreads();
        if (kt + 1 < nk) {
            stash(kt + 1);
        } else if (Eg) {
#pragma unroll
            for (int q = 0; q < EQ; ++q)
                *(uint4 *)&lds[tile_idx<BM>(er + q * ES, ec * 8)] = pf[q];
        }
        __syncthreads();
    };
    if (pre) fetch(0);
    if (!begin()) return false;
    stash(0);
    __syncthreads();
    if (!live) {
        for (int kt = 0; kt < nk; ++kt) {
            ahead(kt);
            settle(kt);
        }
        return true;
    }
    v16f acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    for (int kt = 0; kt < nk; ++kt) {
        ahead(kt);
        // the loads stay ahead of the products: otherwise the compiler sinks
        // them behind the MFMAs, next to their use, and every slice waits out
        // the full load latency
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < LBK; kk += 16) {
            vec a[NB], b[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i)
                a[i] = *(const vec *)(lb + ((ra ^ (((kk >> 3) ^ (4 * i)) << 4)) + i * 32 * LBK * 2));
#pragma unroll
            for (int j = 0; j < NB; ++j)
                b[j] = *(const vec *)(lb + ((rb ^ (((kk >> 3) ^ (4 * j)) << 4)) + j * 32 * LBK * 2));
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[i][j] = Lp<T>::mma(b[j], a[i], acc[i][j]);
        }
        settle(kt);
    }
    finish(acc);
    return true;
}
