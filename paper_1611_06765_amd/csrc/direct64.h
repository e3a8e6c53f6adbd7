// Device code shared by the neutron and the isospin sweeps: descriptors in scalar
// registers and the FP64 product item of chi_klij.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ccd_internal.h"

namespace ccd {

// A descriptor that is the same in every lane, in scalar registers.  A kernel that
// loops over work items and stores in between cannot load it there by itself, and
// then carries every field and address in vector registers.  The tables do not change
// while a kernel runs, so it is read as constant memory, by scalar loads: a launch of
// many small items is bound by the chain item -> channel -> group (vector loads of all
// their words with a readfirstlane each, then scalar ones, us: k_update over a thousand
// boxes of N=14, n^2<=4 147 -> 115, over 64 twists at N=66, n^2<=20 223 -> 201, their
// product items 150 -> 141, ladders 262 -> 254).
template <typename T>
__device__ __forceinline__ T uni(const T& v) {
    static_assert(sizeof(T) % 4 == 0, "whole words");
    struct Words { int32_t w[sizeof(T) / 4]; };
    using Constant = const __attribute__((address_space(4))) int32_t;
    Constant* p = (Constant*)(uintptr_t)&v;
    Words x;
#pragma unroll
    for (size_t k = 0; k < sizeof(T) / 4; k++) x.w[k] = __builtin_amdgcn_readfirstlane(p[k]);
    return __builtin_bit_cast(T, x);
}

typedef double dbl4 __attribute__((ext_vector_type(4)));

// a product item: rows k0 .. k1 of an amplitude-shaped block ([n_pp][n_hh], row
// major) of <ab||ij> and of t
struct DirItem {
    const double* t;
    const double* vt;
    double* rows;   // row sums of the channel
    double* part;   // the item's part of chi_klij, [n_hh][n_hh]
    double* colp;   // and of the column sums, [n_hh]
    int nhh, k0, k1;
};
// D = A B + C for 16x16x4 FP64 tiles (lane l: A[l%16][l/16], B[l/16][l%16], D[l/16 + 4r][l%16])
__device__ __forceinline__ dbl4 mfma_d(double a, double b, dbl4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// The item on NW waves (8 or 16).  A chunk of whole rows (all 256 of an item where
// n_hh <= 16) is one contiguous run of memory, at most 8 (4) doubles of each operand per
// thread, loaded one chunk ahead of the work and kept in LDS as it is, with row stride
// n_hh: a product tile that reads past a row's end gets the next row's numbers,
// which reach only outputs outside the block.  With at most four 16x16 output
// tiles (n_hh <= 32) every wave computes all tiles over every NW-th 4-row K step;
// with more, the waves split into four groups, each of tiles g, g + 4, ..., and
// share the K steps inside a group.  The partial tiles are added in LDS in a fixed
// order.  The item is a chain of loads, barriers and short MFMA runs, so it is bound
// by latency: few and large chunks, eight waves and four threads per row sum shorten
// that chain.
//
// CH: doubles of each operand staged at a time, a chunk or half of one.  On eight waves
// half a chunk keeps the kernel within 128 registers, with two blocks a compute unit:
// with whole chunks the launch of product items alone spills 21 of them (64 twists at
// N=66, n^2<=20 225 -> 147 us, forty densities 145 -> 99, one density at n^2<=36 26 ->
// 27).  The K steps are shared out by whole chunks in both, so the bits are the same.
constexpr int kDirChunk = 4096;
constexpr int kDirHalf = kDirChunk / 2;
// two operands, each with the last tile's overhang
constexpr size_t dir64_lds(int staged) { return 2 * (size_t)(staged + 64) * 8; }
template <int NW, int CH = kDirChunk>
__device__ __forceinline__ void direct64(const DirItem& it, bool rowsums, bool quad, double* lds) {
    double* vs = lds;
    double* ts = lds + CH + 64;
    constexpr int TH = 64 * NW, NK = NW / 4;  // NK: waves of a group with more than four tiles
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int nhh = it.nhh, nt = (nhh + 15) >> 4, ntt = nt * nt;
    const int crows = min(kDirSplit, (kDirChunk / nhh) & ~3);  // rows of a chunk, in which the K steps are shared out
    const int srows = CH == kDirChunk ? crows : min(crows, (CH / nhh) & ~3);  // and rows staged at a time
    const bool split = ntt <= 4;
    constexpr int kPer = CH / TH;
    double vr[kPer] = {}, tr[kPer] = {};
    // the staged rows from r0 on end with the chunk (that of c0) or the item
    auto rows_at = [&](int r0, int c0) { return min(min(srows, c0 + crows - r0), it.k1 - r0); };
    auto load_chunk = [&](int r0, int rc) {
        const int ne = rc * nhh;
        const double* vp = it.vt + (int64_t)r0 * nhh;
        const double* tp = it.t + (int64_t)r0 * nhh;
#pragma unroll
        for (int i = 0; i < kPer; i++)
            if (TH * i < ne) {
                const int e = min(tid + TH * i, ne - 1);
                vr[i] = vp[e];
                tr[i] = tp[e];
            }
    };
    int c0 = it.k0, rc = rows_at(it.k0, it.k0);
    load_chunk(it.k0, rc);
    dbl4 acc[4];
#pragma unroll
    for (int k = 0; k < 4; k++) acc[k] = dbl4{0, 0, 0, 0};
    for (int r0 = it.k0; r0 < it.k1;) {
        const int rpad = (rc + 3) & ~3, ne = rc * nhh;
        __syncthreads();  // the previous chunk's (or item's) reads are done
#pragma unroll
        for (int i = 0; i < kPer; i++)
            if (TH * i < rpad * nhh) {  // zero in the rows up to the K step
                const int e = tid + TH * i;
                vs[e] = e < ne ? vr[i] : 0.0;
                ts[e] = e < ne ? tr[i] : 0.0;
            }
        __syncthreads();
        const int off = CH == kDirChunk ? 0 : (r0 - c0) >> 2;  // K steps of the chunk before these rows
        const int rn = r0 + rc, rows = rc;
        if (rn == c0 + crows) c0 = rn;
        rc = rows_at(rn, c0);
        if (rn < it.k1) load_chunk(rn, rc);
        // row sums of t v (one-body particle terms): four threads per row
        if (rowsums) {
            for (int x = tid; x < 4 * rows; x += TH) {
                const int o = (x >> 2) * nhh;
                double sum = 0.0;
#pragma unroll 2
                for (int j = x & 3; j < nhh; j += 4) sum += ts[o + j] * vs[o + j];
                sum += __shfl_xor(sum, 1);
                sum += __shfl_xor(sum, 2);
                if ((x & 3) == 0) it.rows[r0 + (x >> 2)] = sum;
            }
        }
        if (quad) {
            const int col = lane & 15, rq = lane >> 4;
            if (nt == 1) {
#pragma unroll 2
                for (int kk = 4 * ((w - off) & (NW - 1)); kk < rpad; kk += 4 * NW) {
                    const int o = (kk + rq) * nhh + col;
                    acc[0] = mfma_d(vs[o], ts[o], acc[0]);
                }
            } else if (split) {
#pragma unroll 2
                for (int kk = 4 * ((w - off) & (NW - 1)); kk < rpad; kk += 4 * NW) {
                    const int o = (kk + rq) * nhh + col;
                    const double a0 = vs[o], b0 = ts[o], a1 = vs[o + 16], b1 = ts[o + 16];
                    acc[0] = mfma_d(a0, b0, acc[0]);
                    acc[1] = mfma_d(a0, b1, acc[1]);
                    acc[2] = mfma_d(a1, b0, acc[2]);
                    acc[3] = mfma_d(a1, b1, acc[3]);
                }
            } else {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int tile = w / NK + 4 * k;
                    if (tile < ntt) {
                        const double* vp = vs + rq * nhh + col + 16 * (tile / nt);
                        const double* tp = ts + rq * nhh + col + 16 * (tile % nt);
#pragma unroll 2
                        for (int kk = 4 * ((w - off) & (NK - 1)); kk < rpad; kk += 4 * NK)
                            acc[k] = mfma_d(vp[kk * nhh], tp[kk * nhh], acc[k]);
                    }
                }
            }
        }
        r0 = rn;
    }
    if (!quad) return;
    // add the waves' partial tiles: with sixteen waves the upper half of a tile's
    // first to the lower half, then the rest in wave order
    dbl4* red = (dbl4*)lds;  // [tile][wave of the tile][64], at most 32 entries
    auto put = [&](const dbl4& sum, int ti, int tj) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int kl = ti * 16 + (lane >> 4) + 4 * q, ij = tj * 16 + (lane & 15);
            if (kl < nhh && ij < nhh) {
                it.part[kl * nhh + ij] = sum[q];
                if (kl == ij) it.colp[kl] = sum[q];
            }
        }
    };
    auto in_order = [&](const dbl4* p) {  // the eight waves' tiles
        dbl4 sum = p[0];
#pragma unroll 1
        for (int q = 1; q < 8; q++) sum += p[q * 64];
        return sum;
    };
    if constexpr (CH != kDirChunk) {  // less LDS: a tile, or a tile of each group, at a time
        static_assert(NW == 8, "eight shares of a tile, or two");
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int tile = split ? k : w / NK + 4 * k;
            if (split ? k >= ntt : 4 * k >= ntt) break;
            __syncthreads();
            if (split) red[w * 64 + lane] = acc[k];
            else if (tile < ntt && w % NK == 1) red[(w / NK) * 64 + lane] = acc[k];
            __syncthreads();
            if (split && w == k) put(in_order(red + lane), k / nt, k % nt);
            if (!split && tile < ntt && w % NK == 0) put(acc[k] + red[(w / NK) * 64 + lane], tile / nt, tile % nt);
        }
        return;
    }
    const int ki = split ? w : w % NK;                 // this wave's place among its tiles' waves
    const int nk = split ? 8 : 2;                      // places left when the sums are put together
    const int nown = split ? ntt : 4;
    auto tile_of = [&](int k) { return split ? k : w / NK + 4 * k; };
    __syncthreads();
    if (NW == 16) {
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (k < nown && tile_of(k) < ntt && ki >= nk) red[(tile_of(k) * nk + ki - nk) * 64 + lane] = acc[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (k < nown && tile_of(k) < ntt && ki < nk) acc[k] += red[(tile_of(k) * nk + ki) * 64 + lane];
        __syncthreads();
    }
    if (split) {
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (k < ntt && ki < 8) red[(k * 8 + w) * 64 + lane] = acc[k];
        __syncthreads();
        if (w < ntt) put(in_order(red + w * 8 * 64 + lane), w / nt, w % nt);
    } else {
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (tile_of(k) < ntt && ki == 1) red[tile_of(k) * 64 + lane] = acc[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (tile_of(k) < ntt && ki == 0) put(acc[k] + red[tile_of(k) * 64 + lane], tile_of(k) / nt, tile_of(k) % nt);
    }
}

}  // namespace ccd
