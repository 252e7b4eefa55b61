// Device helpers shared by the kernel sources: complex arithmetic, the in-LDS Stockham FFT
// with its twiddle staging, the column-pass helpers and the bilinear sample of the sky.
#pragma once

#include "ivx_internal.hpp"

#include <math.h>

namespace ivx {

constexpr int NT = 256; // threads per block of every kernel

__device__ __forceinline__ cpx cmul(cpx a, cpx b) {
    return cpx{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ cpx cadd(cpx a, cpx b) { return cpx{a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cpx csub(cpx a, cpx b) { return cpx{a.re - b.re, a.im - b.im}; }

// ------------------------------------------------------------------------------ FFT
// In-LDS Stockham autosort FFT of CB transforms of length N = 2^LOGN in place: element i of
// transform c is buf[Fft<LOGN, CB, PAIR>::at(i, c)].  The stages are radix 2 first when LOGN is odd, then
// radix 4.  Each reads all of a thread's inputs into registers, synchronises, then writes the
// outputs.  Twiddles come from a table tw[t] = exp(-2 pi i t / N), t < 3N/4, staged in LDS through
// TwStage (conjugated for the inverse); no scaling is applied in either direction.
//
// PAIR runs the stages two at a time in registers, 16 (or 8) points a thread, so that a 1024-point
// transform passes through LDS three times instead of five, at a quarter of the threads.  Both forms
// do the same operations on the same values.  Each kernel takes the one that measured faster (single :
// paired, us, 36 images of 1024-point columns unless stated):
//   forward columns 91 : 80, inverse rows 34 : 30, plane passes of the full model 315 : 292 together
//   image rows 44.6 : 47.2 (cube of 128 channels 4,240 : 4,540); at 2048 points 13.9 : 12.0
//   fold + inverse columns 198 : 207 (cube 19,150 : 20,400): bound by its slot loads, whose
//   threads a paired stage leaves idle
//   one column a block of one 1024-point image: the same; of the double build 27.3 : 24.6
// Below 1024 points a block pairing leaves less than a wave at work (4 of the 70 us of a 64^2 field).
template <int LOGN> constexpr int tw_len() { return 3 * (1 << LOGN) / 4; }

// The twiddle table is fetched into registers at the start of a kernel and stored to LDS
// only after the kernel's own data loads have been issued, so the two global-memory
// latencies overlap instead of following each other.
template <int LOGN> struct TwStage {
    static constexpr int PER = (tw_len<LOGN>() + NT - 1) / NT;
    cpx v[PER];
    __device__ __forceinline__ void fetch(const cpx *__restrict__ tw) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = threadIdx.x + u * NT;
            if (i < tw_len<LOGN>()) v[u] = tw[i];
        }
    }
    __device__ __forceinline__ void store(cpx *tws) const {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = threadIdx.x + u * NT;
            if (i < tw_len<LOGN>()) tws[i] = v[u];
        }
    }
};

// Paired stages: the low four bits of an index are xored with the next four, since the outputs
// of a 16-point thread at the first stages are 16 elements apart from lane to lane, which without it
// meet in one bank.  Transforms are N + 16 apart, so that lanes that walk c and lanes that walk i
// both spread over the banks.  Single stages: transforms interleaved.
__device__ __forceinline__ int fft_swz(int i) { return i ^ ((i >> 4) & 15); }
template <int LOGN, int CB> constexpr int fft_ld() { return CB > 1 ? (1 << LOGN) + 16 : 1 << LOGN; }

// (a0, a1, a2, a3) -> their 4-point transform in place
template <bool INV> __device__ __forceinline__ void radix4(cpx &a0, cpx &a1, cpx &a2, cpx &a3) {
    const cpx s02 = cadd(a0, a2), d02 = csub(a0, a2);
    const cpx s13 = cadd(a1, a3), d13 = csub(a1, a3);
    // forward: y1 = d02 - i d13, y3 = d02 + i d13; inverse swaps the signs
    const cpx id13 = INV ? cpx{-d13.im, d13.re} : cpx{d13.im, -d13.re};
    a0 = cadd(s02, s13);
    a1 = cadd(d02, id13);
    a2 = csub(s02, s13);
    a3 = csub(d02, id13);
}

// A radix-RA stage at stride NS and, if TWO, the radix-4 stage after it.  A thread's R points are
// positions jj + r N / R: the RA points of first-stage butterfly q are r = q + 4 r', and output s of
// the four butterflies are the inputs of one second-stage butterfly.
template <int LOGN, int CB, bool INV, int NS, int RA, bool TWO>
__device__ __forceinline__ void fft_pass(cpx *buf, const cpx *tw) {
    constexpr int N = 1 << LOGN, NB = TWO ? 4 : 1, R = RA * NB, S = N / R, TOT = CB * S, BPT = (TOT + NT - 1) / NT;
    cpx v[BPT][R];
#pragma unroll
    for (int t = 0; t < BPT; ++t) {
        const int u = threadIdx.x + t * NT;
        if (TOT % NT != 0 && u >= TOT) break;
        const int c = u / S, jj = u & (S - 1), k = jj & (NS - 1);
        const cpx *b = buf + c * fft_ld<LOGN, CB>();
        const int sj = fft_swz(jj);
#pragma unroll
        for (int r = 0; r < R; ++r) // (S a multiple of 16: jj >> 4 and r S / 16 have no bit in common)
            v[t][r] = b[S % 16 == 0 ? (sj ^ ((r * (S / 16)) & 15)) + r * S : fft_swz(jj + r * S)];
        auto twiddle = [&](cpx x, int at) {
            cpx w = tw[at];
            if (INV) w.im = -w.im;
            return cmul(x, w);
        };
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            if (NS > 1)
#pragma unroll
                for (int r = 1; r < RA; ++r) v[t][q + NB * r] = twiddle(v[t][q + NB * r], k * r * (N / (RA * NS)));
            if constexpr (RA == 2) {
                const cpx a = v[t][q], d = v[t][q + NB];
                v[t][q] = cadd(a, d);
                v[t][q + NB] = csub(a, d);
            } else {
                radix4<INV>(v[t][q], v[t][q + NB], v[t][q + 2 * NB], v[t][q + 3 * NB]);
            }
        }
        if constexpr (TWO) {
#pragma unroll
            for (int s = 0; s < RA; ++s) {
#pragma unroll
                for (int q = 1; q < 4; ++q)
                    if (NS > 1 || s > 0) v[t][q + 4 * s] = twiddle(v[t][q + 4 * s], (k + s * NS) * q * (N / (R * NS)));
                radix4<INV>(v[t][4 * s], v[t][4 * s + 1], v[t][4 * s + 2], v[t][4 * s + 3]);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < BPT; ++t) {
        const int u = threadIdx.x + t * NT;
        if (TOT % NT != 0 && u >= TOT) break;
        const int c = u / S, jj = u & (S - 1), k = jj & (NS - 1);
        cpx *b = buf + c * fft_ld<LOGN, CB>();
        const int o = R * (jj - k) + k, so = fft_swz(o);
#pragma unroll
        for (int p = 0; p < NB; ++p)
#pragma unroll
            for (int s = 0; s < RA; ++s) {
                // output e is element o + e NS; its two parts have no bit in common
                const int e = s + p * RA, d = e * NS;
                const bool split = NS % 16 == 0 || NS == 1 || NS == 8;
                b[split ? (so ^ (d & 15) ^ ((d >> 4) & 15)) + (d & ~15) : fft_swz(o + d)] = v[t][TWO ? p + 4 * s : s];
            }
    }
    __syncthreads();
}

template <int LOGN, int CB, bool INV, int NS = 1> __device__ __forceinline__ void fft_paired(cpx *buf, const cpx *tw) {
    constexpr int N = 1 << LOGN;
    if constexpr (NS == 1 && (LOGN & 1)) {
        fft_pass<LOGN, CB, INV, NS, 2, true>(buf, tw);
        fft_paired<LOGN, CB, INV, 8>(buf, tw);
    } else if constexpr (N / NS >= 16) {
        fft_pass<LOGN, CB, INV, NS, 4, true>(buf, tw);
        fft_paired<LOGN, CB, INV, 16 * NS>(buf, tw);
    } else if constexpr (N / NS >= 4) {
        fft_pass<LOGN, CB, INV, NS, 4, false>(buf, tw);
        fft_paired<LOGN, CB, INV, 4 * NS>(buf, tw);
    }
}

template <int LOGN, int CB, bool INV> __device__ __forceinline__ void fft_single(cpx *buf, const cpx *tw) {
    constexpr int N = 1 << LOGN;
    const int tid = threadIdx.x;
    int Ns = 1;
    if constexpr (LOGN & 1) {
        constexpr int TOT = CB * (N / 2);
        constexpr int BPT = (TOT + NT - 1) / NT;
        cpx v0[BPT], v1[BPT];
#pragma unroll
        for (int t = 0; t < BPT; ++t) {
            const int u = tid + t * NT;
            if (u < TOT) {
                const int c = u % CB, jj = u / CB;
                v0[t] = buf[jj * CB + c];
                v1[t] = buf[(jj + N / 2) * CB + c];
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < BPT; ++t) {
            const int u = tid + t * NT;
            if (u < TOT) {
                const int c = u % CB, jj = u / CB;
                buf[(2 * jj) * CB + c] = cadd(v0[t], v1[t]);
                buf[(2 * jj + 1) * CB + c] = csub(v0[t], v1[t]);
            }
        }
        __syncthreads();
        Ns = 2;
    }
#pragma unroll
    for (int s = 0; s < LOGN / 2; ++s) {
        constexpr int TOT = CB * (N / 4);
        constexpr int BPT = (TOT + NT - 1) / NT;
        cpx v[BPT][4];
        const int st = N / (4 * Ns);
#pragma unroll
        for (int t = 0; t < BPT; ++t) {
            const int u = tid + t * NT;
            if (u < TOT) {
                const int c = u % CB, jj = u / CB;
                const int k = jj & (Ns - 1);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    cpx x = buf[(jj + r * (N / 4)) * CB + c];
                    if (r > 0) {
                        cpx w = tw[k * r * st];
                        if (INV) w.im = -w.im;
                        x = cmul(x, w);
                    }
                    v[t][r] = x;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < BPT; ++t) {
            const int u = tid + t * NT;
            if (u < TOT) {
                const int c = u % CB, jj = u / CB;
                const int k = jj & (Ns - 1);
                radix4<INV>(v[t][0], v[t][1], v[t][2], v[t][3]);
                const int o = ((jj - k) << 2) + k;
#pragma unroll
                for (int r = 0; r < 4; ++r) buf[(o + r * Ns) * CB + c] = v[t][r];
            }
        }
        __syncthreads();
        Ns *= 4;
    }
}

template <int LOGN, int CB, bool PAIR> struct Fft {
    static constexpr int LEN = PAIR ? CB * fft_ld<LOGN, CB>() : CB << LOGN;
    static __device__ __forceinline__ int at(int i, int c = 0) {
        return PAIR ? c * fft_ld<LOGN, CB>() + fft_swz(i) : i * CB + c;
    }
    static __device__ __forceinline__ void forward(cpx *buf, const cpx *tw) {
        if constexpr (PAIR) fft_paired<LOGN, CB, false>(buf, tw);
        else fft_single<LOGN, CB, false>(buf, tw);
    }
    static __device__ __forceinline__ void inverse(cpx *buf, const cpx *tw) {
        if constexpr (PAIR) fft_paired<LOGN, CB, true>(buf, tw);
        else fft_single<LOGN, CB, true>(buf, tw);
    }
};
template <int LOGN> using RowFft = Fft<LOGN, 1, (LOGN >= 10)>;
// (a block of one column pairs from 16 KB of it on)
template <int LOGN, int CB>
using ColFft = Fft<LOGN, CB, (CB << LOGN) >= 1024 && (CB > 1 || sizeof(cpx) << LOGN >= 16384)>;

// Global loads each thread of a column pass issues before it waits for the first: with a few
// blocks of LDS-resident columns per compute unit, one load at a time leaves the latency of
// every row exposed.
constexpr int COL_LOADS = 8;

// Columns per block of a column pass: at most 32 KB of LDS columns, so that four blocks share
// a compute unit (at 1024-point columns 4 per block measured faster than 8 and 2).
// Work index of a column-pass block.  Blocks are dealt to the eight XCDs round-robin by
// launch index; block b takes work index (b % 8) * per + b / 8 of the (item, column group)
// pairs, so each XCD runs one contiguous range of them and neighbouring column groups, which
// share the cache lines of their row segments, meet in the same L2.  The launch has
// 8 * per blocks; false for the padding blocks past the last pair.
template <int CB> __device__ __forceinline__ bool col_block(const Geom &g, int &item, int &c0) {
    const int64_t ngrp = (g.rw + CB - 1) / CB, total = ngrp * g.C * g.P, per = (total + 7) / 8;
    const int64_t b = blockIdx.x, w = (b & 7) * per + (b >> 3);
    if (w >= total) return false;
    item = (int)(w / ngrp);
    c0 = (int)(w - (w / ngrp) * ngrp) * CB;
    return true;
}

template <int LOGN> constexpr int col_batch() {
    constexpr int b = 32768 / ((1 << LOGN) * (int)sizeof(cpx));
    return b > 16 ? 16 : (b < 1 ? 1 : b);
}

// --------------------------------------------------------------------- reprojection
// Bilinear sample at (row sy, col sx); pixel (i, j) sits at (i, j); outside pixels are 0.
// Branch-free: a tap outside the image reads a clamped pixel inside it and is scaled by 0, and
// a sample outside (or a NaN coordinate) evaluates at (0, 0) and is scaled by 0, so the loads
// of several samples can be in flight together (behind a branch each would wait for the last).
// Taps: the four pixel offsets (row-major, N^2 < 2^31) and their 0/1 masks; combine() forms
// the sample from the four loaded pixels.
struct BilinearTaps {
    int o[4];
    real m[4];
    real fy, fx, in;
    __device__ __forceinline__ real combine(real p00, real p01, real p10, real p11) const {
        const real x00 = p00 * m[0], x01 = p01 * m[1], x10 = p10 * m[2], x11 = p11 * m[3];
        const real v = (real(1) - fy) * ((real(1) - fx) * x00 + fx * x01) + fy * ((real(1) - fx) * x10 + fx * x11);
        return v * in;
    }
};

__device__ __forceinline__ BilinearTaps bilinear_taps(int N, real sy, real sx) {
    BilinearTaps t;
    const bool in = sy > real(-1) && sy < real(N) && sx > real(-1) && sx < real(N);
    const real cy = in ? sy : real(0), cx = in ? sx : real(0);
    const real fi = floor(cy), fj = floor(cx);
    const int i0 = (int)fi, j0 = (int)fj;
    t.fy = cy - fi;
    t.fx = cx - fj;
    t.in = in ? real(1) : real(0);
    const bool r0 = i0 >= 0, r1 = i0 + 1 < N, c0 = j0 >= 0, c1 = j0 + 1 < N;
    const int ia = (r0 ? i0 : 0) * N, ib = (r1 ? i0 + 1 : N - 1) * N;
    const int ja = c0 ? j0 : 0, jb = c1 ? j0 + 1 : N - 1;
    t.o[0] = ia + ja;
    t.o[1] = ia + jb;
    t.o[2] = ib + ja;
    t.o[3] = ib + jb;
    t.m[0] = (r0 && c0) ? real(1) : real(0);
    t.m[1] = (r0 && c1) ? real(1) : real(0);
    t.m[2] = (r1 && c0) ? real(1) : real(0);
    t.m[3] = (r1 && c1) ? real(1) : real(0);
    return t;
}

__device__ __forceinline__ real bilinear(const real *__restrict__ sky, int N, real sy, real sx) {
    const BilinearTaps t = bilinear_taps(N, sy, sx);
    return t.combine(sky[t.o[0]], sky[t.o[1]], sky[t.o[2]], sky[t.o[3]]);
}

} // namespace ivx
