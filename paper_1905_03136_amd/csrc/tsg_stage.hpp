// tsg_stage.hpp -- TSMTTSM on the matrix cores with the rows of A and B
// brought straight into LDS (tsmttsm_stage), for widths above 16.
//
// P = X^T Y for two tall matrices, X (K x MX) the wider one and Y (K x NY):
// the launcher gives A and B in that order and sets `swap` where X is B, so
// that C = P or C = P^T.  A block brings stages of RT rows of X and Y into
// LDS with direct loads (global_load_lds_dwordx4: 16 bytes a lane, no
// register holds the data), NS stages in turn, NS - 1 of them in flight while
// one is multiplied.  Wave w of the WM waves of a block owns MB blocks of 16
// columns of X against every column of Y: NB blocks of 16 (one
// v_mfma_f64_16x16x4f64 each and four rows) and NQ groups of 4
// (v_mfma_f64_4x4x4f64, a quarter of the time of a 16-wide block), so the
// padding is to 16 in X and to 4 in Y.  The widths are run-time values; the
// block counts are not.
//
// What bounds it: HBM for real widths and narrow complex ones, the FP64
// matrix cores for wide complex ones.  The register-ring kernels it replaced
// for these layouts were held back by three things.
//  * Their accumulators sat in accumulation registers, where a 16x16x4 product
//    takes 104 to 141 cycles, not 65 (see STAGE_FLAGS of the build).
//  * Every vector instruction costs matrix-core time (3 to 6 cycles each
//    beside a stream of products): row guards, address clamps and sign flips
//    were a fifth of the loop.  Here the addresses are one scalar base a tile
//    plus lane offsets fixed before the loop, whole tiles need no guard, and
//    the ragged last tile goes through ordinary loads that write zeros.
//  * A block of three waves (33 .. 48 columns) leaves the fourth SIMD idle:
//    waves are dealt to the SIMDs from the first one on.  KG row groups of WM
//    waves (each takes every KG-th group of four rows of a stage, summed in
//    order at the end) make whole rounds of the four SIMDs: twelve waves for
//    three column blocks (complex64 40x40 at 2^23 rows: 2.50 -> 1.99 ms).
// The loads are non-temporal: cached ones reached 6.0, these 6.8 TB/s.
// Two stages of 16 to 32 KB keep enough bytes in flight; the height, stages
// and row groups of every class are the autotuner's choice.
// Measured at 2^23 rows, before and after: real 24x24 582 -> 487 us, 40x40
// 1034 -> 772, 48x48 1078 -> 905 (7.1 TB/s), 56x56 1650 -> 1214, 64x64 1754 ->
// 1354; complex 40x24 2306 -> 1497, 48x48 3380 -> 2624, 64x64 (three
// products) 4528 -> 3632; complex64 48x48 2940 -> 2316.
// SYM (A^T A): one matrix is staged and each wave forms half of its row of
// blocks (wave w block columns w, w + 1, .. around the circle), writing the
// mirrored entries too: real 40x40 at 2^21 rows 200 -> 144 us.
#pragma once
#include "tsg_kernels.hpp"

namespace tsg {

// Four independent 4 x 4 x 4 products (b = 0..3): lane 16 k + 4 b + i supplies
// A_b(i, k) and B_b(k, i), lane 16 i + 4 b + j holds D_b(i, j) (checked on
// gfx950 with an in-bounds probe).
__device__ __forceinline__ double mfma4(double a, double b, double c)
{
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// One direct load of a wave: 64 lanes x 16 bytes from base + off into 1 KB of
// LDS at byte lds_off (lane l at lds_off + 16 l).  The compiler does not count
// this load: stage_wait waits for it.  (The load writes no register.)
__device__ __forceinline__ void dma_load(const char* base, uint32_t off, uint32_t lds_off)
{
    // wave-uniform by construction: into scalar registers
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)base);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uintptr_t)base >> 32));
    const uint64_t b = ((uint64_t)hi << 32) | lo;
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :: "s"(__builtin_amdgcn_readfirstlane(lds_off)), "v"(off), "s"(b) : "memory", "m0");
}

// Wait until at most N of the wave's loads are outstanding (and its LDS reads
// have completed: the barrier that follows hands their buffer over).
template <int N>
__device__ __forceinline__ void stage_wait()
{
    static_assert(N < 64, "vmcnt holds six bits");
    __asm__ volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N) : "memory");
}

// Byte offset (from the first row of a tile) of the 16-byte chunk that lane
// `lane` of piece p brings: chunk 64 p + lane of the tile's packed rows (rb
// bytes each, starts ld bytes apart).  Contiguous rows: chunks may straddle
// rows; else rb is a multiple of 16.  Chunks past the tile repeat its last one
// (their place in LDS is padding).
__device__ __forceinline__ uint32_t chunk_off(int p, int lane, uint32_t rb, uint32_t ld, uint32_t tile)
{
    uint32_t byte = (uint32_t)(64 * p + lane) * 16;
    byte = byte < tile ? byte : tile - 16;
    if (rb == ld) return byte;
    const uint32_t row = byte / rb;
    return row * ld + (byte - row * rb);
}

// Wait until at most `a` (uniform, at most 16) of the wave's loads are outstanding.
__device__ __forceinline__ void stage_wait_upto(int a)
{
    if (a < 4) {
        if (a < 2) {
            if (a < 1) stage_wait<0>(); else stage_wait<1>();
        } else {
            if (a < 3) stage_wait<2>(); else stage_wait<3>();
        }
    } else if (a < 8) {
        if (a < 6) {
            if (a < 5) stage_wait<4>(); else stage_wait<5>();
        } else {
            if (a < 7) stage_wait<6>(); else stage_wait<7>();
        }
    } else if (a < 12) {
        if (a < 10) stage_wait<8>(); else stage_wait<10>();
    } else {
        if (a < 16) stage_wait<12>(); else stage_wait<16>();
    }
}

__device__ __forceinline__ double flip_sign(double v, int mask)
{
    return __hiloint2double(__double2hiint(v) ^ mask, __double2loint(v));
}

template <int NB, int NQ, int WM, int KG, int RT, int NS, bool CPLX, bool F32, bool G3, bool SYM, int OCC>
__global__ void __launch_bounds__(WM * KG * kWave, OCC)
tsmttsm_stage(int64_t K, int MX, int NY, const void* __restrict__ Xv, int64_t ldx, const void* __restrict__ Yv,
              int64_t ldy, double* __restrict__ C, int64_t ldc, double* __restrict__ ws, int conj, int swap)
{
    using S = typename storage<CPLX, F32>::type;
    using T = elem_t<CPLX>;
    constexpr int CW = CPLX ? 2 : 1;
    constexpr int WPB = WM * KG;
    constexpr int KS = RT / (4 * KG);  // steps of four rows of a wave and stage
    static_assert(RT % (4 * KG) == 0, "whole steps");
    constexpr int ES = sizeof(S);
    // direct loads of one wave and stage at most (widths of the class)
    constexpr int XP = (RT * 16 * WM * ES / 1024 + WPB - 1) / WPB;
    constexpr int YP = SYM ? 1 : (RT * (16 * NB + 4 * NQ) * ES / 1024 + WPB) / WPB;
    static_assert(CPLX || !G3, "the three-product form is for complex data");
    static_assert(!SYM || (NQ == 0 && NB == WM / 2 + 1), "the symmetric form: half of the blocks of P");
    extern __shared__ __attribute__((aligned(1024))) char sm[];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lr = lane >> 4, lc = lane & 15;
    const int wm = wave % WM, kg = wave / WM;

    // a stage: X's tile of RT packed rows in whole pieces of 1 KB, then Y's;
    // wave w brings pieces w, w + WPB, ... of each
    const uint32_t xr = (uint32_t)MX * ES, yr = (uint32_t)NY * ES;  // bytes of a row
    const uint32_t xt = xr * RT, yt = SYM ? 0u : yr * RT;           // bytes of a tile
    const int px = (int)((xt + 1023) >> 10), py = (int)((yt + 1023) >> 10);
    const uint32_t sbytes = (uint32_t)(px + py) << 10;
    const int cx = (px - wave + WPB - 1) / WPB, cy = SYM ? 0 : (py - wave + WPB - 1) / WPB;
    const int cnt = cx + cy;
    const int64_t xld = ldx * ES, yld = ldy * ES;
    uint32_t xoff[XP], yoff[YP];
#pragma unroll
    for (int i = 0; i < XP; ++i) xoff[i] = chunk_off(wave + i * WPB, lane, xr, (uint32_t)xld, xt);
#pragma unroll
    for (int i = 0; i < YP; ++i) yoff[i] = SYM ? 0u : chunk_off(wave + i * WPB, lane, yr, (uint32_t)yld, yt);
    const uint32_t lbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)sm;
    const char* const xb = static_cast<const char*>(Xv);
    const char* const yb = static_cast<const char*>(Yv);
    auto issue = [&](int64_t t, int buf) {
        const uint32_t l0 = lbase + (uint32_t)buf * sbytes + ((uint32_t)wave << 10);
        const char* xs = xb + t * RT * xld;
#pragma unroll
        for (int i = 0; i < XP; ++i)
            if (i < cx) dma_load(xs, xoff[i], l0 + (i * WPB << 10));
        if constexpr (!SYM) {
            const char* ys = yb + t * RT * yld;
            const uint32_t l1 = l0 + ((uint32_t)px << 10);
#pragma unroll
            for (int i = 0; i < YP; ++i)
                if (i < cy) dma_load(ys, yoff[i], l1 + (i * WPB << 10));
        }
    };

    // G3: P1 in acc, P2 in acci, P3 in accs
    dbl4 acc[NB ? NB : 1], acci[CPLX && NB ? NB : 1], accs[G3 && NB ? NB : 1];
    double qa[NQ ? NQ : 1], qi[CPLX && NQ ? NQ : 1], qs[G3 && NQ ? NQ : 1];
    const dbl4 z4 = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        acc[j] = z4;
        if constexpr (CPLX) acci[j] = z4;
        if constexpr (G3) accs[j] = z4;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        qa[q] = 0.0;
        if constexpr (CPLX) qi[q] = 0.0;
        if constexpr (G3) qs[q] = 0.0;
    }

    // element offsets of this lane's operands in a packed tile (columns past a
    // width read a neighbouring element: such products reach only entries that
    // are never stored)
    const int xo = (4 * kg + lr) * MX + 16 * wm + lc;
    const int yo = (4 * kg + lr) * NY + lc, yq = (4 * kg + lr) * NY + 16 * NB + (lane & 3);
    int bsym[SYM ? NB : 1];  // SYM: the wave's blocks of Y, (wm + j) mod WM
#pragma unroll
    for (int j = 0; j < (SYM ? NB : 0); ++j) bsym[j] = 16 * ((wm + j) % WM);
    const int cmask = conj ? (int)0x80000000 : 0;
    // blocks halfway round the circle are the work of the lower waves only
    const bool half = !SYM || (WM & 1) || wm < WM / 2;

    auto multiply = [&](const char* st) {
        const S* xs = reinterpret_cast<const S*>(st);
        const S* ys = SYM ? xs : reinterpret_cast<const S*>(st + ((uint32_t)px << 10));
        auto rd = [](const S* p) -> T {
            if constexpr (CPLX) return zd{(double)p->re, (double)p->im};
            else return (double)*p;
        };
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            T yv[NB ? NB : 1], qv[NQ ? NQ : 1];
            const T xv = rd(xs + (4 * KG * s * MX + xo));
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if constexpr (SYM)
                    yv[j] = rd(ys + (4 * KG * s * NY + yo) + bsym[j]);
                else
                    yv[j] = rd(ys + (4 * KG * s * NY + yo) + 16 * j);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) qv[q] = rd(ys + (4 * KG * s * NY + yq) + 4 * q);
            if constexpr (!CPLX) {
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    if (!SYM || j < WM / 2 || (WM & 1) || half) acc[j] = mfma16(xv, yv[j], acc[j]);
#pragma unroll
                for (int q = 0; q < NQ; ++q) qa[q] = mfma4(xv, qv[q], qa[q]);
            } else if constexpr (G3) {
                const double xi = flip_sign(xv.im, cmask), sx = xv.re + xi;
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[j] = mfma16(xv.re, yv[j].re, acc[j]);
#pragma unroll
                for (int q = 0; q < NQ; ++q) qa[q] = mfma4(xv.re, qv[q].re, qa[q]);
#pragma unroll
                for (int j = 0; j < NB; ++j) acci[j] = mfma16(xi, yv[j].im, acci[j]);
#pragma unroll
                for (int q = 0; q < NQ; ++q) qi[q] = mfma4(xi, qv[q].im, qi[q]);
#pragma unroll
                for (int j = 0; j < NB; ++j) accs[j] = mfma16(sx, yv[j].re + yv[j].im, accs[j]);
#pragma unroll
                for (int q = 0; q < NQ; ++q) qs[q] = mfma4(sx, qv[q].re + qv[q].im, qs[q]);
            } else {
                // all products with Re(x) first, so that the two updates of one
                // accumulator are apart
                const double xi = flip_sign(xv.im, cmask), xn = -xi;
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    if (!SYM || j < WM / 2 || (WM & 1) || half) {
                        acc[j] = mfma16(xv.re, yv[j].re, acc[j]);
                        acci[j] = mfma16(xv.re, yv[j].im, acci[j]);
                    }
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    qa[q] = mfma4(xv.re, qv[q].re, qa[q]);
                    qi[q] = mfma4(xv.re, qv[q].im, qi[q]);
                }
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    if (!SYM || j < WM / 2 || (WM & 1) || half) {
                        acc[j] = mfma16(xn, yv[j].im, acc[j]);
                        acci[j] = mfma16(xi, yv[j].re, acci[j]);
                    }
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    qa[q] = mfma4(xn, qv[q].im, qa[q]);
                    qi[q] = mfma4(xi, qv[q].re, qi[q]);
                }
            }
        }
    };

    const int64_t nfull = K / RT;
    const int64_t G = gridDim.x;
    int64_t t = blockIdx.x;
#pragma unroll
    for (int i = 0; i < NS - 1; ++i)
        if (t + i * G < nfull) issue(t + i * G, i);
    for (int buf = 0; t < nfull; t += G) {
        // stages t + G .. t + (NS - 2) G may stay in flight
        int later = 0;
#pragma unroll
        for (int i = 1; i < NS - 1; ++i)
            if (t + i * G < nfull) later += cnt;
        stage_wait_upto(later);
        // every wave's loads of the stage have landed, and every wave has read
        // the buffer that the next loads go to (stage t - G's)
        __builtin_amdgcn_s_barrier();
        __asm__ volatile("" ::: "memory");
        if (t + (NS - 1) * G < nfull) issue(t + (NS - 1) * G, buf == 0 ? NS - 1 : buf - 1);
        multiply(sm + (uint32_t)buf * sbytes);
        buf = buf == NS - 1 ? 0 : buf + 1;
    }
    // the ragged last tile, brought by ordinary loads, rows past K zero
    if (K % RT != 0 && nfull % G == blockIdx.x) {
        __syncthreads();
        const int rows = (int)(K - nfull * RT);
        auto fill = [&](const S* g, int64_t ld, int width, char* dst) {
            using SR = typename real_of<S>::type;
            SR* d = reinterpret_cast<SR*>(dst);
            const int w = width * CW;
            for (int e = threadIdx.x; e < RT * w; e += WPB * kWave) {
                const int r = e / w, c = e - r * w;
                d[e] = r < rows ? reinterpret_cast<const SR*>(g + (nfull * RT + r) * ld)[c] : (SR)0;
            }
        };
        fill(static_cast<const S*>(Xv), ldx, MX, sm);
        if constexpr (!SYM) fill(static_cast<const S*>(Yv), ldy, NY, sm + ((uint32_t)px << 10));
        __syncthreads();
        multiply(sm);
    }

    if constexpr (G3) {
        // Re = P1 - P2, Im = P3 - P1 - P2
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const dbl4 p1 = acc[j], p2 = acci[j];
            acc[j] = p1 - p2;
            acci[j] = accs[j] - p1 - p2;
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const double p1 = qa[q], p2 = qi[q];
            qa[q] = p1 - p2;
            qi[q] = qs[q] - p1 - p2;
        }
    }
    // row groups: the sums of groups 1, 2, ... are added to group 0's in order
    if constexpr (KG > 1) {
        constexpr int NA = 4 * NB + NQ;  // doubles of a lane and part (the host sizes LDS for them)
        double* const fold = reinterpret_cast<double*>(sm) + wm * (NA * CW * kWave) + lane;
        auto each = [&](auto fn) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    double v = acc[j][r];
                    fn(v, 4 * j + r);
                    acc[j][r] = v;
                    if constexpr (CPLX) {
                        double w = acci[j][r];
                        fn(w, NA + 4 * j + r);
                        acci[j][r] = w;
                    }
                }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                fn(qa[q], 4 * NB + q);
                if constexpr (CPLX) fn(qi[q], NA + 4 * NB + q);
            }
        };
        for (int g = 1; g < KG; ++g) {
            __syncthreads();
            if (kg == g) each([&](double& v, int i) { fold[i * kWave] = v; });
            __syncthreads();
            if (kg == 0) each([&](double& v, int i) { v += fold[i * kWave]; });
        }
        if (kg != 0) return;
    }

    // the waves own disjoint entries: each lane writes its own to the block's
    // slot of the workspace, or to C if there is one block only
    const int ncol = swap ? MX : NY;
    const bool direct = gridDim.x == 1;
    double* const slot = ws + (direct ? 0 : (size_t)blockIdx.x * ((size_t)MX * NY * CW));
    auto put = [&](int m, int n, double re, double im) {
        if (m >= MX || n >= NY) return;
        const int row = swap ? n : m, col = swap ? m : n;
        double* p = direct ? C + ((int64_t)row * ldc + col) * CW : slot + (row * ncol + col) * CW;
        p[0] = re;
        if constexpr (CPLX) p[1] = im;
    };
    // conj(X)^T Y was summed for conj; with X and Y exchanged its conjugate is wanted
    const bool neg = conj && swap;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        if (SYM && j == WM / 2 && !(WM & 1) && !half) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * wm + lr + 4 * r;
            const int n = (SYM ? bsym[j] : 16 * j) + lc;
            const double re = acc[j][r];
            double im = 0.0;
            if constexpr (CPLX) im = acci[j][r];
            put(m, n, re, neg ? -im : im);
            if (SYM && j > 0) put(n, m, re, conj ? -im : im);
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int m = 16 * wm + 4 * ((lane >> 2) & 3) + lr;
        const int n = 16 * NB + 4 * q + (lane & 3);
        double im = 0.0;
        if constexpr (CPLX) im = qi[q];
        put(m, n, qa[q], neg ? -im : im);
    }
}

}  // namespace tsg
