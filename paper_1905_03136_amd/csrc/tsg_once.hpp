// tsg_once.hpp -- TSMM on the matrix cores, one small tile a wave (tsmm_once).
//
// B = alpha op(A) C + beta B for run-time widths, MS slices of four columns
// of A and NB blocks of 16 and NQ groups of 4 columns of B.  A wave takes
// R = 16 U rows: it brings them into its own part of LDS with direct 16-byte
// loads (1 KB of consecutive bytes a load, no register holds them), reads the
// matrix-core operands from there, writes the results over them and stores
// those as runs of 1 KB.  So every access to memory is a whole line whatever
// the widths, and nothing but the ragged last tile needs a row guard.
//
// What bounds it: a read and a write stream of HBM.  Their rate depends on
// how compact the addresses in flight are: a copy by persistent blocks that
// stride over the matrix reaches 5.4 TB/s, by blocks launched in order for
// 4 KB each 6.6, for 8 KB 6.4, for 16 KB 6.0, and blocks that work through
// runs of tiles fall back to 5.4 within 16 tiles, however short their tiles
// (the blocks drift apart).  Hence one tile a wave, about 2 KB of it, and a
// grid of all tiles.  C is small: each wave reads its operands from the
// caches while its rows are on the way (CL: too many for registers, the block
// shares a copy in LDS).
//
// Wide matrices (large C, or bound by the matrix cores) would spend more on C
// than on their tile: DB keeps a block on its copy of C, for tiles a grid
// apart, with the next tile's rows brought while one is multiplied.
//
// Measured on 2^22 rows in GB/s read and written, tsmm_mfma's before -> this
// one: binary64 12 x 16 5454 -> 6002, 8 x 28 4687 -> 5874, 20 x 20 5385 ->
// 5939, 28 x 56 3995 -> 5128 (DB); complex 20 x 16 4950 -> 5660, 20 x 20 4239
// -> 5501; binary32 storage 24 x 16 2630 -> 4972, 48 x 48 2111 -> 4034 (DB);
// complex of it 20 x 20 2409 -> 3848, 40 x 24 2123 -> 3425 (DB).  Where C
// outgrows this form tsmm_mfma's persistent waves with operands in registers
// stay ahead (32 x 32 is the last binary64 square: 2^21 rows 196 us there, 190
// here with registers for four waves a SIMD, 178 for two, which lets more of C
// be read ahead of the products): binary64 48 x 48 614 us against 655 here, complex 48 x 48 1413
// against more than 1600, complex 64 x 64 2108 against 4444.
#pragma once
#include "tsg_stage.hpp"
#include "tsg_registry.hpp"

namespace tsg {

constexpr int kOncePiece = 1024 + 16;  // LDS bytes from one 1 KB piece to the next: rows of a power
                                       // of two bytes would all start in the same bank

// LDS byte of byte b of a wave's run.
__device__ __forceinline__ int once_at(int b) { return b + ((b >> 10) << 4); }

// Byte offset in memory of byte b of a run of packed rows of rb bytes (starts
// ld bytes apart, magic = ceil(2^32 / rb); b below 64 KB): rows contiguous, or
// whole 16-byte chunks.
__device__ __forceinline__ uint32_t once_off(uint32_t b, uint32_t rb, uint32_t ld, uint32_t magic)
{
    if (rb == ld) return b;
    const uint32_t row = __umulhi(b, magic);
    return row * ld + (b - row * rb);
}

template <int MS, int NB, int NQ, int U, int WPB, bool CPLX, bool F32, bool CL, bool DB, int OCC>
__global__ void __launch_bounds__(WPB * kWave, OCC)
tsmm_once(int64_t K, int M, int N, const void* __restrict__ Av, int64_t lda, const double* __restrict__ Cm,
          int64_t ldc, void* __restrict__ Bv, int64_t ldb, double alpha, double beta, int conj, int opc,
          uint32_t amagic, uint32_t bmagic, int wbytes)
{
    using S = typename storage<CPLX, F32>::type;
    using T = elem_t<CPLX>;
    using SR = typename real_of<S>::type;
    constexpr int CW = CPLX ? 2 : 1;
    constexpr int ES = sizeof(S);
    constexpr int R = 16 * U;
    constexpr int NG = NB + NQ;
    constexpr int NP = 16 * NB + 4 * NQ;
    // C in LDS: rows of CLD elements, real ones 128 bytes apart modulo 256, so
    // that the two rows of a half-wave's read lie in different banks
    constexpr int CLD = CPLX ? NP : NP + (48 - NP % 32) % 32;
    constexpr int CBYTES = CL ? 4 * MS * CLD * CW * 8 : 0;
    constexpr int PA = (R * 4 * MS * ES + 1023) / 1024;  // pieces at most
    constexpr int PB = (R * NP * ES + 1023) / 1024;
    extern __shared__ __attribute__((aligned(1024))) char sm[];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lr = lane >> 4, lc = lane & 15;
    const uint32_t arow = (uint32_t)M * ES, brow = (uint32_t)N * ES;
    const uint32_t at = arow * R, bt = brow * R;  // bytes of a tile
    const uint32_t ald = (uint32_t)(lda * ES), bld = (uint32_t)(ldb * ES);
    const bool flat = brow == bld;
    const bool read_b = beta != 0.0;
    // the wave's part of LDS: A's rows, then B's, and the old rows of B; with
    // DB two of them in turn
    char* run = sm + CBYTES + wave * (DB ? 2 * wbytes : wbytes);
    const int oldat = (((at > bt ? at : bt) + 1023) >> 10) * kOncePiece + 256;
    const int npb = (int)((bt + 1023) >> 10);  // stores of a tile
    const int64_t ntiles = (K + R - 1) / R;

    // a run of `bytes` in whole pieces (lanes past it repeat its last 16 bytes)
    auto bring = [&](auto P, const char* base, uint32_t rb, uint32_t ld, uint32_t magic, uint32_t bytes, uint32_t lds) {
#pragma unroll
        for (int p = 0; p < decltype(P)::value; ++p)
            if ((uint32_t)p << 10 < bytes) {
                uint32_t b = ((uint32_t)p << 10) + 16 * lane;
                b = b < bytes ? b : bytes - 16;
                dma_load(base, once_off(b, rb, ld, magic), lds + p * kOncePiece);
            }
    };
    // the ragged last tile: ordinary loads, rows past K zero
    auto fill = [&](const S* base, int64_t ld, int width, int rows, char* dst) {
        const int w = width * CW;
        for (int e = lane; e < R * w; e += kWave) {
            const int r = e / w, c = e - r * w;
            *reinterpret_cast<SR*>(dst + once_at(e * (int)sizeof(SR))) =
                r < rows ? reinterpret_cast<const SR*>(base + r * ld)[c] : (SR)0;
        }
    };
    auto rows_in = [&](int64_t t, char* run) {
        char* const old = run + oldat;
        const uint32_t lrun = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)run;
        const uint32_t lold = lrun + oldat;
        const int64_t r0 = t * R;
        const S* a = static_cast<const S*>(Av) + r0 * lda;
        const S* b = static_cast<const S*>(Bv) + r0 * ldb;
        if (r0 + R <= K) {
            bring(std::integral_constant<int, PA>{}, reinterpret_cast<const char*>(a), arow, ald, amagic, at, lrun);
            if (read_b)
                bring(std::integral_constant<int, PB>{}, reinterpret_cast<const char*>(b), brow, bld, bmagic, bt, lold);
        } else {
            fill(a, lda, M, (int)(K - r0), run);
            if (read_b) fill(b, ldb, N, (int)(K - r0), old);
        }
    };

    int64_t t = (int64_t)blockIdx.x * WPB + wave;
    if (t < ntiles) rows_in(t, run);

    // element (m, n) of the small operand, zero past the widths
    auto small = [&](int m, int n) -> T {
        const bool ok = m < M && n < N;
        const int64_t i = ok ? small_index(m, n, ldc, opc) : 0;
        if constexpr (CPLX) {
            const double re = Cm[2 * i], im = Cm[2 * i + 1];
            return zd{ok ? re : 0.0, ok ? (opc == 2 ? -im : im) : 0.0};
        } else {
            const double v = Cm[i];
            return ok ? v : 0.0;
        }
    };
    T cr[CL ? 1 : MS][CL ? 1 : NG];
    T* const cl = reinterpret_cast<T*>(sm);
    if constexpr (CL) {
        constexpr int E = 4 * MS * CLD, TH = WPB * kWave, STEP = 8;
#pragma unroll 1
        for (int e0 = 0; e0 < E; e0 += STEP * TH) {
            T v[STEP];
#pragma unroll
            for (int i = 0; i < STEP; ++i) {
                const int e = e0 + i * TH + (int)threadIdx.x;
                if (e0 + i * TH < E) v[i] = small(e / CLD, e - e / CLD * CLD);
            }
#pragma unroll
            for (int i = 0; i < STEP; ++i) {
                const int e = e0 + i * TH + (int)threadIdx.x;
                if (e < E) cl[e] = v[i];
            }
        }
        __syncthreads();
    } else {
#pragma unroll
        for (int s = 0; s < MS; ++s) {
#pragma unroll
            for (int j = 0; j < NB; ++j) cr[s][j] = small(4 * s + lr, 16 * j + lc);
#pragma unroll
            for (int q = 0; q < NQ; ++q) cr[s][NB + q] = small(4 * s + lr, 16 * NB + 4 * q + (lane & 3));
        }
    }
    auto copnd = [&](int s, int g) -> T {
        if constexpr (!CL) return cr[s][g];
        else return cl[(4 * s + lr) * CLD + (g < NB ? 16 * g + lc : 16 * NB + 4 * (g - NB) + (lane & 3))];
    };
    const int cmask = conj ? (int)0x80000000 : 0;

    char* next = run + (DB ? wbytes : 0);
    for (bool first = true; t < ntiles; t += (int64_t)gridDim.x * WPB, first = false) {
        const int64_t tn = t + (int64_t)gridDim.x * WPB;
        // the tile's rows (before them: nothing; after them: the stores of the tile before)
        if (DB && !first) stage_wait_upto(npb);
        else stage_wait<0>();
        if (DB && tn < ntiles) rows_in(tn, next);
        char* const old = run + oldat;
        dbl4 acc[U][NB ? NB : 1], acci[CPLX ? U : 1][CPLX && NB ? NB : 1];
        double qa[U][NQ ? NQ : 1], qi[CPLX ? U : 1][CPLX && NQ ? NQ : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                acc[u][j] = dbl4{0.0, 0.0, 0.0, 0.0};
                if constexpr (CPLX) acci[u][j] = dbl4{0.0, 0.0, 0.0, 0.0};
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                qa[u][q] = 0.0;
                if constexpr (CPLX) qi[u][q] = 0.0;
            }
        }
#pragma unroll
        for (int s = 0; s < MS; ++s) {
            T av[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const S* p = reinterpret_cast<const S*>(run + once_at(((16 * u + lc) * M + 4 * s + lr) * ES));
                // columns past M hold the next row's values: zero
                const bool ok = 4 * s + 3 < 4 * (MS - 2) || 4 * s + lr < M;
                if constexpr (CPLX) av[u] = keep(ok, zd{(double)p->re, (double)p->im});
                else av[u] = keep(ok, (double)*p);
            }
            if constexpr (!CPLX) {
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const double c = copnd(s, g);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (g < NB) acc[u][g < NB ? g : 0] = mfma16(av[u], c, acc[u][g < NB ? g : 0]);
                        else qa[u][g < NB ? 0 : g - NB] = mfma4(av[u], c, qa[u][g < NB ? 0 : g - NB]);
                    }
                }
            } else {
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const zd c = copnd(s, g);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const double ai = flip_sign(av[u].im, cmask);
                        if (g < NB) {
                            const int j = g < NB ? g : 0;
                            acc[u][j] = mfma16(av[u].re, c.re, acc[u][j]);
                            acci[u][j] = mfma16(av[u].re, c.im, acci[u][j]);
                            acc[u][j] = mfma16(ai, -c.im, acc[u][j]);
                            acci[u][j] = mfma16(ai, c.re, acci[u][j]);
                        } else {
                            const int q = g < NB ? 0 : g - NB;
                            qa[u][q] = mfma4(av[u].re, c.re, qa[u][q]);
                            qi[u][q] = mfma4(av[u].re, c.im, qi[u][q]);
                            qa[u][q] = mfma4(ai, -c.im, qa[u][q]);
                            qi[u][q] = mfma4(ai, c.re, qi[u][q]);
                        }
                    }
                }
            }
        }
        // results over the rows of A (this wave's reads of them are done)
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        auto put = [&](int row, int n, double re, double im) {
            if (n >= N) return;
            const int o = once_at((row * N + n) * ES);
            if constexpr (!CPLX) {
                double v = alpha * re;
                if (read_b) v = __builtin_fma(beta, (double)*reinterpret_cast<const S*>(old + o), v);
                *reinterpret_cast<S*>(run + o) = (S)v;
            } else {
                zd v = zd{alpha * re, alpha * im};
                if (read_b) {
                    const S w = *reinterpret_cast<const S*>(old + o);
                    v = zd{__builtin_fma(beta, (double)w.re, v.re), __builtin_fma(beta, (double)w.im, v.im)};
                }
                *reinterpret_cast<S*>(run + o) = S{(SR)v.re, (SR)v.im};
            }
        };
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    double im = 0.0;
                    if constexpr (CPLX) im = acci[u][j][r];
                    put(16 * u + lr + 4 * r, 16 * j + lc, acc[u][j][r], im);
                }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                double im = 0.0;
                if constexpr (CPLX) im = qi[u][q];
                put(16 * u + 4 * ((lane >> 2) & 3) + lr, 16 * NB + 4 * q + (lane & 3), qa[u][q], im);
            }
        }
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int64_t r0 = t * R;
        char* const bb = reinterpret_cast<char*>(static_cast<S*>(Bv) + r0 * ldb);
        if (r0 + R <= K) {
            typedef uint32_t u4 __attribute__((ext_vector_type(4)));
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                const uint32_t b = ((uint32_t)p << 10) + 16 * lane;
                if (p >= npb) break;
                if (b < bt) {
                    const u4 v = *reinterpret_cast<const u4*>(run + p * kOncePiece + 16 * lane);
                    u4* q = reinterpret_cast<u4*>(bb + once_off(b, brow, bld, bmagic));
                    // whole lines past the caches; segments of padded rows are
                    // merged there
                    if (flat) __builtin_nontemporal_store(v, q);
                    else *q = v;
                }
            }
        } else {
            const int w = N * CW, rows = (int)(K - r0);
            for (int e = lane; e < rows * w; e += kWave) {
                const int r = e / w, c = e - r * w;
                reinterpret_cast<SR*>(bb + (size_t)r * bld)[c] =
                    *reinterpret_cast<const SR*>(run + once_at(e * (int)sizeof(SR)));
            }
        }
        __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (!DB && tn < ntiles) rows_in(tn, run);
        if (DB) {
            char* const r = run;
            run = next;
            next = r;
        }
    }
}

}  // namespace tsg
