// tsg_runtime.hip -- host side of libtsgemm: argument validation, choice of
// the kernel variant, per-(device, stream) workspace, grid sizing and launch.
// The C ABI is declared in include/tsgemm.h.
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

#include "../../include/tsgemm.h"
#include "tsg_registry.hpp"


namespace tsg {

// Sum of the G per-block partials of a TSMTTSM launch (slot b holds E doubles
// at ws + b * E) into C, in a fixed order: each block of kFoldThreads threads
// takes EB consecutive entries (EB a power of two <= 8) and S = kFoldThreads /
// EB slices; slice s sums slots s, s + S, s + 2S, ... in increasing order
// (loads issued eight at a time, the additions in slot order), and the slices
// are combined by a fixed pairwise tree.  The result is bitwise reproducible
// for a given grid.  Wide blocks keep the chain of dependent loads of a
// thread short (G <= 2048 slots: at most two batches of eight), which is what
// the fold's time is made of at small K.
constexpr int kFoldThreads = 1024;

template <int CW>
__global__ void __launch_bounds__(kFoldThreads)
fold_partials(const double* __restrict__ ws, int G, int E, int EB, int N, double* __restrict__ C, int64_t ldc)
{
    __shared__ double red[kFoldThreads];
    const int S = kFoldThreads / EB;
    const int el = threadIdx.x & (EB - 1);
    const int s = threadIdx.x / EB;
    const int e = blockIdx.x * EB + el;
    double v = 0.0;
    if (e < E) {
        int b = s;
        for (; b + 7 * S < G; b += 8 * S) {
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = ws[(size_t)(b + u * S) * E + e];
#pragma unroll
            for (int u = 0; u < 8; ++u) v += x[u];
        }
        for (; b < G; b += S) v += ws[(size_t)b * E + e];
    }
    red[threadIdx.x] = v;
    __syncthreads();
    for (int h = S / 2; h >= 1; h >>= 1) {
        if (s < h) red[threadIdx.x] += red[threadIdx.x + h * EB];
        __syncthreads();
    }
    if (s == 0 && e < E) {
        const int q = e / CW;
        const int m = q / N, n = q - m * N;
        C[((int64_t)m * ldc + n) * CW + (e - q * CW)] = red[el];
    }
}

// Reduction ablation only (never the default): every block's partial is
// added into C with global FP64 atomics, as the paper's global-atomic variant
// does (Section 3.2); C is cleared first.  Thread (b, e) adds slot b, entry e;
// the order of the additions, and so the rounding, varies from run to run.
template <int CW>
__global__ void __launch_bounds__(256)
atomic_partials(const double* __restrict__ ws, int G, int E, int N, double* __restrict__ C, int64_t ldc)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)G * E) return;
    const int b = (int)(i / E), e = (int)(i - (int64_t)b * E);
    const int q = e / CW;
    const int m = q / N, n = q - m * N;
    atomicAdd(C + ((int64_t)m * ldc + n) * CW + (e - q * CW), ws[(size_t)b * E + e]);
}

__global__ void __launch_bounds__(256) clear_small(double* __restrict__ C, int M, int N, int CW, int64_t ldc)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= M * N * CW) return;
    const int q = i / CW;
    const int m = q / N, n = q - m * N;
    C[((int64_t)m * ldc + n) * CW + (i - q * CW)] = 0.0;
}

// Fixed scratch of tsg_tsmttsm_noalloc: the per-block partial sums of one
// launch (a slot of M N (x2 complex) doubles per block).  Every device the
// library runs on holds its own copy for the life of the process.  In host
// code the array's name is only a stand-in; kernels and copies take the
// device address obtained once per device with hipGetSymbolAddress.
constexpr size_t kScratchBytes = size_t(32) << 20;
static __device__ __align__(256) double scratch[kScratchBytes / sizeof(double)];

__global__ void clear_counter(unsigned* c)
{
    if (threadIdx.x == 0) *c = 0u;
}

}  // namespace tsg

namespace {

thread_local std::string g_err;
thread_local std::string g_force;  // variant forced by tsg_force_variant ("" = automatic choice)
thread_local int g_grid_cap = 0;   // block cap set by tsg_set_grid_limit (0 = none)
thread_local int g_reduction = 0;  // cross-block reduction set by tsg_set_reduction (0 = fixed-order fold)

void set_error(const char* msg) noexcept
{
    try {
        g_err = msg;
    } catch (...) {
        g_err.clear();
    }
}

tsg_status fail(tsg_status s, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    set_error(buf);
    return s;
}

// What an entry point returns whose host allocation failed (the index of the
// variants on the first call, a workspace's entry, a name): no exception
// leaves it.
template <class R>
R no_memory(R r)
{
    set_error("host allocation failed");
    return r;
}

constexpr int kMaxWidth = 64;

}  // namespace

namespace tsg {
size_t orth_workspace_size(int64_t K, int32_t M, int32_t N, int32_t count);  // tsg_batched.hip

// Error detail for tsg_last_error() from the library's other units.
tsg_status report(tsg_status s, const char* msg)
{
    set_error(msg);
    return s;
}
}  // namespace tsg

namespace {

struct DeviceInfo {
    int cus = 0;
    bool ok = false;
};

struct Workspace {
    void* data = nullptr;  // `bytes` of it, and a counter (zero between launches)
    size_t bytes = 0;
    std::mutex* calls = nullptr;  // held while a call's launches are enqueued: another thread's on the same stream
                                  // would write its slots between a kernel and the sum of its slots
    double* slots() const { return static_cast<double*>(data); }
    unsigned* counter() const { return reinterpret_cast<unsigned*>(static_cast<char*>(data) + bytes); }
};

std::mutex g_mu;
std::map<int, DeviceInfo> g_dev;
std::map<std::pair<int, hipStream_t>, Workspace> g_ws;
std::map<std::pair<int, hipStream_t>, std::mutex> g_ws_calls;  // never erased: calls hold pointers to them
// Outgrown workspaces, kept until tsg_finalize: a graph captured earlier on
// the stream may still hold one of them and write its partial sums there.
std::vector<std::pair<int, void*>> g_retired;
// (device, variant, LDS bytes of a block) -> blocks per CU
std::map<std::tuple<int, const tsg::Variant*, size_t>, int> g_occ;
// (device, variant) whose kernel may ask for all of a compute unit's LDS
std::set<std::pair<int, const tsg::Variant*>> g_lds;

std::map<int, double*> g_scratch;  // device -> device address of its no-alloc scratch

int is_complex(tsg_dtype dt) { return dt == TSG_C128 || dt == TSG_C64 || dt == TSG_C64_ACC32; }
size_t elem_bytes(tsg_dtype dt)
{
    switch (dt) {
    case TSG_R64: return 8;
    case TSG_C128: return 16;
    case TSG_R32: return 4;
    case TSG_C64: return 8;
    case TSG_R32_ACC32: return 4;
    case TSG_C64_ACC32: return 8;
    }
    return 0;
}
// Binary64-arithmetic type whose kernels also serve a binary32-arithmetic
// type (they are at least as accurate); -1 for the other types.
int twin_of(tsg_dtype dt)
{
    return dt == TSG_R32_ACC32 ? (int)TSG_R32 : dt == TSG_C64_ACC32 ? (int)TSG_C64 : -1;
}

tsg_status device_info(int dev, DeviceInfo* out)
{
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_dev.find(dev);
    if (it != g_dev.end() && it->second.ok) {
        *out = it->second;
        return TSG_OK;
    }
    DeviceInfo d;
    hipError_t e = hipDeviceGetAttribute(&d.cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return fail(TSG_E_HIP, "hipDeviceGetAttribute: %s", hipGetErrorString(e));
    d.ok = true;
    g_dev[dev] = d;
    *out = d;
    return TSG_OK;
}

tsg_status current_device(int* dev)
{
    hipError_t e = hipGetDevice(dev);
    if (e != hipSuccess) return fail(TSG_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    return TSG_OK;
}

constexpr size_t kLdsBytes = 160 * 1024;  // of a compute unit

// Lets a kernel ask for more than the 64 KB of LDS that a block may have by
// default: all of it, once, as its blocks' sizes vary with the widths and with
// beta, and a smaller one must not take from a larger one (g_mu held).
hipError_t allow_lds(int dev, const tsg::Variant& v, size_t lds)
{
    if (lds <= (64u << 10) || g_lds.count({dev, &v})) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(v.kernel(), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
    if (e == hipSuccess) g_lds.insert({dev, &v});
    return e;
}

// The same for a call about to launch `v`.
tsg_status lds_ready(int dev, const tsg::Variant& v, size_t lds)
{
    if (lds <= (64u << 10)) return TSG_OK;
    std::lock_guard<std::mutex> lk(g_mu);
    const hipError_t e = allow_lds(dev, v, lds);
    return e == hipSuccess ? TSG_OK : fail(TSG_E_HIP, "%zu bytes of LDS for %s: %s", lds, v.name, hipGetErrorString(e));
}

int occupancy(int dev, const tsg::Variant& v, size_t lds)
{
    std::lock_guard<std::mutex> lk(g_mu);
    auto key = std::make_tuple(dev, &v, lds);
    auto it = g_occ.find(key);
    if (it != g_occ.end()) return it->second;
    int blocks = 0;
    if (allow_lds(dev, v, lds) != hipSuccess) return 1;  // lds_ready reports it
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, v.kernel(), v.threads, lds) != hipSuccess || blocks < 1)
        blocks = 1;
    g_occ[key] = blocks;
    return blocks;
}

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Device address of `dev`'s scratch array; `dev` must be the current device.
// Resolved on the first use per device (tsg_init or the first no-alloc call).
tsg_status scratch_of(int dev, double** out)
{
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_scratch.find(dev);
    if (it != g_scratch.end()) {
        *out = it->second;
        return TSG_OK;
    }
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(tsg::scratch));
    if (e != hipSuccess || !p)
        return fail(TSG_E_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
    g_scratch[dev] = static_cast<double*>(p);
    *out = static_cast<double*>(p);
    return TSG_OK;
}

// Choose the variant: the exact (op, dtype, M, N) one if its access
// requirements hold, else the first run-time-width variant covering (M, N).
const tsg::Variant* pick_for(int op, int dt, int M, int N, const void* A, int64_t lda, const void* X,
                             int64_t ldx, bool beta_nz, int64_t K);

// The variant of (op, dt): for a binary32-arithmetic type, its own exact-width
// variant if there is one, else what its binary64-arithmetic twin would run
// (K: rows of the call, many if not given).
const tsg::Variant* pick(int op, tsg_dtype dt, int M, int N, const void* A, int64_t lda, const void* X,
                         int64_t ldx, bool beta_nz = false, int64_t K = INT64_MAX)
{
    if (elem_bytes(dt) == 0) return nullptr;
    const tsg::Variant* v = pick_for(op, (int)dt, M, N, A, lda, X, ldx, beta_nz, K);
    const int twin = twin_of(dt);
    if (twin >= 0 && (!v || v->M == 0)) {
        const tsg::Variant* w = pick_for(op, twin, M, N, A, lda, X, ldx, beta_nz, K);
        if (w) return w;
    }
    return v;
}

// The kernel that stages its rows in LDS serves every width above 16 (up to
// 16 x 16 row packing reads as fast and fills its fragments), of the layouts
// stage_reads takes; odd real leading dimensions and unaligned matrices stay
// with the register rings (24 columns of a 64-column basis against 8: 66 us
// at 2^20 rows by either).
//
// Whether it can read a tall matrix of width W: 16-byte chunks of a tile's packed rows, so contiguous rows of any
// width, or rows that are whole chunks 16-byte aligned (and a tile that spans
// less than 2^31 bytes, the reach of its 32-bit offsets).
bool stage_reads(const tsg::Variant& v, size_t es, int W, const void* p, int64_t ld)
{
    if (!aligned(p, 16)) return false;
    if (ld == W) return true;
    return W * es % 16 == 0 && ld * es % 16 == 0 && ld < (int64_t)((size_t)1 << 31) / (int64_t)(es * v.rows_per_tile);
}

// Complex widths summed in Gauss's three-product form, whose imaginary part
// has the larger error bound: squares of 49 .. 64 columns (64 x 64 at 2^22
// rows: 1.87 ms, four products 2.22 ms) and 49 .. 64 columns of A against 33
// .. 48 of B (64 x 48: 1.47 and 1.76 ms), which the kernels before this one
// summed that way too; no other width trades accuracy for it.
bool stage_gauss(int dt, int M, int N)
{
    if (dt == TSG_C64) return M == 64 && N == 64;
    return dt == TSG_C128 && M > 48 && (M == N || (N > 32 && N <= 48));
}

bool stage_serves(const tsg::Variant& v, int M, int N, const void* A, int64_t lda, const void* B, int64_t ldb)
{
    const int wide = M > N ? M : N, narrow = M > N ? N : M;
    const size_t es = elem_bytes((tsg_dtype)v.dt);
    if (v.maxM != (wide + 15) / 16 * 16) return false;
    if (v.maxN != (narrow + 3) / 4 * 4) return false;
    if (v.stage == 2) return M == N && A == B && lda == ldb && stage_reads(v, es, M, A, lda);
    return stage_reads(v, es, M, A, lda) && stage_reads(v, es, N, B, ldb);
}

// The table of variants by what a call asks for, each list in the order of the
// table.  A scan of its 2000 entries, for some types four of them a call, took
// 0.6 to 2 us of a small call's 4 to 6 (8958 x 16 by 16 in complex64 with
// binary32 arithmetic, in Python: 12.3 -> 7.9 us with the native calls).
struct VariantIndex {
    static constexpr int kW = kMaxWidth + 1, kTypes = 6;
    struct PerType {
        std::vector<const tsg::Variant*> exact[kW * kW], ranges, stage;
        const tsg::Variant* once[kW * kW] = {};
    };
    std::vector<PerType> of{2 * kTypes};

    VariantIndex()
    {
        for (int i = 0; i < tsg::kNumVariants; ++i) {
            const tsg::Variant& v = tsg::kVariants[i];
            PerType& t = of[v.op * kTypes + v.dt];
            if (v.stage) t.stage.push_back(&v);
            else if (v.once) {
                for (int m = v.once_m + 1; m <= v.maxM; ++m)
                    for (int n = v.once_n + 1; n <= v.maxN; ++n)
                        if (!t.once[m * kW + n]) t.once[m * kW + n] = &v;
            } else if (v.M) t.exact[v.M * kW + v.N].push_back(&v);
            else t.ranges.push_back(&v);
        }
    }
    const PerType& type(int op, int dt) const { return of[op * kTypes + dt]; }
    static const VariantIndex& get()
    {
        static const VariantIndex ix;
        return ix;
    }
};

// The LDS-staged kernel of a TSMTTSM, or null: widths above 16, 16-byte
// aligned matrices of a layout it can read; a matrix with itself (a Gram
// matrix) takes the form that reads it once and forms half of the products.
const tsg::Variant* pick_stage(int dt, int M, int N, const void* A, int64_t lda, const void* B, int64_t ldb, int64_t K)
{
    if (M <= 16 && N <= 16) return nullptr;
    if (dt == TSG_C128) {
        const int wide = M > N ? M : N, narrow = M > N ? N : M;
        const int padded = (wide + 15) / 16 * 16 * ((narrow + 3) / 4 * 4);  // products it forms, a row
        // few rows of wide matrices: its blocks of many row groups get one or
        // two tiles each (58 x 16, 10007 rows: 14.4 us against 10.8, 100003 rows
        // 32 and 29; 64 x 28, 30000 rows 1.25 of the others' time, 100003 1.00).
        // Squares stay: 64 x 64, 30000 rows 35 us against 39
        if (M != N && wide > 48 && narrow > 8 && K < 65536) return nullptr;
        // bound by the matrix cores: squares whose products it pads by more than
        // 1.6 (17 to 19 columns) have kernels of their widths (2^20 rows of 17 x
        // 17: 0.79 of its time; 20 x 20 1.17).  For 13 to 16 columns against 17
        // to 47 there are register rings in the three-product form (six real
        // products for eight): at 2^20 and 2^22 rows 0.89 to 1.03 of its time (33
        // x 16 0.89 and 0.96, 40 x 14 0.92 and 0.95, 17 x 16 0.93 and 0.96, 24 x 16
        // 1.01 and 0.95, 40 x 16 1.00 and 0.96, 31 x 16 1.03 twice), at 2^19 level
        // (0.93 to 1.05), at 2^18 1.04 to 1.10 and at 100003 rows 1.08 to 1.20
        if (M == N && 10 * padded > 16 * M * N) return nullptr;
        if (narrow > 12 && narrow <= 16 && wide <= 48 && wide % 16 && K >= (1 << 19)) return nullptr;
    }
    const bool sym = M == N && A == B && lda == ldb;
    const int gauss = !sym && stage_gauss(dt, M, N);
    for (const tsg::Variant* v : VariantIndex::get().type(tsg::OP_TSMTTSM, dt).stage)
        if (v->stage == (sym ? 2 : 1) && v->gauss == gauss && stage_serves(*v, M, N, A, lda, B, ldb)) return v;
    return nullptr;
}

// LDS bytes of a block that the launch asks for (kernels with run-time sizes).
size_t lds_for(const tsg::Variant& v, int M, int N, bool beta_nz = false)
{
    const size_t es = elem_bytes((tsg_dtype)v.dt);
    if (v.once) return v.once_c + (v.once_db ? 2 : 1) * (v.threads / 64) * tsg::once_wave_bytes(M, N, es, v.once, beta_nz);
    if (!v.stage) return 0;
    const int wide = M > N ? M : N, narrow = M > N ? N : M;
    return tsg::stage_lds_bytes(wide, narrow, es, v.rows_per_tile, v.stages, v.stage == 2, v.fold);
}

// The same for the one-tile kernel of TSMM (its tile: v.once rows): contiguous
// rows or whole 16-byte chunks, widths that fill its slices and groups but for
// the last (it masks no others, and a class that is not in the table was no
// faster than the kernels below, so no larger one stands in for it), tiles
// that fit LDS (with beta != 0 the old rows too).
bool once_serves(const tsg::Variant& v, int M, int N, const void* A, int64_t lda, const void* B, int64_t ldb,
                 bool beta_nz)
{
    if (M > v.maxM || N > v.maxN || M <= v.once_m || N <= v.once_n) return false;
    const size_t es = elem_bytes((tsg_dtype)v.dt);
    auto reads = [&](int W, const void* p, int64_t ld) {
        return aligned(p, 16) && (ld == W || (W * es % 16 == 0 && ld * es % 16 == 0 &&
                                              ld < (int64_t)((size_t)1 << 31) / (int64_t)(es * v.once)));
    };
    return reads(M, A, lda) && reads(N, B, ldb) && lds_for(v, M, N, beta_nz) <= kLdsBytes;
}

const tsg::Variant* pick_once(int dt, int M, int N, const void* A, int64_t lda, const void* B, int64_t ldb,
                              bool beta_nz, int64_t K)
{
    // the narrow non-square pairs in binary64 have kernels of their exact
    // widths, which multiply no zeros (2^22 rows, 4 x 8: 71 us there, 69 here;
    // 4 x 4, on the matrix cores both times: 52 and 46)
    if (M <= 8 && N <= 8 && M != N && (dt == TSG_R64 || dt == TSG_C128)) return nullptr;
    const tsg::Variant* v = VariantIndex::get().type(tsg::OP_TSMM, dt).once[M * VariantIndex::kW + N];
    if (!v || !once_serves(*v, M, N, A, lda, B, ldb, beta_nz)) return nullptr;
    // Few rows: a wave's chain of load, multiply, exchange and store is what the
    // call takes, and tiles of several 16 rows make it longer than in the
    // kernels with more and smaller waves: 30000 rows, tiles of 64 in binary32
    // 15 x 15 5.0 -> 6.7 us, 32 x 16 5.2 -> 10.0 (300000 rows 28 -> 20); tiles of
    // 16 rows gain at any length (doubles 12 x 40, 10007 rows: 8.2 -> 4.3), but
    // for the old rows of an update of a few (complex64 20 x 20, 10007 rows:
    // 5.4 -> 6.5, 30000: 7.7 -> 6.0).
    const int64_t tiles = K / v->once;
    if (v->once > 16 ? tiles < (beta_nz && v->once > 32 ? 6144 : 4096) : beta_nz && tiles < 1024) return nullptr;
    const int call = (M == v->maxM && N == v->maxN ? 2 : 1) * (beta_nz ? 4 : 1);
    return v->once_for & call ? v : nullptr;
}

const tsg::Variant* pick_for(int op, int dt, int M, int N, const void* A, int64_t lda, const void* X,
                             int64_t ldx, bool beta_nz, int64_t K)
{
    const bool a_pairs = (lda % 2 == 0) && aligned(A, 16);
    const bool x_pairs = (ldx % 2 == 0) && aligned(X, 16);
    // slab reads: the rows of A (TSMTTSM: and of B) are one contiguous run
    const bool rows_contiguous = lda == M && (op != tsg::OP_TSMTTSM || ldx == N);
    const bool ax16 = aligned(A, 16) && aligned(X, 16);
    if (!g_force.empty()) {
        for (int i = 0; i < tsg::kNumVariants; ++i) {
            const tsg::Variant& v = tsg::kVariants[i];
            if (g_force != v.name) continue;
            if (v.stage) return v.op == op && v.dt == dt && stage_serves(v, M, N, A, lda, X, ldx) ? &v : nullptr;
            if (v.once) return v.op == op && v.dt == dt && once_serves(v, M, N, A, lda, X, ldx, beta_nz) ? &v : nullptr;
            const bool serves = (v.M == M && v.N == N) || (v.M == 0 && M <= v.maxM && N <= v.maxN);
            if (v.op == op && v.dt == dt && serves && (!v.pairA || a_pairs) && (!v.pairX || x_pairs) &&
                (!v.flatA || rows_contiguous) && (!v.readB || beta_nz) && (!v.align16 || ax16))
                return &v;
        }
        return nullptr;
    }
    if (op == tsg::OP_TSMTTSM)
        if (const tsg::Variant* v = pick_stage(dt, M, N, A, lda, X, ldx, K)) return v;
    if (op == tsg::OP_TSMM)
        if (const tsg::Variant* v = pick_once(dt, M, N, A, lda, X, ldx, beta_nz, K)) return v;
    auto can = [&](const tsg::Variant& v) {
        return (!v.pairA || a_pairs) && (!v.pairX || x_pairs) && (!v.flatA || rows_contiguous) &&
               (!v.readB || beta_nz) && (!v.align16 || ax16);
    };
    const VariantIndex::PerType& t = VariantIndex::get().type(op, dt);
    auto covers = [&](const tsg::Variant& v) {
        return M <= v.maxM && N <= v.maxN && (!v.evenW || (M % 2 == 0 && N % 2 == 0)) && can(v);
    };
    // wide complex B += A C: a kernel that reads the old B along with A, of
    // these widths or, where their own would spill, of a range (2^20 rows,
    // 33 x 33 625 -> 369 us, 48 x 48 728 -> 456, 16 x 40 583 -> 299)
    if (op == tsg::OP_TSMM && beta_nz && (dt == TSG_C128 || dt == TSG_C64) && (M > 16 || N > 16)) {
        for (const tsg::Variant* v : t.exact[M * VariantIndex::kW + N])
            if (v->readB && can(*v)) return v;
        for (const tsg::Variant* v : t.ranges)
            if (v->readB && covers(*v)) return v;
    }
    for (const tsg::Variant* v : t.exact[M * VariantIndex::kW + N])
        if (can(*v)) return v;
    for (const tsg::Variant* v : t.ranges)
        if (covers(*v)) return v;
    return nullptr;
}

// The workspace of (dev, stream), `bytes` of it at least, as it is now: another
// thread may grow it at any time, and an outgrown one stays valid.
tsg_status get_workspace(int dev, hipStream_t stream, size_t bytes, Workspace* out)
{
    std::lock_guard<std::mutex> lk(g_mu);
    const char* lim = getenv("TSG_MAX_WORKSPACE");
    if (lim && bytes > (size_t)strtoull(lim, nullptr, 10))
        return fail(TSG_E_NOMEM, "workspace of %zu bytes exceeds TSG_MAX_WORKSPACE=%s", bytes, lim);
    const auto key = std::make_pair(dev, stream);
    Workspace& w = g_ws[key];
    if (w.data && w.bytes >= bytes) {
        *out = w;
        return TSG_OK;
    }
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
        return fail(TSG_E_CAPTURE, "workspace must grow to %zu bytes while the stream is captured; "
                                   "run the call once before capture or use tsg_reserve", bytes);
    hipError_t e;
    // the outgrown buffer is retired, not freed (see g_retired)
    const size_t grow = bytes < (1u << 20) ? (1u << 20) : bytes;
    Workspace fresh;
    fresh.bytes = grow;
    fresh.calls = &g_ws_calls[key];
    g_retired.reserve(g_retired.size() + 1);
    e = hipMalloc(&fresh.data, grow + 256);
    if (e != hipSuccess) return fail(TSG_E_NOMEM, "hipMalloc(%zu): %s", grow + 256, hipGetErrorString(e));
    hipLaunchKernelGGL(tsg::clear_counter, dim3(1), dim3(64), 0, stream, fresh.counter());
    if ((e = hipGetLastError()) != hipSuccess) {
        hipFree(fresh.data);
        return fail(TSG_E_HIP, "clearing a workspace's counter: %s", hipGetErrorString(e));
    }
    if (w.data) g_retired.emplace_back(dev, w.data);
    *out = w = fresh;
    return TSG_OK;
}

tsg_status validate(tsg_dtype dt, int64_t K, int32_t M, int32_t N, const void* A, int64_t lda, const void* X,
                    int64_t ldx, const void* Y, int64_t ldy, int op)
{
    if (elem_bytes(dt) == 0) return fail(TSG_E_ARG, "unknown dtype %d", (int)dt);
    if (K < 0) return fail(TSG_E_ARG, "K = %lld < 0", (long long)K);
    if (M < 1 || N < 1) return fail(TSG_E_ARG, "M = %d, N = %d: widths must be >= 1", M, N);
    if (M > kMaxWidth || N > kMaxWidth)
        return fail(TSG_E_UNSUPPORTED, "M = %d, N = %d: widths above %d are not supported", M, N, kMaxWidth);
    const size_t es = elem_bytes(dt);
    if (op == tsg::OP_TSMTTSM) {
        // A (K x M), X = B (K x N), Y = C (M x N)
        if (lda < M) return fail(TSG_E_ARG, "lda = %lld < M = %d", (long long)lda, M);
        if (ldx < N) return fail(TSG_E_ARG, "ldb = %lld < N = %d", (long long)ldx, N);
        if (ldy < N) return fail(TSG_E_ARG, "ldc = %lld < N = %d", (long long)ldy, N);
        if (!Y) return fail(TSG_E_ARG, "C is NULL");
        if (K > 0 && (!A || !X)) return fail(TSG_E_ARG, "A or B is NULL");
        if ((A && !aligned(A, es)) || (X && !aligned(X, es)))
            return fail(TSG_E_ARG, "A and B must be aligned to %zu bytes", es);
        if (!aligned(Y, is_complex(dt) ? 16 : 8)) return fail(TSG_E_ARG, "C must be aligned to its element size");
    } else {
        // A (K x M), X = C (M x N), Y = B (K x N)
        if (lda < M) return fail(TSG_E_ARG, "lda = %lld < M = %d", (long long)lda, M);
        if (ldx < N) return fail(TSG_E_ARG, "ldc = %lld < N = %d", (long long)ldx, N);
        if (ldy < N) return fail(TSG_E_ARG, "ldb = %lld < N = %d", (long long)ldy, N);
        if (K > 0 && (!A || !X || !Y)) return fail(TSG_E_ARG, "A, B or C is NULL");
        if ((A && !aligned(A, es)) || (Y && !aligned(Y, es)))
            return fail(TSG_E_ARG, "A and B must be aligned to %zu bytes", es);
        if (X && !aligned(X, is_complex(dt) ? 16 : 8)) return fail(TSG_E_ARG, "C must be aligned to its element size");
    }
    return TSG_OK;
}

int grid_for(int dev, const tsg::Variant& v, int64_t K, int M, int N, int cus, bool beta_nz = false)
{
    if (v.stage == 2) {
        // a matrix with itself: the grid of two matrices of its width, whose
        // kernel has the same stages and row groups, so that A^T A is summed
        // in the order of A^T B (that kernel needs more registers and LDS)
        const int gauss = stage_gauss(v.dt, M, N);
        for (const tsg::Variant* w : VariantIndex::get().type(tsg::OP_TSMTTSM, v.dt).stage)
            if (w->stage == 1 && w->gauss == gauss && w->maxM == v.maxM && w->maxN == v.maxN)
                return grid_for(dev, *w, K, M, N, cus);
    }
    int64_t rows = v.rows_per_tile;
    if (v.pack == 1) rows *= 16 / (M > N ? M : N);
    if (v.pack == 2) rows *= 16 / N;
    const int64_t tiles = (K + rows - 1) / rows;
    // the one-tile kernel of TSMM: a block for every tile, as many as a launch
    // may have (fewer than 2^32 work items); its blocks stride over the rest
    const size_t lds = lds_for(v, M, N, beta_nz);
    const int blocks = v.once && !v.once_db && lds <= (64u << 10) ? 0 : occupancy(dev, v, lds);
    const int64_t cap = v.once && !v.once_db ? (((int64_t)1 << 32) - 1) / v.threads : (int64_t)cus * blocks;
    int64_t g = tiles < cap ? tiles : cap;
    if (v.op == tsg::OP_TSMTTSM) {
        // the per-block partial sums of a launch always fit the no-alloc
        // scratch, so both TSMTTSM entry points run the same grid (and give
        // the same bits) for every shape
        const int64_t E = (int64_t)M * N * (is_complex((tsg_dtype)v.dt) ? 2 : 1);
        const int64_t gmax = (int64_t)(tsg::kScratchBytes / (E * sizeof(double)));
        if (g > gmax) g = gmax;
    }
    if (g_grid_cap > 0 && g > g_grid_cap) g = g_grid_cap;
    return g < 1 ? 1 : (int)g;
}

size_t tsmttsm_ws_bytes(int grid, int M, int N, bool cplx)
{
    const size_t E = (size_t)M * N * (cplx ? 2 : 1);
    return grid > 1 ? (size_t)grid * E * sizeof(double) : 0;
}

// Launch the fold of the per-block partials (grid > 1) into C.
hipError_t launch_fold(const tsg::Launch& p, bool cplx)
{
    const int E = p.M * p.N * (cplx ? 2 : 1);
    int eb = 1;
    while (eb < E && eb < 8) eb <<= 1;
    const int blocks = (E + eb - 1) / eb;
    if (cplx)
        hipLaunchKernelGGL((tsg::fold_partials<2>), dim3(blocks), dim3(tsg::kFoldThreads), 0, p.stream, p.ws, p.grid,
                           E, eb, p.N, static_cast<double*>(p.Y), p.ldy);
    else
        hipLaunchKernelGGL((tsg::fold_partials<1>), dim3(blocks), dim3(tsg::kFoldThreads), 0, p.stream, p.ws, p.grid,
                           E, eb, p.N, static_cast<double*>(p.Y), p.ldy);
    return hipGetLastError();
}

// Whether the kernel sums over its blocks itself (block_sum) instead of
// leaving it to fold_partials: few blocks with few partial sums, where the
// launch saved is more than one compute unit's reading of them.  Calls in a
// row, two launches -> one: 10007 x 4 and 4 (20 blocks, 3 KB) 6.0 -> 4.6 us,
// complex 8 and 8 (40 blocks, 40 KB) 6.6 -> 6.2; on the other side 40000 x 8
// and 8 (79 blocks, 40 KB) 6.35 and 6.40, 10007 x 16 and 4 (157 blocks, 80 KB)
// 7.1 and 8.1, 200000 x 2 and 2 (196 blocks, 6 KB) 5.8 and 6.6.
//
// Launches that count together must not overlap, not even by mistake: a count
// left over would spoil every later one.  So only where the stream orders
// them: not in a graph (replayed anywhere), not in the no-alloc calls (one
// scratch for all streams), not on the handle of the per-thread streams.
constexpr int kSelfSumBlocks = 64;
constexpr size_t kSelfSumBytes = 40960;

bool sums_itself(const tsg::Variant& v, int grid, size_t bytes, hipStream_t stream)
{
    if (!v.sums || grid <= 1 || grid > kSelfSumBlocks || bytes > kSelfSumBytes || g_reduction != TSG_REDUCE_FOLD ||
        stream == hipStreamPerThread)
        return false;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    return stream == nullptr || (hipStreamIsCapturing(stream, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone);
}

// TSMTTSM launch shared by tsg_tsmttsm (per-stream workspace, allocated on
// first need) and tsg_tsmttsm_noalloc (the device's fixed scratch array).
tsg_status tsmttsm_call(tsg_dtype dt, tsg_op op, int64_t K, int32_t M, int32_t N, const void* A, int64_t lda,
                        const void* B, int64_t ldb, void* C, int64_t ldc, void* stream, bool noalloc)
{
    g_err.clear();
    if (op != TSG_OP_T && op != TSG_OP_C) return fail(TSG_E_ARG, "unknown op %d", (int)op);
    tsg_status s = validate(dt, K, M, N, A, lda, B, ldb, C, ldc, tsg::OP_TSMTTSM);
    if (s != TSG_OK) return s;
    int dev;
    if ((s = current_device(&dev)) != TSG_OK) return s;
    DeviceInfo di;
    if ((s = device_info(dev, &di)) != TSG_OK) return s;
    const tsg::Variant* v = pick(tsg::OP_TSMTTSM, dt, M, N, A, lda, B, ldb, false, K);
    if (!v) return fail(TSG_E_UNSUPPORTED, "no kernel variant for TSMTTSM %dx%d%s", M, N,
                        g_force.empty() ? "" : " (a forced variant does not apply)");
    tsg::Launch p{};
    p.stream = static_cast<hipStream_t>(stream);
    p.grid = grid_for(dev, *v, K, M, N, di.cus);
    p.K = K;
    p.M = M;
    p.N = N;
    p.conj = (op == TSG_OP_C && is_complex(dt)) ? 1 : 0;
    p.A = A;
    p.lda = lda;
    p.X = B;
    p.ldx = ldb;
    p.Y = C;
    p.ldy = ldc;
    const size_t need = tsmttsm_ws_bytes(p.grid, M, N, is_complex(dt));
    std::unique_lock<std::mutex> calls;
    if (noalloc) {
        if (need > tsg::kScratchBytes)
            return fail(TSG_E_UNSUPPORTED, "TSMTTSM %dx%d on %d blocks needs %zu bytes of partial sums, more than "
                        "the %zu bytes of the no-alloc scratch", M, N, p.grid, need, tsg::kScratchBytes);
        if ((s = scratch_of(dev, &p.ws)) != TSG_OK) return s;
    } else {
        Workspace w;
        if ((s = get_workspace(dev, p.stream, need, &w)) != TSG_OK) return s;
        p.ws = w.slots();
        if (sums_itself(*v, p.grid, need, p.stream)) p.arrived = w.counter();
        calls = std::unique_lock<std::mutex>(*w.calls);
    }
    p.lds = lds_for(*v, M, N);
    if ((s = lds_ready(dev, *v, p.lds)) != TSG_OK) return s;
    v->launch(p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(TSG_E_HIP, "launch of %s: %s", v->name, hipGetErrorString(e));
    if (p.arrived) return TSG_OK;
    if (p.grid > 1 && g_reduction == TSG_REDUCE_ATOMIC) {
        const int cw = is_complex(dt) ? 2 : 1;
        const int E = M * N * cw;
        double* Cd = static_cast<double*>(C);
        hipLaunchKernelGGL(tsg::clear_small, dim3((E + 255) / 256), dim3(256), 0, p.stream, Cd, M, N, cw, ldc);
        const int64_t n = (int64_t)p.grid * E;
        if (cw == 2)
            hipLaunchKernelGGL((tsg::atomic_partials<2>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, p.stream,
                               p.ws, p.grid, E, N, Cd, ldc);
        else
            hipLaunchKernelGGL((tsg::atomic_partials<1>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, p.stream,
                               p.ws, p.grid, E, N, Cd, ldc);
        if ((e = hipGetLastError()) != hipSuccess)
            return fail(TSG_E_HIP, "launch of the atomic reduction: %s", hipGetErrorString(e));
        return TSG_OK;
    }
    if (p.grid > 1 && g_reduction == TSG_REDUCE_NONE) return TSG_OK;  // ablation: partials left in the workspace
    if (p.grid > 1 && (e = launch_fold(p, is_complex(dt))) != hipSuccess)
        return fail(TSG_E_HIP, "launch of the partial fold: %s", hipGetErrorString(e));
    return TSG_OK;
}

}  // namespace

extern "C" {

tsg_status tsg_tsmttsm(tsg_dtype dt, tsg_op op, int64_t K, int32_t M, int32_t N, const void* A, int64_t lda,
                       const void* B, int64_t ldb, void* C, int64_t ldc, void* stream)
try {
    return tsmttsm_call(dt, op, K, M, N, A, lda, B, ldb, C, ldc, stream, false);
} catch (...) {
    return no_memory(TSG_E_NOMEM);
}

tsg_status tsg_tsmttsm_noalloc(tsg_dtype dt, tsg_op op, int64_t K, int32_t M, int32_t N, const void* A,
                               int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc, void* stream)
try {
    return tsmttsm_call(dt, op, K, M, N, A, lda, B, ldb, C, ldc, stream, true);
} catch (...) {
    return no_memory(TSG_E_NOMEM);
}

tsg_status tsg_tsmm_op(tsg_dtype dt, int32_t conjA, tsg_op opC, int64_t K, int32_t M, int32_t N, const void* A,
                       int64_t lda, const void* C, int64_t ldc, void* B, int64_t ldb, double alpha, double beta,
                       void* stream)
try {
    g_err.clear();
    if (opC != TSG_OP_N && opC != TSG_OP_T && opC != TSG_OP_C) return fail(TSG_E_ARG, "unknown opC %d", (int)opC);
    if (opC != TSG_OP_N && M >= 1 && ldc < M)
        return fail(TSG_E_ARG, "ldc = %lld < M = %d for a transposed small matrix", (long long)ldc, M);
    const int64_t ldc_check = opC == TSG_OP_N ? ldc : (ldc > N ? ldc : (int64_t)N);
    tsg_status s = validate(dt, K, M, N, A, lda, C, ldc_check, B, ldb, tsg::OP_TSMM);
    if (s != TSG_OK) return s;
    if (K == 0) return TSG_OK;
    int dev;
    if ((s = current_device(&dev)) != TSG_OK) return s;
    DeviceInfo di;
    if ((s = device_info(dev, &di)) != TSG_OK) return s;
    const tsg::Variant* v = pick(tsg::OP_TSMM, dt, M, N, A, lda, B, ldb, beta != 0.0, K);
    if (!v) return fail(TSG_E_UNSUPPORTED, "no kernel variant for TSMM %dx%d%s", M, N,
                        g_force.empty() ? "" : " (a forced variant does not apply)");
    tsg::Launch p{};
    p.stream = static_cast<hipStream_t>(stream);
    p.grid = grid_for(dev, *v, K, M, N, di.cus, beta != 0.0);
    p.K = K;
    p.M = M;
    p.N = N;
    p.conj = (conjA && is_complex(dt)) ? 1 : 0;
    p.opc = opC == TSG_OP_N ? 0 : ((opC == TSG_OP_C && is_complex(dt)) ? 2 : 1);
    p.A = A;
    p.lda = lda;
    p.X = C;
    p.ldx = ldc;
    p.Y = B;
    p.ldy = ldb;
    p.alpha = alpha;
    p.beta = beta;
    p.lds = lds_for(*v, M, N, beta != 0.0);
    if ((s = lds_ready(dev, *v, p.lds)) != TSG_OK) return s;
    v->launch(p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(TSG_E_HIP, "launch of %s: %s", v->name, hipGetErrorString(e));
    return TSG_OK;
} catch (...) {
    return no_memory(TSG_E_NOMEM);
}

tsg_status tsg_tsmm(tsg_dtype dt, int32_t conjA, int64_t K, int32_t M, int32_t N, const void* A, int64_t lda,
                    const void* C, int64_t ldc, void* B, int64_t ldb, double alpha, double beta, void* stream)
{
    return tsg_tsmm_op(dt, conjA, TSG_OP_N, K, M, N, A, lda, C, ldc, B, ldb, alpha, beta, stream);
}

size_t tsg_workspace_size(int32_t op_kind, tsg_dtype dt, int64_t K, int32_t M, int32_t N, int32_t count)
try {
    if (op_kind == TSG_KIND_TSMM) return 0;
    if (op_kind == TSG_KIND_ORTH) return dt == TSG_R64 ? tsg::orth_workspace_size(K, M, N, count) : 0;
    if (op_kind != TSG_KIND_TSMTTSM) return 0;
    if (M < 1 || N < 1 || M > kMaxWidth || N > kMaxWidth || K < 0) return 0;
    int dev;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    DeviceInfo di;
    if (device_info(dev, &di) != TSG_OK) return 0;
    // the larger need of contiguous and of padded rows (aligned matrices; one
    // with itself runs the grid of two)
    alignas(16) static const char buf16[32] = {0};
    size_t need = 0;
    for (int pad = 0; pad < 2; ++pad) {
        const tsg::Variant* v = pick(tsg::OP_TSMTTSM, dt, M, N, buf16, M + pad * (M & 1), buf16 + 16, N + pad * (N & 1), false, K);
        if (!v) continue;
        const size_t b = tsmttsm_ws_bytes(grid_for(dev, *v, K, M, N, di.cus), M, N, is_complex(dt));
        need = need > b ? need : b;
    }
    return need;
} catch (...) {
    return no_memory((size_t)0);
}

tsg_status tsg_reserve(tsg_dtype dt, int64_t K, int32_t M, int32_t N, void* stream)
try {
    g_err.clear();
    if (M < 1 || N < 1 || K < 0) return fail(TSG_E_ARG, "invalid shape");
    if (M > kMaxWidth || N > kMaxWidth) return fail(TSG_E_UNSUPPORTED, "widths above %d", kMaxWidth);
    int dev;
    tsg_status s = current_device(&dev);
    if (s != TSG_OK) return s;
    DeviceInfo di;
    if ((s = device_info(dev, &di)) != TSG_OK) return s;
    // the largest grid any TSMTTSM variant of this shape may use, of the type
    // or of the binary64-arithmetic one whose kernels serve it too
    size_t need = 0;
    for (int i = 0; i < tsg::kNumVariants; ++i) {
        const tsg::Variant& v = tsg::kVariants[i];
        if (v.op != tsg::OP_TSMTTSM || (v.dt != (int)dt && v.dt != twin_of(dt))) continue;
        if (v.stage) {
            const int wide = M > N ? M : N, narrow = M > N ? N : M;
            if (v.maxM != (wide + 15) / 16 * 16 || v.maxN != (narrow + 3) / 4 * 4 || (v.stage == 2 && M != N)) continue;
        } else if (!((v.M == M && v.N == N) || (v.M == 0 && M <= v.maxM && N <= v.maxN))) continue;
        size_t b = tsmttsm_ws_bytes(grid_for(dev, v, K, M, N, di.cus), M, N, is_complex(dt));
        if (b > need) need = b;
    }
    Workspace w;
    return get_workspace(dev, static_cast<hipStream_t>(stream), need, &w);
} catch (...) {
    return no_memory(TSG_E_NOMEM);
}

tsg_status tsg_init(int32_t device)
try {
    g_err.clear();
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess || n == 0) return fail(TSG_E_HIP, "no HIP device: %s", hipGetErrorString(e));
    if (device < 0 || device >= n) return fail(TSG_E_ARG, "device %d out of range [0, %d)", device, n);
    DeviceInfo di;
    tsg_status s = device_info(device, &di);
    if (s != TSG_OK) return s;
    // the no-alloc scratch address of `device`, resolved with it current
    int cur = -1;
    if ((e = hipGetDevice(&cur)) != hipSuccess) return fail(TSG_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (cur != device && (e = hipSetDevice(device)) != hipSuccess)
        return fail(TSG_E_HIP, "hipSetDevice(%d): %s", device, hipGetErrorString(e));
    double* ws = nullptr;
    s = scratch_of(device, &ws);
    if (cur != device) hipSetDevice(cur);
    return s;
} catch (...) {
    return no_memory(TSG_E_NOMEM);
}

void tsg_finalize(void)
{
    std::lock_guard<std::mutex> lk(g_mu);
    int cur = -1;
    hipGetDevice(&cur);
    for (auto& kv : g_ws) {
        hipSetDevice(kv.first.first);
        if (kv.second.data) hipFree(kv.second.data);
    }
    g_ws.clear();
    for (auto& r : g_retired) {
        hipSetDevice(r.first);
        hipFree(r.second);
    }
    g_retired.clear();
    g_occ.clear();
    g_lds.clear();
    if (cur >= 0) hipSetDevice(cur);
}

const char* tsg_status_string(tsg_status s)
{
    switch (s) {
    case TSG_OK: return "TSG_OK";
    case TSG_E_ARG: return "TSG_E_ARG: invalid argument";
    case TSG_E_UNSUPPORTED: return "TSG_E_UNSUPPORTED: outside the supported range";
    case TSG_E_NOMEM: return "TSG_E_NOMEM: workspace allocation failed";
    case TSG_E_HIP: return "TSG_E_HIP: HIP runtime error";
    case TSG_E_CAPTURE: return "TSG_E_CAPTURE: workspace cannot grow during stream capture";
    }
    return "unknown tsg_status";
}

const char* tsg_last_error(void) { return g_err.c_str(); }

tsg_status tsg_force_variant(const char* name)
try {
    g_err.clear();
    if (!name || !*name) {
        g_force.clear();
        return TSG_OK;
    }
    for (int i = 0; i < tsg::kNumVariants; ++i)
        if (!strcmp(tsg::kVariants[i].name, name)) {
            g_force = name;
            return TSG_OK;
        }
    return fail(TSG_E_ARG, "no kernel variant named %s", name);
} catch (...) {
    return no_memory(TSG_E_NOMEM);
}

tsg_status tsg_set_grid_limit(int32_t blocks)
{
    g_err.clear();
    if (blocks < 0) return fail(TSG_E_ARG, "grid limit %d < 0", blocks);
    g_grid_cap = blocks;
    return TSG_OK;
}

tsg_status tsg_set_reduction(int32_t mode)
{
    if (mode != TSG_REDUCE_FOLD && mode != TSG_REDUCE_ATOMIC && mode != TSG_REDUCE_NONE)
        return fail(TSG_E_ARG, "unknown reduction mode %d", (int)mode);
    g_reduction = mode;
    return TSG_OK;
}

int32_t tsg_variant_count(void) { return tsg::kNumVariants; }

const char* tsg_variant_name(int32_t i) { return (i >= 0 && i < tsg::kNumVariants) ? tsg::kVariants[i].name : ""; }

const char* tsg_kernel_name(int32_t op_kind, tsg_dtype dt, int32_t conj, int32_t M, int32_t N)
try {
    (void)conj;
    if (op_kind != 0 && op_kind != 1) return "";
    if (M < 1 || N < 1 || M > kMaxWidth || N > kMaxWidth) return "";
    alignas(16) static const char buf16[32] = {0};
    // contiguous rows (lda = M, ldb = N), two 16-byte aligned operands
    const tsg::Variant* v = pick(op_kind, dt, M, N, buf16, M, buf16 + 16, N);
    return v ? v->name : "";
} catch (...) {
    return no_memory("");
}

}  // extern "C"
