// Device code of the AVU-GSR LSQR library for gfx950 (CDNA4, wave64).
//
// The matrix is the paper's dense per-row coefficient array A_d (Sect. 2)
// held as structure-of-arrays: coefficient c of row i at values[c*m + i], so
// that a wave streams 64 consecutive rows of one coefficient as one coalesced
// 512-byte (FP64) or 256-byte (FP32) request. Index arrays follow the same
// layout. Streaming loads carry the nontemporal hint so that the matrix does not
// evict the gathered vector sections from L2, except where the last-level cache
// holds the matrix from one iteration to the next (kPlain).
//
// Kernels:
//   k_aprod1      y = A x (+ mode-specific update), one row per lane, grid
//                 stride; FP64 sum of squares of the written y per block (the
//                 beta norm of the LSQR step).
//   k_aprod2      x += A^T y over star-aligned per-wave row ranges:
//                   astrometric: segmented reduction over the star key (rows
//                     are sorted by star), plain stores, no atomics;
//                   attitude: left to the bucket-order pass (k_att_hist +
//                     k_slice_reduce: rows sorted by the bucket of their
//                     attitude start, per-workgroup FP64 LDS histograms, no
//                     device atomics) by default; scatter-add with device
//                     atomics in the ATT instances (attitude mode 0);
//                   instrumental: workgroup-private LDS histogram, flushed
//                     once per workgroup (k_instr_tail beyond its columns);
//                   global: wave shuffle -> LDS -> per-workgroup partial,
//                     summed in a deterministic second stage.
//   k_fused       one sweep doing aprod1 and aprod2 of an LSQR step, with both
//                 histograms in LDS where they fit, else without the attitude
//                 section (k_att_dot before and k_att_hist after it, in bucket
//                 order).
//   k_col_a/b     column-vector updates of the LSQR step (FP64), with the norms
//                 and the Givens rotation in every workgroup; the estimates and
//                 stopping tests run in the next row pass.
//   k_scalar_*    single-workgroup kernels: the norms at the start, the tests
//                 after a launch's last iteration, all FP64.
//   namespace batched: the same steps for a k-tile of right-hand sides.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace avugsr {

constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;

// Row layout of the paper (Sect. 2): 5 astrometric, 3 axes x 4 attitude,
// 6 instrumental, 1 global coefficient.
constexpr int kAstro = 5;
constexpr int kAxes = 3;
constexpr int kParAxis = 4;
constexpr int kInstr = 6;
constexpr int kPar = 24;
constexpr int kOffAtt = kAstro;
constexpr int kOffInstr = kAstro + kAxes * kParAxis;
constexpr int kOffGlob = kOffInstr + kInstr;
static_assert(kOffGlob + 1 == kPar, "row layout");

constexpr int64_t kNoStar = INT64_MAX;

struct SysView {
    const void* val;       // [kPar][m]
    const int64_t* star;   // [m]
    const int64_t* att;    // [m]
    const int32_t* instr;  // [kInstr][m]
    int64_t m;
    int64_t n;
    int64_t n_stars;
    int64_t n_dfa;
    int64_t n_instr_cols;
    int64_t att_base;
    int64_t instr_base;
    int64_t glob_base;
    // section sizes and value-row offsets (general layouts; the full layout
    // is 5, 12, 6, 1 at offsets 5, 17, 23)
    int32_t na, natt, ni, ng;
    int32_t off_att, off_instr, off_glob;
    // compact copies of the star and instrumental indices read by the fused
    // passes (CIDX), or null
    const int32_t* star32;    // [m]
    const uint16_t* instr16;  // [kInstr][m]
};

// LSQR state kept on the device so that a whole iteration runs without a
// host round trip (and can be captured into a graph).
struct Scalars {
    double alpha, beta, rhobar, phibar, bnorm;
    double anorm, ddnorm, xnorm, rnorm, arnorm, acond;
    double rho, c, s, theta, phi;
    double t1, t2, inv_alpha, coef_u;
    double atol, btol, ctol;
    double dmax, xmax;  // refinement: ||d||_inf, ||x||_inf of the last outer step
    double arnorm0;     // alpha_1 beta_1 = ||Abar^T b||, the initial normal-equation residual
    double rel_ar;      // > 0: also stop (istop 2) once arnorm <= rel_ar * arnorm0
    int32_t itn, itn_limit, istop, done;
    int32_t tests, beta_zero, pad0, pad1;
};

template <typename T>
__device__ __forceinline__ T ldnt(const T* p)
{
    return __builtin_nontemporal_load(p);
}

// A load of a streamed column: nontemporal, or PLAIN where the columns do not
// start on a 128-byte line, so that the line a wave's step shares with its
// next step stays in L2 until that step reads it (nontemporal lines go
// first: at 1e9 rows, m = 8 mod 16, about 2-3 ms less per instrumental tail
// window of 10.7-11.4 ms; with aligned columns plain loads gain nothing).
template <bool PLAIN, typename T>
__device__ __forceinline__ T ld_stream(const T* p)
{
    if constexpr (PLAIN)
        return *p;
    else
        return ldnt(p);
}

// base[i], i small and per lane, base the same over the wave (in scalar
// registers): the address takes one vector register, not two per column.
template <bool PLAIN = false, typename T>
__device__ __forceinline__ T ld_off(const T* base, uint32_t i)
{
    return ld_stream<PLAIN>(reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) +
                                                       (uint32_t)(i * sizeof(T))));
}

// A value that is the same over the wave, moved to scalar registers.
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v)
{
    const int32_t lo = uniform((int32_t)v), hi = uniform((int32_t)(v >> 32));
    return (int64_t)(uint32_t)lo | ((int64_t)hi << 32);
}

// Star and instrumental index of row ic, from the compact copies when CIDX.
template <bool CIDX, bool PLAIN = false>
__device__ __forceinline__ int64_t star_of(const SysView& s, int64_t ic)
{
    return CIDX ? (int64_t)ld_stream<PLAIN>(&s.star32[ic]) : ld_stream<PLAIN>(&s.star[ic]);
}
template <bool CIDX, bool PLAIN = false>
__device__ __forceinline__ int32_t instr_of(const SysView& s, int j, int64_t ic)
{
    return CIDX ? (int32_t)ld_stream<PLAIN>(&s.instr16[j * s.m + ic])
                : ld_stream<PLAIN>(&s.instr[j * s.m + ic]);
}

// ---------------------------------------------------------------- reductions
// Deterministic block sum of one double per thread; result valid on thread 0.
__device__ __forceinline__ double block_sum(double v, double* lds /* >= kWavesPerBlock */)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) lds[w] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < kWavesPerBlock; ++k) r += lds[k];
    return r;
}

__device__ __forceinline__ double block_max(double v, double* lds)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v = fmax(v, __shfl_down(v, off));
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) lds[w] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < kWavesPerBlock; ++k) r = fmax(r, lds[k]);
    return r;
}

template <int NT>
__device__ __forceinline__ double block_sum_n(double v, double* lds /* >= NT / kWave */)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) lds[w] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < NT / kWave; ++k) r += lds[k];
    return r;
}

// Sum of n partials by one block, fixed order (deterministic). Thread 0.
__device__ __forceinline__ double sum_partials(const double* part, int n, double* lds)
{
    double v = 0.0;
    for (int k = threadIdx.x; k < n; k += kBlock) v += part[k];
    return block_sum(v, lds);
}

__device__ __forceinline__ double max_partials(const double* part, int n, double* lds)
{
    double v = 0.0;
    for (int k = threadIdx.x; k < n; k += kBlock) v = fmax(v, part[k]);
    return block_max(v, lds);
}

// ------------------------------------------------------- histogram slices
// The LDS histograms of a section, one slice per workgroup: slice of bucket b's
// workgroup g at S[((b G + g) K + r) naxes span + axis span + off], column
// b width + off of an axis of len columns (off < span; with several buckets
// span > width, so that a column lies in the windows of at most two). gl threads share
// the G slices of one column.
struct SliceView {
    const double* S;
    int64_t nb, width, span, len, base;
    int32_t naxes, G, gl;
    __device__ __host__ int64_t cols() const { return naxes * len; }
    __device__ __host__ int ct() const { return kBlock / gl; }  // columns per tile
    __device__ __host__ int64_t tiles() const { return (cols() + ct() - 1) / ct(); }
};

// Sum of the slices of column `col` (axis-major within the section) and
// right-hand side r, valid on threads [0, ct): a tile of ct columns, gl threads
// each taking every gl-th slice, then the gl partial sums in a fixed order.
// With one thread per column the sum is a serial chain of G loads: 44-59 us
// for one bucket's 256 slices whatever the columns (n_dfa = 60 ... 10^4);
// all threads of the block call this.
template <int K>
__device__ __forceinline__ double slice_tile_sum(const SliceView& V, bool ok, int64_t col, int r,
                                                 double* red /* kBlock */)
{
    const int ct = V.ct(), g0 = threadIdx.x / ct;
    double sum = 0.0;
    if (ok) {
        int64_t c = col;
        int ax = 0;
        while (c >= V.len) {
            c -= V.len;
            ++ax;
        }
        const int64_t bq = c / V.width, bhi = bq < V.nb - 1 ? bq : V.nb - 1;
        const int64_t slice = (int64_t)K * V.naxes * V.span;
        for (int64_t bk = bhi; bk >= 0 && c - bk * V.width < V.span; --bk) {
            const double* p =
                V.S + bk * V.G * slice + ((int64_t)r * V.naxes + ax) * V.span + (c - bk * V.width);
            int g = g0;
            auto batch = [&](auto n) {  // n loads in flight
                constexpr int N = decltype(n)::value;
                for (; g + (N - 1) * V.gl < V.G; g += N * V.gl) {
                    double a[N];
#pragma unroll
                    for (int k = 0; k < N; ++k) a[k] = p[(g + k * V.gl) * slice];
#pragma unroll
                    for (int k = 0; k < N; ++k) sum += a[k];
                }
            };
            batch(std::integral_constant<int, 8>());
            batch(std::integral_constant<int, 4>());
            batch(std::integral_constant<int, 1>());
        }
    }
    if (V.gl == 1) return sum;
    __syncthreads();
    red[threadIdx.x] = sum;
    __syncthreads();
    if (g0 == 0)
        for (int l = 1; l < V.gl; ++l) sum += red[l * ct + threadIdx.x];
    return sum;
}

// Runs f(section, column, sum) for every column of the two slice sections, on
// the thread that holds its sum, and plain(j) for the other columns, tile by
// tile over the grid (the slice tiles first: they take longest). plain columns:
// [0, n) without the sections (att before ins).
template <typename F, typename P>
__device__ __forceinline__ void for_columns(const SliceView& att, const SliceView& ins, int64_t n,
                                            double* red /* kBlock */, F&& slice, P&& plain)
{
    const int64_t na = att.tiles(), ni = na + ins.tiles();
    const int64_t np = n - att.cols() - ins.cols();
    const int64_t nt = ni + (np + kBlock - 1) / kBlock;
    for (int64_t tile = blockIdx.x; tile < nt; tile += gridDim.x) {
        if (tile < ni) {
            const bool first = tile < na;
            const SliceView& V = first ? att : ins;
            const int64_t col =
                (first ? tile : tile - na) * V.ct() + (threadIdx.x & (V.ct() - 1));
            const bool ok = col < V.cols();
            const double sum = slice_tile_sum<1>(V, ok, col, 0, red);
            if (ok && threadIdx.x < V.ct()) slice(V.base + col, sum);
        } else {
            int64_t j = (tile - ni) * kBlock + threadIdx.x;
            if (j >= np) continue;
            if (j >= att.base) j += att.cols();
            if (j >= ins.base) j += ins.cols();
            plain(j);
        }
    }
}

// Partials of the global columns: gpart[blk stride + g], blk < nblk, g < ng.
struct GlobView {
    const void* part;
    int64_t base;
    int32_t nblk, stride, ng;
};

// f(column, sum of its partials) on thread 0 of the last block.
template <typename Acc, typename F>
__device__ __forceinline__ void for_globals(const GlobView& G, double* red, F&& f)
{
    if (blockIdx.x != gridDim.x - 1) return;
    const Acc* part = static_cast<const Acc*>(G.part);
    for (int g = 0; g < G.ng; ++g) {
        double v = 0.0;
        for (int k = threadIdx.x; k < G.nblk; k += kBlock)
            v += (double)part[(int64_t)k * G.stride + g];
        const double r = block_sum(v, red);
        if (threadIdx.x == 0) f(G.base + g, r);
    }
}

// q += the slices' sums and the global columns' partials (the last step of an
// aprod2 outside the iterations, where k_col_a does the same on the way).
template <typename Acc>
__global__ __launch_bounds__(kBlock) void k_section_sums(SliceView att, SliceView ins, GlobView glob,
                                                          Acc* __restrict__ q,
                                                          const Scalars* __restrict__ sc)
{
    __shared__ double red[kBlock];
    if (sc != nullptr && sc->done) return;
    auto add = [q](int64_t j, double sum) { q[j] = (Acc)((double)q[j] + sum); };
    for_columns(att, ins, att.cols() + ins.cols(), red, add, [](int64_t) {});
    for_globals<Acc>(glob, red, add);
}

// ------------------------------------------------------------ stopping tests
// ddnorm, xnorm, acond and the stopping tests of Paige & Saunders: what one
// iteration adds to the state s. (The state itself is not copied into
// registers: it would go through scratch.)
struct StopUpdate {
    double ddnorm, xnorm, acond;
    int32_t itn, istop, done;
};

__device__ __forceinline__ StopUpdate stop_update(const Scalars& s, double dd, double xx)
{
    StopUpdate o;
    const double ddnorm = s.ddnorm + dd;
    const double xnorm = sqrt(xx);
    const double anorm = s.anorm;
    const double acond = anorm * sqrt(ddnorm);
    const double rnorm = s.rnorm, arnorm = s.arnorm, bnorm = s.bnorm;
    o.ddnorm = ddnorm;
    o.xnorm = xnorm;
    o.acond = acond;
    o.itn = s.itn + 1;

    const double test1 = rnorm / bnorm;
    const double test2 = (anorm * rnorm) > 0.0 ? arnorm / (anorm * rnorm) : 0.0;
    const double test3 = acond > 0.0 ? 1.0 / acond : 0.0;
    const double t1 = test1 / (1.0 + anorm * xnorm / bnorm);
    const double rtol = s.btol + s.atol * anorm * xnorm / bnorm;
    int32_t istop = 0;
    if (o.itn >= s.itn_limit) istop = 7;
    if (s.tests) {
        if (1.0 + test3 <= 1.0) istop = 6;
        if (1.0 + test2 <= 1.0) istop = 5;
        if (1.0 + t1 <= 1.0) istop = 4;
        if (test3 <= s.ctol) istop = 3;
        if (test2 <= s.atol) istop = 2;
        if (test1 <= rtol) istop = 1;
    }
    // Relative form of the normal-equation test, for correction problems whose
    // residual is dominated by the irreducible least-squares residual.
    if (s.rel_ar > 0.0 && arnorm <= s.rel_ar * s.arnorm0) istop = 2;
    o.istop = istop;
    o.done = istop != 0 ? 1 : s.done;
    return o;
}

// *to = *from by the first threads of a block (the caller synchronises).
__device__ __forceinline__ void copy_state(Scalars* to, const Scalars* from)
{
    static_assert(sizeof(Scalars) % 4 == 0 && sizeof(Scalars) / 4 <= kBlock, "one word a thread");
    if (threadIdx.x < sizeof(Scalars) / 4)
        reinterpret_cast<uint32_t*>(to)[threadIdx.x] =
            reinterpret_cast<const uint32_t*>(from)[threadIdx.x];
}

// The stopping tests of the previous iteration, made by the first row pass of
// the next one. A single-workgroup kernel for them costs 4-5 us and a launch
// gap per iteration; here every workgroup sums the same partials in the same
// order beside staging its LDS, and workgroup 0 stores the state. The state is
// read from B (written by k_col_b) and stored to A, which no workgroup of this
// pass reads, so the order of the workgroups does not matter; the kernels that
// follow read A. B null: nothing pending, A is current.
struct Gate {
    const Scalars* B;
    Scalars* A;
    const double* dd;
    const double* xx;
    int32_t n;
};

// The gate's loads (each thread's partials, the state's flag), issued before
// the staging of LDS so that they arrive beside it.
struct GateIn {
    double dd, xx;
    int32_t done;
    double coef;
};

__device__ __forceinline__ GateIn gate_load(const Gate& G)
{
    GateIn in = {0.0, 0.0, 0, 0.0};
    const Scalars* s = G.B ? G.B : G.A;
    if (s == nullptr) return in;  // an operator, outside a solve
    if (G.B != nullptr && threadIdx.x < kBlock)
        for (int k = threadIdx.x; k < G.n; k += kBlock) {  // as sum_partials
            in.dd += G.dd[k];
            in.xx += G.xx[k];
        }
    in.done = s->done;
    in.coef = s->coef_u;
    return in;
}

// True while the solve runs (uniform over the block). red: 2 kWavesPerBlock.
// All threads of the block call this.
__device__ __forceinline__ bool gate_open(const Gate& G, const GateIn& in, double* red,
                                          int32_t* flag)
{
    if (in.done) return false;  // B pending: A was final already
    if (G.B == nullptr) return true;
    if (blockIdx.x == 0) copy_state(G.A, G.B);  // before the barriers of the sums
    double dd = in.dd, xx = in.xx;
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        dd += __shfl_down(dd, off);
        xx += __shfl_down(xx, off);
    }
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (lane == 0 && w < kWavesPerBlock) {
        red[w] = dd;
        red[kWavesPerBlock + w] = xx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sd = 0.0, sx = 0.0;
        for (int k = 0; k < kWavesPerBlock; ++k) {
            sd += red[k];
            sx += red[kWavesPerBlock + k];
        }
        const StopUpdate o = stop_update(*G.B, sd, sx);
        *flag = o.done;
        if (blockIdx.x == 0) {
            G.A->ddnorm = o.ddnorm;
            G.A->xnorm = o.xnorm;
            G.A->acond = o.acond;
            G.A->itn = o.itn;
            G.A->istop = o.istop;
            G.A->done = o.done;
        }
    }
    __syncthreads();
    return *flag == 0;
}

// dst[0, n) = src[0, n) by the block's NT threads, four loads in flight each.
template <int NT, typename V>
__device__ __forceinline__ void stage(V* dst, const V* src, int64_t n)
{
    for (int64_t j = threadIdx.x; j < n; j += 4 * NT) {
        V v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (j + k * NT < n) v[k] = src[j + k * NT];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (j + k * NT < n) dst[j + k * NT] = v[k];
    }
}

// The same as a kernel of its own: after the last iteration of a launch, and
// where the next iteration's first pass has no gate.
__global__ __launch_bounds__(kBlock) void k_scalar_stop(Gate gate)
{
    __shared__ double red[2 * kWavesPerBlock];
    __shared__ int32_t flag;
    (void)gate_open(gate, gate_load(gate), red, &flag);
}

// ------------------------------------------------------------------- aprod 1
constexpr int kGlobMax = 5;  // global columns of a general layout

enum Aprod1Mode : int {
    A1_ACCUM = 0,  // y += A x
    A1_LSQR = 1,   // y = A x - coef_u * y, coef_u = alpha/beta from the scalars
    A1_RESID = 2,  // y = b - A x
};

// Where Eq. (2) reads the attitude values of a row (columns t..t+3 of the three
// axes): three windows of x; 12 consecutive elements of x3, the section
// interleaved by axis (x3[3 c + axis] = x[att_base + axis n_dfa + c]: about 1.7
// cache lines per row instead of 3.6); such a copy that the workgroup makes
// in LDS; or nowhere: k_att_dot has left every row's attitude part in datt, in
// bucket order (row i at datt[place[i]]).
enum Aprod1Att : int { kWindows = 0, kInterleaved = 1, kStaged = 2, kPrepass = 3 };

// Eq. (2): 64-row steps over the grid's waves, one row per lane; part[blockIdx.x]
// receives the FP64 sum of squares of the stored y (LSQR, RESID). LDSX: the
// instrumental slice of x (n_instr_cols values) is first copied into LDS, so
// that the six random instrumental gathers per row hit LDS instead of L2.
// inv (optional, LSQR and RESID modes): placement of the row vector, the value
// of row i lives at y[inv[i]] (the attitude-bucket order of the solver's work
// vector); nullptr: y[i]. GEN: section sizes from the system view.
// A step's coefficients, then the gathers that its indices address, then the
// next step's indices go out together, one round trip a step at 16 waves a
// compute unit. What bounds it with attitude gathers is their requests (12
// values at a random place per row, 1.7 lines; 1.5e7 rows, 1e5 starts: 1.05 ms,
// 3.5 TB/s, whatever the schedule), hence the pre-pass form.
template <typename T, typename Acc, typename VX, typename VY, int MODE, int NT, bool LDSX, int XA,
          bool GEN = false>
__global__ __launch_bounds__(NT) void k_aprod1(SysView s, const VX* __restrict__ x,
                                                VY* __restrict__ y, const double* __restrict__ b,
                                                const Scalars* __restrict__ sc,
                                                double* __restrict__ part,
                                                const int32_t* __restrict__ inv,
                                                const VX* __restrict__ x3,
                                                const Acc* __restrict__ datt,
                                                const int32_t* __restrict__ place)
{
    constexpr int kAtt = kAxes * kParAxis, W = NT / kWave, NG = GEN ? kGlobMax : 1;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[W];
    if (MODE == A1_LSQR && sc->done) return;
    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t m = s.m;
    const int na = GEN ? s.na : kAstro, ni = GEN ? s.ni : kInstr, ng = GEN ? s.ng : 1;
    const bool att = XA != kPrepass && (!GEN || s.natt > 0);
    const int oatt = GEN ? s.off_att : kOffAtt, oins = GEN ? s.off_instr : kOffInstr,
              oglob = GEN ? s.off_glob : kOffGlob;
    // inv, if given, is place in the pre-pass form
    const int32_t* __restrict__ pl = XA == kPrepass ? place : (MODE != A1_ACCUM ? inv : nullptr);

    const int lane = threadIdx.x & (kWave - 1);
    const int32_t wave = uniform((int32_t)(blockIdx.x * W + threadIdx.x / kWave));
    const int64_t stride = (int64_t)gridDim.x * NT;
    // a section in LDS has few columns: the low word of its starts is enough
    using Start = std::conditional_t<XA == kStaged, int32_t, int64_t>;
    struct Idx {
        int64_t star;
        Start t;
        int32_t place, ix[kInstr];
    };
    auto lane_off = [&](int64_t r0) {  // the lane's row, the last one past the end
        return (uint32_t)(lane < m - r0 ? lane : m - 1 - r0);
    };
    auto load_idx = [&](Idx& w, int64_t r0) {
        const int64_t base = r0 < m ? r0 : m - 1;
        const uint32_t o = r0 < m ? lane_off(r0) : 0u;
        w.star = na > 0 ? ld_off(&s.star[base], o) : 0;
        if (att) {
            constexpr uint32_t words = sizeof(int64_t) / sizeof(Start);
            w.t = ld_off(reinterpret_cast<const Start*>(&s.att[base]), words * o);
        }
        if (pl) w.place = ld_off(&pl[base], o);
#pragma unroll
        for (int j = 0; j < kInstr; ++j)
            w.ix[j] = !GEN || j < ni ? ld_off(&s.instr[j * m + base], o) : 0;
    };
    Idx nx = {};
    int64_t r0 = (int64_t)wave * kWave;
    if (r0 < m) load_idx(nx, r0);

    const VX* xi = x + s.instr_base;
    const VX* xw = x3;
    if (LDSX) {
        VX* xl = reinterpret_cast<VX*>(smem_raw);
        for (int64_t j = threadIdx.x; j < s.n_instr_cols; j += NT) xl[j] = xi[j];
        xi = xl;
        if (XA == kStaged) {
            VX* wl = xl + s.n_instr_cols;
            const VX* xa = x + s.att_base;
            for (int ax = 0; ax < kAxes; ++ax)
                for (int64_t c = threadIdx.x; c < s.n_dfa; c += NT)
                    wl[kAxes * c + ax] = xa[ax * s.n_dfa + c];
            xw = wl;
        }
        __syncthreads();
    }
    const Acc coef = (MODE == A1_LSQR) ? (Acc)sc->coef_u : (Acc)0;
    Acc xg[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) xg[g] = g < ng ? (Acc)x[s.glob_base + g] : (Acc)0;
    auto att_value = [&](Start t, int e) {
        const int ax = e / kParAxis, qq = e % kParAxis;
        return XA == kWindows ? x[s.att_base + ax * s.n_dfa + t + qq]
                              : xw[kAxes * (t + qq) + ax];
    };

    double ssq = 0.0;
    for (; r0 < m; r0 += stride) {
        const uint32_t o = lane_off(r0);
        const bool ok = lane < m - r0;
        T aa[kAstro], at[kAtt], ai[kInstr], ag[NG];
#pragma unroll
        for (int j = 0; j < kAstro; ++j)
            aa[j] = !GEN || j < na ? ld_off(&val[j * m + r0], o) : (T)0;
        if (att) {
#pragma unroll
            for (int c = 0; c < kAtt; ++c) at[c] = ld_off(&val[(oatt + c) * m + r0], o);
        }
#pragma unroll
        for (int j = 0; j < kInstr; ++j)
            ai[j] = !GEN || j < ni ? ld_off(&val[(oins + j) * m + r0], o) : (T)0;
#pragma unroll
        for (int g = 0; g < NG; ++g)
            ag[g] = !GEN || g < ng ? ld_off(&val[(oglob + g) * m + r0], o) : (T)0;
        __builtin_amdgcn_sched_barrier(0);
        const Idx id = nx;
        VY* yp = (MODE != A1_ACCUM && inv) ? &y[id.place] : &y[r0 + o];
        const VY yo = MODE == A1_RESID ? (VY)0 : *yp;
        const Acc da = XA == kPrepass ? datt[id.place] : (Acc)0;
        const double bo = MODE == A1_RESID ? b[r0 + o] : 0.0;
        VX xs[kAstro], xt[kAtt], xv[kInstr];
        const VX* xa = x + (int64_t)na * id.star;
#pragma unroll
        for (int j = 0; j < kAstro; ++j)
            if (!GEN || j < na) xs[j] = xa[j];
        if (XA != kStaged && att) {
#pragma unroll
            for (int e = 0; e < kAtt; ++e) xt[e] = att_value(id.t, e);
        }
        if (!LDSX) {
#pragma unroll
            for (int j = 0; j < kInstr; ++j)
                if (!GEN || j < ni) xv[j] = xi[id.ix[j]];
        }
        __builtin_amdgcn_sched_barrier(0);
        load_idx(nx, r0 + stride);
        __builtin_amdgcn_sched_barrier(0);

        Acc d = (Acc)0;  // in section order
#pragma unroll
        for (int j = 0; j < kAstro; ++j)
            if (!GEN || j < na) d += (Acc)aa[j] * (Acc)xs[j];
        if (att) {
#pragma unroll
            for (int e = 0; e < kAtt; ++e)
                d += (Acc)at[e] * (Acc)(XA == kStaged ? att_value(id.t, e) : xt[e]);
        }
#pragma unroll
        for (int j = 0; j < kInstr; ++j)
            if (!GEN || j < ni) d += (Acc)ai[j] * (Acc)(LDSX ? xi[id.ix[j]] : xv[j]);
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (!GEN || g < ng) d += (Acc)ag[g] * xg[g];
        if (XA == kPrepass) d += da;
        const VY nv = MODE == A1_ACCUM  ? (VY)((Acc)yo + d)
                      : MODE == A1_LSQR ? (VY)(d - coef * (Acc)yo)
                                        : (VY)((Acc)bo - d);
        if (ok) {
            *yp = nv;
            if (MODE != A1_ACCUM) ssq += (double)nv * (double)nv;
        }
    }
    if (MODE != A1_ACCUM) {
        const double r = block_sum_n<NT>(ssq, red);
        if (threadIdx.x == 0) part[blockIdx.x] = r;
    }
}

// x3[3 c + axis] = x[att_base + axis * n_dfa + c]
template <typename V>
__global__ __launch_bounds__(kBlock) void k_interleave_att(const V* __restrict__ x,
                                                            int64_t att_base, int64_t n_dfa,
                                                            V* __restrict__ x3,
                                                            const Scalars* __restrict__ sc)
{
    if (sc != nullptr && sc->done) return;
    const int64_t total = (int64_t)kAxes * n_dfa;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < total;
         j += (int64_t)gridDim.x * kBlock) {
        const int64_t c = j / kAxes, ax = j - c * kAxes;
        x3[j] = x[att_base + ax * n_dfa + c];
    }
}

// ------------------------------------------------------------------- aprod 2
// Inclusive segmented scan over the wave of five values keyed by a
// non-decreasing key: equal keys at distance `off` imply the whole span in
// between carries the same key.
template <typename Acc>
__device__ __forceinline__ void seg_scan5(int64_t key, Acc (&v)[kAstro], int lane)
{
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int64_t ko = __shfl_up(key, off);
        Acc vo[kAstro];
#pragma unroll
        for (int j = 0; j < kAstro; ++j) vo[j] = __shfl_up(v[j], off);
        if (lane >= off && ko == key) {
#pragma unroll
            for (int j = 0; j < kAstro; ++j) v[j] += vo[j];
        }
    }
}

// Wave-wide sum, result in every lane.
template <typename Acc>
__device__ __forceinline__ Acc wave_sum(Acc v)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Cross-lane moves in the vector unit (no LDS): a reduction by ds_bpermute of the
// five sums of a star takes 60 LDS instructions, and 16 waves of a compute unit
// share one LDS (4000 cycles for each end of a star).
template <typename V, typename F>
__device__ __forceinline__ V by_words(V a, F&& f)
{
    if constexpr (sizeof(V) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, a);
        const uint32_t lo = f((uint32_t)b), hi = f((uint32_t)(b >> 32));
        return __builtin_bit_cast(V, (uint64_t)lo | ((uint64_t)hi << 32));
    } else {
        return __builtin_bit_cast(V, f(__builtin_bit_cast(uint32_t, a)));
    }
}

// Lane l of the result: the sum of a (l < 32) or b over lanes l mod 32 and
// l mod 32 + 32.
template <typename V>
__device__ __forceinline__ V half_sum(V a, V b)
{
    if constexpr (sizeof(V) == 8) {
        const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32),
                                                         false, false);
        return __builtin_bit_cast(V, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)) +
               __builtin_bit_cast(V, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32));
    } else {
        const uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
        const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        return __builtin_bit_cast(V, (uint32_t)r[0]) + __builtin_bit_cast(V, (uint32_t)r[1]);
    }
}

// Rows of 16 lanes: row r of the result is the sum of two rows of a (r even) or
// b: rows 0, 1 (r < 2) or 2, 3.
template <typename V>
__device__ __forceinline__ V row_pair_sum(V a, V b)
{
    if constexpr (sizeof(V) == 8) {
        const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32),
                                                         false, false);
        return __builtin_bit_cast(V, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)) +
               __builtin_bit_cast(V, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32));
    } else {
        const auto w = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a),
                                                        __builtin_bit_cast(uint32_t, b), false,
                                                        false);
        return __builtin_bit_cast(V, (uint32_t)w[0]) + __builtin_bit_cast(V, (uint32_t)w[1]);
    }
}

// Sum over the lanes of a row of 16 that are equal mod K, in all of them.
template <int K, typename V>
__device__ __forceinline__ V row_sum(V v)
{
    auto ror = [](V x, auto n) {
        return by_words(x, [](uint32_t w) {
            return (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x120 + decltype(n)::value, 0xf, 0xf,
                                                      false);
        });
    };
    if constexpr (K <= 8) v += ror(v, std::integral_constant<int, 8>());
    if constexpr (K <= 4) v += ror(v, std::integral_constant<int, 4>());
    if constexpr (K <= 2) v += ror(v, std::integral_constant<int, 2>());
    if constexpr (K <= 1) v += ror(v, std::integral_constant<int, 1>());
    return v;
}

// Sums of a star's five values over the lanes equal mod K, then
// put(j, r, sum) once for each value j and right-hand side r < K, on K lanes a
// value. Four values share the moves: one each in the four rows of a register.
// Every lane of the wave must be active.
template <int K, typename V, typename F>
__device__ __forceinline__ void star_put(const V (&v)[kAstro], int lane, F&& put)
{
    static_assert(kAstro == 5 && K <= 16, "four packed values and one");
    const V p = row_sum<K>(row_pair_sum(half_sum(v[0], v[1]), half_sum(v[2], v[3])));
    const V h = half_sum(v[4], v[4]);
    const V e = row_sum<K>(row_pair_sum(h, h));
    const int c = lane & 15, row = lane >> 4;
    const int j = ((row & 1) << 1) | (row >> 1);  // the value of this row of p
    if constexpr (K <= 8) {
        const bool last = row == 0 && c >= K && c < 2 * K;
        if (c < K || last) put(last ? 4 : j, c & (K - 1), last ? e : p);
    } else {
        put(j, c, p);
        if (row == 0) put(4, c, e);
    }
}

// Reduction of NV values per row over segments of equal, non-decreasing keys,
// one 64-row chunk at a time. Each lane keeps running partials of the segment
// that is still open at the end of the previous chunk; cross-lane work
// happens only where a segment ends (a wave sum per finished segment), so a
// segment longer than a chunk costs one vector add per lane per chunk.
// Invalid lanes (past the end of the range) carry key kNoStar.
template <typename Acc, int NV>
struct SegAcc {
    int64_t key = -1;  // open segment (wave-uniform), -1: none
    Acc acc[NV];
    __device__ SegAcc()
    {
#pragma unroll
        for (int j = 0; j < NV; ++j) acc[j] = (Acc)0;
    }
};

// emit(key, values) runs on the whole wave once per finished segment, with each
// lane's share of its sums.
template <typename Acc, int NV, typename Emit>
__device__ __forceinline__ void seg_chunk(SegAcc<Acc, NV>& S, int64_t key, const Acc (&v)[NV],
                                          int lane, Emit&& emit)
{
    const bool cont = key == S.key;
#pragma unroll
    for (int j = 0; j < NV; ++j) S.acc[j] += cont ? v[j] : (Acc)0;
    uint64_t rest = __ballot(!cont);
    if (rest == 0) return;  // the whole chunk continues the open segment
    if (S.key >= 0) {       // keys are sorted: the open segment ends here
        emit(S.key, S.acc);
    }
    S.key = -1;
#pragma unroll
    for (int j = 0; j < NV; ++j) S.acc[j] = (Acc)0;
    while (rest != 0) {
        const int l0 = __ffsll((unsigned long long)rest) - 1;
        const int64_t k2 = __shfl(key, l0);
        if (k2 == kNoStar) break;  // only lanes past the end remain
        const bool mine = key == k2;
        const uint64_t same = __ballot(mine);
        if ((same >> (kWave - 1)) & 1ull) {  // reaches the last lane: stays open
            S.key = k2;
#pragma unroll
            for (int j = 0; j < NV; ++j) S.acc[j] = mine ? v[j] : (Acc)0;
            break;
        }
        Acc t[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) t[j] = mine ? v[j] : (Acc)0;
        emit(k2, t);
        rest &= ~same;
    }
}

template <typename Acc, int NV, typename Emit>
__device__ __forceinline__ void seg_finish(SegAcc<Acc, NV>& S, int lane, Emit&& emit)
{
    if (S.key < 0) return;
    emit(S.key, S.acc);
    S.key = -1;
}

// Stateless variant: every segment present in the chunk is reduced and
// emitted at once (a segment spanning several chunks is emitted once per
// chunk, so emit must accumulate). Keeps no registers across chunks.
template <typename Acc, int NV, typename Emit>
__device__ __forceinline__ void seg_flush(int64_t key, const Acc (&v)[NV], int lane, Emit&& emit)
{
    uint64_t rest = __ballot(key != kNoStar);
    while (rest != 0) {
        const int l0 = __ffsll((unsigned long long)rest) - 1;
        const int64_t k2 = __shfl(key, l0);
        const bool mine = key == k2;
        const uint64_t same = __ballot(mine);
        Acc t[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) t[j] = mine ? v[j] : (Acc)0;
        emit(k2, t);
        rest &= ~same;
    }
}

// x += A^T y (SQUARE: x_j += sum of squared coefficients of column j, used
// for the column norms). wb: star-aligned row boundaries, one range per wave
// (gridDim.x * kWavesPerBlock ranges). Instrumental columns [0, hcols) are
// accumulated in an FP64 LDS histogram (hcols * 8 bytes of dynamic shared
// memory) flushed with one device atomic per column per workgroup; columns
// from hcols on are left to k_instr_tail. gpart[blockIdx.x] gets the
// workgroup's global-column partial; a later kernel adds them up.
// ATT = false leaves the attitude columns to the bucket-order pass
// (k_att_hist) and skips loading them. SCAN selects the astrometric
// reduction: a segmented scan every chunk (true) or the accumulate-and-flush
// segments of seg_chunk (false).
// inv (optional): the value of row i is u[inv[i]].
template <typename T, typename Acc, typename VU, bool SQUARE, bool ATT = true, bool SCAN = true,
          int NT = kBlock>
__global__ __launch_bounds__(NT) void k_aprod2(SysView s, const VU* __restrict__ u,
                                                    Acc* __restrict__ q,
                                                    const int64_t* __restrict__ wb,
                                                    Acc* __restrict__ gpart, int64_t hcols,
                                                    const Scalars* __restrict__ sc,
                                                    const int32_t* __restrict__ inv = nullptr)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* lds = reinterpret_cast<double*>(smem_raw);  // FP64 histogram (see k_att_hist)
    __shared__ Acc gred[NT / kWave];
    if (sc != nullptr && sc->done) return;

    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t m = s.m;
    for (int64_t j = threadIdx.x; j < hcols; j += NT) lds[j] = 0.0;
    __syncthreads();

    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave = (int64_t)blockIdx.x * (NT / kWave) + threadIdx.x / kWave;
    const int64_t rb = wb[wave], re = wb[wave + 1];
    Acc* __restrict__ qatt = q + s.att_base;
    Acc* __restrict__ qins = q + s.instr_base;

    int64_t carry_star = -1;
    Acc carry[kAstro];
#pragma unroll
    for (int j = 0; j < kAstro; ++j) carry[j] = (Acc)0;
    Acc gsum = (Acc)0;
    SegAcc<Acc, kAstro> seg;
    auto astro_emit = [q, lane](int64_t star, const Acc (&v)[kAstro]) {
        star_put<1>(v, lane, [&](int j, int, Acc sum) { q[kAstro * star + j] += sum; });
    };

    // Chunks start on 64-row boundaries so that every coefficient stream is
    // read in whole cache lines; lanes before rb (owned by the previous wave)
    // take the first row's star with zero contributions.
    for (int64_t r0 = rb < re ? (rb & ~(int64_t)(kWave - 1)) : re; r0 < re; r0 += kWave) {
        const int64_t i = r0 + lane;
        const bool ok = i >= rb && i < re;
        const int64_t ic = i < rb ? rb : (i < re ? i : re - 1);
        const int64_t st = i < re ? ldnt(&s.star[ic]) : kNoStar;
        const int64_t t = ATT ? ldnt(&s.att[ic]) : 0;
        T a[kPar];
#pragma unroll
        for (int c = 0; c < kPar; ++c)
            a[c] = (ATT || c < kOffAtt || c >= kOffInstr) ? ldnt(&val[c * m + ic]) : (T)0;
        int32_t ix[kInstr];
#pragma unroll
        for (int j = 0; j < kInstr; ++j) ix[j] = ldnt(&s.instr[j * m + ic]);
        Acc ui = (Acc)0;
        if (!SQUARE) ui = ok ? (Acc)u[inv ? (int64_t)ldnt(&inv[ic]) : ic] : (Acc)0;

        Acc contrib[kPar];
#pragma unroll
        for (int c = 0; c < kPar; ++c)
            contrib[c] = SQUARE ? (ok ? (Acc)a[c] * (Acc)a[c] : (Acc)0) : (Acc)a[c] * ui;

        // attitude: 3 axes x 4 consecutive columns from the row's start t
        if (ok) {
            if (ATT) {
#pragma unroll
                for (int ax = 0; ax < kAxes; ++ax) {
                    Acc* dst = qatt + ax * s.n_dfa + t;
#pragma unroll
                    for (int qq = 0; qq < kParAxis; ++qq)
                        atomicAdd(dst + qq, contrib[kOffAtt + ax * kParAxis + qq]);
                }
            }
            // instrumental
#pragma unroll
            for (int j = 0; j < kInstr; ++j)
                if (ix[j] < hcols) atomicAdd(&lds[ix[j]], (double)contrib[kOffInstr + j]);
        }
        gsum += contrib[kOffGlob];

        // astrometric: per-star segmented reduction across chunks
        Acc pa[kAstro];
#pragma unroll
        for (int j = 0; j < kAstro; ++j) pa[j] = contrib[j];
        if (!SCAN) {
            seg_chunk(seg, st, pa, lane, astro_emit);
            continue;
        }
        if (carry_star >= 0) {
            const int64_t st0 = __shfl(st, 0);
            if (lane == 0) {
                if (st0 == carry_star) {
#pragma unroll
                    for (int j = 0; j < kAstro; ++j) pa[j] += carry[j];
                } else {
#pragma unroll
                    for (int j = 0; j < kAstro; ++j) q[kAstro * carry_star + j] += carry[j];
                }
            }
        }
        seg_scan5<Acc>(st, pa, lane);
        const int64_t snext = __shfl_down(st, 1);
        if (ok && lane != kWave - 1 && snext != st) {
#pragma unroll
            for (int j = 0; j < kAstro; ++j) q[kAstro * st + j] += pa[j];
        }
        carry_star = __shfl(st, kWave - 1);
#pragma unroll
        for (int j = 0; j < kAstro; ++j) carry[j] = __shfl(pa[j], kWave - 1);
        if (carry_star == kNoStar) carry_star = -1;
    }
    if (carry_star >= 0 && lane == 0) {
#pragma unroll
        for (int j = 0; j < kAstro; ++j) q[kAstro * carry_star + j] += carry[j];
    }
    if (!SCAN) seg_finish(seg, lane, astro_emit);

    // global column: wave shuffle -> LDS -> one partial per workgroup
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) gsum += __shfl_down(gsum, off);
    if (lane == 0) gred[threadIdx.x / kWave] = gsum;
    __syncthreads();
    if (threadIdx.x == 0) {
        Acc g = (Acc)0;
        for (int k = 0; k < NT / kWave; ++k) g += gred[k];
        gpart[blockIdx.x] = g;
    }
    // instrumental flush: one device atomic per column per workgroup
    for (int64_t j = threadIdx.x; j < hcols; j += NT) {
        const double v = lds[j];
        if (v != 0.0) atomicAdd(&qins[j], (Acc)v);
    }
}

// ------------------------------------------------------ fused iteration pass
// One sweep over the rows in star order doing both operator products of an
// LSQR step (Eq. 2 and Eq. 3). Because u~_{i+1} = Abar v_i - (alpha_i/beta_i) u~_i
// is row-local, each row's new value is known as soon as the row's
// coefficients are in registers, and the same registers then feed
// A^T u~_{i+1} for the astrometric (per-star segments), instrumental (LDS
// histogram) and global (per-workgroup partial) columns. beta_{i+1} = ||u~||
// is applied afterwards by the column kernel (v~ = p .* A^T u~ / beta - beta v),
// so A is read once per iteration for these sections; the attitude columns
// are left to the bucket-order pass, which reads u~_{i+1}, except in kAttAll.
//   x: vp = p .* v (Acc), x3: its interleaved attitude section,
//   u: u~ [m], overwritten (row i at u[inv[i]], or u[i] without inv),
//   part[blockIdx.x]: FP64 sum of squares of the
//   stored u~, q: A^T u~ accumulator (astro, instr, glob sections),
//   gpart[blockIdx.x]: global-column partials, steps: the waves' rows.
// Dynamic LDS: the FP64 histogram of instrumental columns [0, hcols) (see
// k_att_hist; columns from hcols on are left to k_instr_tail), in kAttAll that
// of the attitude columns ([axis][n_dfa], of FP64 products as in k_att_hist), then
// the instrumental slice of x (LDSX, n_instr_cols Acc) and the interleaved
// attitude section (WIN).
// AM, the attitude part of the dot product: kAttX reads three 4-value windows
// of x, kAttX3 one 12-value window of x3, kAttPre none: k_att_dot has already
// replaced u~ by (attitude part of A vp) - coef u~, so the row adds that;
// kAttGather: k_att_dot has written the attitude part of every row to datt in
// bucket order, the row reads it at datt[inv[i]] and keeps u~ in star order
// (u[i]), so that u~ is read and written sequentially and the only permuted
// access is that read. kAttAll: the attitude values come from x3 (WIN: its copy
// in LDS) and the attitude columns are scattered into their LDS histogram too,
// so the iteration reads A once, in one pass.
// us (optional): a star-order copy of the new u~ (us[i]), written
// sequentially for the instrumental tail passes that follow, which then read
// it without the permutation.
// satt (kAttAll), sins (optional): the workgroup's histograms are stored as
// slices there (SliceView) instead of being added to q with device atomics.
// GEN > 0: section sizes from the system view (general layouts with at most GEN
// global columns: five of them cost 20 registers more); the loads stay unrolled,
// each under a uniform test. A2: Eq. (3) alone, u unchanged. kPlain: loads without
// the nontemporal hint, for a matrix that the last-level cache holds from one
// iteration to the next.
// The rows are dealt to the waves in whole 64-row steps, an equal number each
// but for one (WaveSteps), not in ranges that begin with a star: a range of a
// few steps otherwise takes one or two more, and the waves wait for the
// longest (a solve of 1e6 rows, layout 3 + 12 + 2 + 3: 3.00 -> 2.42 ms). Stars
// cut by a step's end make more star sums, which pays with lane swaps only: with
// ds_bpermute sums a solve of 3e5 rows was 9% slower.
enum { kAttX = 0, kAttX3 = 1, kAttPre = 2, kAttGather = 3, kAttAll = 4 };

// PIECE > 0: a workgroup's waves walk its rows together, PIECE steps each in
// turn, so that the bucket-order lines of u~ that a workgroup has begun to write
// (one per bucket and piece) are full before L2 evicts them: 1e8 rows, 62
// buckets, FP32 inner iterations 210.7 -> 205.0 ms, FP64 81.6 -> 79.7 ms (5e7
// rows). The first and last star of every piece cost device atomics: 16 buckets
// 144.1 -> 146.3 ms.

// Step ranges of the waves: wave w takes `each` 64-row steps, and one more if
// w < more, from first(w).
struct WaveSteps {
    int64_t each;
    int32_t more;
    __device__ int64_t first(int32_t w) const { return w * each + (w < more ? w : more); }
};
template <typename T, typename Acc, int NT, bool LDSX, int AM, bool CIDX, int GEN = 0,
          bool WIN = false, bool A2 = false, bool kPlain = false, int PIECE = 0>
__global__ __launch_bounds__(NT) void k_fused(SysView s, const Acc* __restrict__ x,
                                               const Acc* __restrict__ x3, Acc* __restrict__ u,
                                               Acc* __restrict__ q, WaveSteps steps,
                                               Acc* __restrict__ gpart, double* __restrict__ part,
                                               int64_t hcols, Gate gate,
                                               const int32_t* __restrict__ inv,
                                               const Acc* __restrict__ datt = nullptr,
                                               Acc* __restrict__ us = nullptr,
                                               double* __restrict__ satt = nullptr,
                                               double* __restrict__ sins = nullptr)
{
    constexpr bool kNoAtt = AM == kAttPre || AM == kAttGather;
    constexpr int kAtt = kAxes * kParAxis;
    constexpr int NG = GEN ? GEN : 1;
    constexpr int W = NT / kWave;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ Acc gred[NG * W];
    __shared__ double sred[W < 2 * kWavesPerBlock ? 2 * kWavesPerBlock : W];
    __shared__ int32_t gflag;
    const int na = GEN ? s.na : kAstro, ni = GEN ? s.ni : kInstr, ng = GEN ? s.ng : 1;
    const bool att = !kNoAtt && (!GEN || s.natt > 0);
    const int oatt = GEN ? s.off_att : kOffAtt, oins = GEN ? s.off_instr : kOffInstr,
              oglob = GEN ? s.off_glob : kOffGlob;

    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t m = s.m;
    const int64_t ninst = GEN && ni == 0 ? 0 : s.n_instr_cols;
    const int64_t hatt = AM == kAttAll && att ? kAxes * s.n_dfa : 0;
    double* hist = reinterpret_cast<double*>(smem_raw);
    double* ahist = hist + hcols;
    const Acc* xi = A2 ? nullptr : x + s.instr_base;
    const Acc* xw = x3;
    const GateIn gin = gate_load(gate);
    for (int64_t j = threadIdx.x; j < hcols + hatt; j += NT) hist[j] = 0.0;
    if (LDSX && !A2) {
        const int64_t off = ((hcols + hatt) * 8 + 15) & ~(int64_t)15;
        Acc* xl = reinterpret_cast<Acc*>(smem_raw + off);
        stage<NT>(xl, xi, ninst);
        xi = xl;
        if (WIN) {
            Acc* wl = xl + ninst;
            stage<NT>(wl, x3, hatt);
            xw = wl;
        }
    }
    Acc coef = (Acc)0;
    if (!A2) {
        if (!gate_open(gate, gin, sred, &gflag)) return;
        coef = (Acc)gin.coef;
    } else if (gate.A != nullptr && gate.A->done) {
        return;
    }
    __syncthreads();

    Acc xg[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) xg[g] = (!A2 && g < ng) ? x[s.glob_base + g] : (Acc)0;
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t wave = (int32_t)(blockIdx.x * W + threadIdx.x / kWave);
    // [p0, p1): the wave's steps (PIECE: its workgroup's, of which it takes
    // pieces of PIECE, every W-th)
    const int32_t w0 = blockIdx.x * W;
    const int64_t p0 = PIECE ? steps.first(w0) + (wave - w0) * PIECE : steps.first(wave);
    const int64_t p1 = steps.first(PIECE ? w0 + W : wave + 1);
    Acc* __restrict__ qins = q + s.instr_base;

    double ssq = 0.0;
    Acc gsum[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) gsum[g] = (Acc)0;
    SegAcc<Acc, kAstro> seg;
    // Every star's columns of q are zero here in an LSQR step (the column kernel
    // leaves them so), so a step stores a star's sums; an addition would make
    // the wave wait for its loads, and with them for every load issued before
    // (loads return in issue order), at each end of a star. Only the first and
    // the last star of a wave's rows may go on in another wave's: their sums are
    // added with device atomics, so the rounding of a star over three or more
    // waves' rows (A2: of any such star, q not being zero) depends on their order
    // of arrival.
    bool shared = true;
    auto astro_emit = [=, &shared](int64_t star, const Acc (&v)[kAstro]) {
        star_put<1>(v, lane, [&](int j, int, Acc sum) {
            if (GEN && j >= na) return;
            Acc* dst = &q[(int64_t)na * star + j];
            if (shared) atomicAdd(dst, sum);
            else if (A2) *dst += sum;
            else *dst = sum;
        });
        shared = false;
    };

    // 64-row steps, all the wave's or (PIECE) piece by piece; lanes past the last
    // row compute on it and contribute nothing.
    int64_t q0 = p0;
    if (PIECE == 0 || p0 < p1) do {
        const int64_t q1 = PIECE == 0 || q0 + PIECE > p1 ? p1 : q0 + PIECE;
        const int64_t rb = q0 * kWave, re = q1 * kWave < m ? q1 * kWave : m;
        shared = true;  // the first star of a piece
        for (int64_t r0 = rb; r0 < re; r0 += kWave) {
            const int64_t i = r0 + lane;
            const bool ok = i < re;
            const int64_t ic = ok ? i : re - 1;
            const int64_t stc = star_of<CIDX, kPlain>(s, ic);
            const int64_t st = ok ? stc : kNoStar;
            const int64_t t = att ? ld_stream<kPlain>(&s.att[ic]) : 0;
            T aa[kAstro], at[kAtt], ai[kInstr], ag[NG];
            int32_t ix[kInstr];
#pragma unroll
            for (int j = 0; j < kAstro; ++j)
                aa[j] = !GEN || j < na ? ld_stream<kPlain>(&val[j * m + ic]) : (T)0;
            if (!kNoAtt) {
                if (att) {
#pragma unroll
                    for (int c = 0; c < kAtt; ++c) at[c] = ld_stream<kPlain>(&val[(oatt + c) * m + ic]);
                }
            }
#pragma unroll
            for (int j = 0; j < kInstr; ++j)
                ai[j] = !GEN || j < ni ? ld_stream<kPlain>(&val[(oins + j) * m + ic]) : (T)0;
#pragma unroll
            for (int g = 0; g < NG; ++g)
                ag[g] = !GEN || g < ng ? ld_stream<kPlain>(&val[(oglob + g) * m + ic]) : (T)0;
#pragma unroll
            for (int j = 0; j < kInstr; ++j) ix[j] = !GEN || j < ni ? instr_of<CIDX, kPlain>(s, j, ic) : 0;
            const int64_t pu = (AM != kAttGather && inv) ? (int64_t)ldnt(&inv[ic]) : ic;
            const Acc dg = AM == kAttGather ? datt[ldnt(&inv[ic])] : (Acc)0;
            const Acc uo = u[pu];

            Acc d = (Acc)0;
            if (A2) {
                d = ok ? uo : (Acc)0;
            } else {
                // Eq. (2): the row's dot product with vp, in section order
                const Acc* xa = x + na * stc;
#pragma unroll
                for (int j = 0; j < kAstro; ++j)
                    if (!GEN || j < na) d += (Acc)aa[j] * xa[j];
                if (!kNoAtt) {
                    if (att) {
#pragma unroll
                        for (int ax = 0; ax < kAxes; ++ax) {
#pragma unroll
                            for (int qq = 0; qq < kParAxis; ++qq) {
                                const Acc xv = AM == kAttX ? x[s.att_base + ax * s.n_dfa + t + qq]
                                                           : xw[kAxes * (t + qq) + ax];
                                d += (Acc)at[ax * kParAxis + qq] * xv;
                            }
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < kInstr; ++j)
                    if (!GEN || j < ni) d += (Acc)ai[j] * xi[ix[j]];
#pragma unroll
                for (int g = 0; g < NG; ++g)
                    if (!GEN || g < ng) d += (Acc)ag[g] * xg[g];
                if (AM == kAttPre)
                    d += uo;
                else if (AM == kAttGather)
                    d += dg - coef * uo;
                else
                    d -= coef * uo;
                if (ok) u[pu] = d;
                if (ok && us) us[ic] = d;
                if (!ok) d = (Acc)0;
                ssq += (double)d * (double)d;
            }

            // Eq. (3) with the new value
            if (ok) {
                if (AM == kAttAll) {
                    if (att) {
#pragma unroll
                        for (int ax = 0; ax < kAxes; ++ax)
#pragma unroll
                            for (int qq = 0; qq < kParAxis; ++qq)
                                atomicAdd(&ahist[ax * s.n_dfa + t + qq],
                                          (double)at[ax * kParAxis + qq] * (double)d);
                    }
                }
#pragma unroll
                for (int j = 0; j < kInstr; ++j) {
                    if ((!GEN || j < ni) && ix[j] < hcols)
                        atomicAdd(&hist[ix[j]], (double)((Acc)ai[j] * d));
                }
            }
#pragma unroll
            for (int g = 0; g < NG; ++g) gsum[g] += (Acc)ag[g] * d;
            Acc pa[kAstro];
#pragma unroll
            for (int j = 0; j < kAstro; ++j) pa[j] = (Acc)aa[j] * d;
            if (!GEN || na > 0) seg_chunk(seg, st, pa, lane, astro_emit);
        }
        shared = true;
        seg_finish(seg, lane, astro_emit);
        q0 += W * PIECE;
    } while (PIECE > 0 && q0 < p1);

    // per-workgroup partials: global columns and ||u~||^2
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
#pragma unroll
        for (int g = 0; g < NG; ++g) gsum[g] += __shfl_down(gsum[g], off);
        if (!A2) ssq += __shfl_down(ssq, off);
    }
    if (lane == 0) {
#pragma unroll
        for (int g = 0; g < NG; ++g) gred[g * W + threadIdx.x / kWave] = gsum[g];
        sred[threadIdx.x / kWave] = ssq;
    }
    __syncthreads();
    if (threadIdx.x < NG) {
        Acc g = (Acc)0;
        for (int k = 0; k < W; ++k) g += gred[threadIdx.x * W + k];
        gpart[(int64_t)blockIdx.x * NG + threadIdx.x] = g;
    }
    if (!A2 && threadIdx.x == 0) {
        double r = 0.0;
        for (int k = 0; k < W; ++k) r += sred[k];
        part[blockIdx.x] = r;
    }
    for (int64_t j = threadIdx.x; j < hcols; j += NT) {
        const double v = hist[j];
        if (sins)
            sins[blockIdx.x * hcols + j] = v;
        else if (v != 0.0)
            atomicAdd(&qins[j], (Acc)v);
    }
    if (AM == kAttAll)
        for (int64_t j = threadIdx.x; j < hatt; j += NT) satt[blockIdx.x * hatt + j] = ahist[j];
}

// Workgroups that read the same rows (the windows of a section, the sweeps of
// a k-tile) side by side: block b's part of the rows and its window or sweep
// (of n), the n of a part next to each other on one accelerator die (block b
// runs on die b mod 8), where a row read by one of them is found in L2 by the
// others. One after the other, each reads all rows from memory again.
constexpr int kDies = 8;
struct SideBySide {
    int64_t part;
    int side;
};
__device__ __forceinline__ SideBySide side_by_side(int64_t block, int n)
{
    const int64_t k = block / kDies;
    return {k / n * kDies + block % kDies, (int)(k % n)};
}

// Instrumental columns [c0, ninst) of Eq. (3) (or of the squared column norms,
// SQUARE) when the row passes keep only the first columns in LDS, in nw
// windows of tw columns: a workgroup sweeps one of P parts of the rows with an
// FP64 LDS histogram of one window (the windows of a part side by side), then
// flushes it with one device atomic per column. U holds K
// values per row, row i at U[inv[i] K + r] (U[i K + r] without inv); frozen
// RHS are skipped.
// GEN: section sizes from the system view (general layouts); otherwise the
// full layout's constants.
// CIDX: the indices from the compact copy (1e7 rows, 30,000 columns, FP32,
// a refined solve: 27.25 -> 26.23 ms).
template <typename T, typename Acc, int K, bool SQUARE, int NT, bool GEN, bool PLAIN = false,
          bool CIDX = false>
__global__ __launch_bounds__(NT) void k_instr_tail(SysView s, const Acc* __restrict__ U,
                                                    const int32_t* __restrict__ inv,
                                                    Acc* __restrict__ Q, int64_t cfirst, int64_t tw,
                                                    int nw, const Scalars* __restrict__ sc)
{
    const SideBySide sb = side_by_side(blockIdx.x, nw);
    const int64_t P = gridDim.x / nw;
    const int64_t c0 = cfirst + sb.side * tw;
    const int64_t c1 = c0 + tw < s.n_instr_cols ? c0 + tw : s.n_instr_cols;
    const int ni = GEN ? s.ni : kInstr, oins = GEN ? s.off_instr : kOffInstr;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* hist = reinterpret_cast<double*>(smem_raw);
    uint32_t live = 0;
#pragma unroll
    for (int r = 0; r < K; ++r)
        live |= (sc != nullptr && sc[r].done) ? 0u : (1u << r);
    if (live == 0) return;
    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t m = s.m, w = c1 - c0;
    for (int64_t e = threadIdx.x; e < w * K; e += NT) hist[e] = 0.0;
    __syncthreads();
    // the workgroup's rows [r0, r1) as one contiguous range per wave, walked
    // in 64-row steps aligned to 64 rows: a line that two steps share is read
    // by the same wave one step apart (an L2 hit), not by two waves at once
    // (which fetches it twice; also where the caller's columns are not
    // line-aligned)
    static_assert(NT % kWave == 0, "whole waves");
    const int64_t r0 = sb.part * m / P, r1 = (sb.part + 1) * m / P;
    constexpr int kW = NT / kWave;
    const int wv = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const int64_t rb = uniform(r0 + (r1 - r0) * wv / kW);
    const int64_t re = uniform(r0 + (r1 - r0) * (wv + 1) / kW);
    // Steps in flight: the streams of the step two ahead are loaded after the
    // current step's values of U have been asked for (one step before they are
    // used), so a step waits neither for memory nor for the permuted read it
    // addresses. Lanes outside [rb, re) repeat a row of the range with weight 0.
    struct Step {
        int32_t ix[kInstr];
        T a[kInstr];
        int32_t pu;
    };
    auto load = [&](Step& st, int64_t i0) {
        // the step's first row (of the range, once past its end) and the lane's
        // row from there
        const int64_t base = i0 < re ? i0 : re - 1;
        const int64_t k = base + lane;
        const uint32_t o = (uint32_t)((k < rb ? rb : (k < re ? k : re - 1)) - base);
#pragma unroll
        for (int j = 0; j < kInstr; ++j) {
            if constexpr (CIDX)
                st.ix[j] = j < ni ? (int32_t)ld_off<PLAIN>(&s.instr16[j * m + base], o) : -1;
            else
                st.ix[j] = j < ni ? ld_off<PLAIN>(&s.instr[j * m + base], o) : -1;
            st.a[j] = j < ni ? ld_off<PLAIN>(&val[(oins + j) * m + base], o) : (T)0;
        }
        st.pu = inv ? ld_off(&inv[base], o) : (int32_t)(base + o - rb);
    };
    auto value = [&](const Step& st, Acc (&u)[K]) {
        if (SQUARE) return;
        const Acc* up = U + (inv ? (int64_t)st.pu : rb + st.pu) * K;
#pragma unroll
        for (int r = 0; r < K; ++r) u[r] = up[r];
    };
    auto scatter = [&](const Step& st, const Acc (&u)[K], int64_t i0) {
        const int64_t k = i0 + lane;
        if (k < rb || k >= re) return;
#pragma unroll
        for (int j = 0; j < kInstr; ++j) {
            const uint32_t c = (uint32_t)(st.ix[j] - (int32_t)c0);  // < 2^31: n_instr_cols
            if (c >= (uint32_t)w) continue;
#pragma unroll
            for (int r = 0; r < K; ++r) {
                if (!((live >> r) & 1u)) continue;
                const double av = (double)(Acc)st.a[j];
                atomicAdd(&hist[r * (uint32_t)w + c],
                          SQUARE ? av * av : (double)((Acc)st.a[j] * u[r]));
            }
        }
    };
    const int64_t istart = rb & ~(int64_t)(kWave - 1);
    if constexpr (K <= 4) {
        if (rb < re) {
            Step A, B, C;
            Acc ua[K], ub[K];
            int64_t i0 = istart;
            load(A, i0);
            load(B, i0 + kWave);
            value(A, ua);
            // step(cur, its U, next, next's U, the buffer two ahead)
            auto step = [&](const Step& cur, const Acc (&uc)[K], const Step& nxt, Acc (&un)[K],
                            Step& far) {
                value(nxt, un);
                __builtin_amdgcn_sched_barrier(0);
                load(far, i0 + 2 * kWave);
                __builtin_amdgcn_sched_barrier(0);
                scatter(cur, uc, i0);
                __builtin_amdgcn_sched_barrier(0);
                i0 += kWave;
                return i0 < re;
            };
            for (;;) {  // six steps: three buffers of rows, two of U
                if (!step(A, ua, B, ub, C)) break;
                if (!step(B, ub, C, ua, A)) break;
                if (!step(C, ua, A, ub, B)) break;
                if (!step(A, ub, B, ua, C)) break;
                if (!step(B, ua, C, ub, A)) break;
                if (!step(C, ub, A, ua, B)) break;
            }
        }
    } else {  // more right-hand sides: their registers leave no room for it
        for (int64_t i0 = istart; i0 < re; i0 += kWave) {
            Step A;
            Acc ua[K];
            load(A, i0);
            value(A, ua);
            scatter(A, ua, i0);
        }
    }
    __syncthreads();
    Acc* __restrict__ qins = Q + (s.instr_base + c0) * K;
    for (int32_t e = threadIdx.x; e < (int32_t)w * K; e += NT) {
        const int32_t c = e / K, r = e - c * K;  // one plane per right-hand side (k_att_dot)
        const double v = hist[r * (int32_t)w + c];
        if (v != 0.0) atomicAdd(&qins[e], (Acc)v);
    }
}

// --------------------------------------------------------- general layouts
// Rows whose sections differ from 5 + 3 x 4 + 6 + 1 (sections absent, fewer
// astrometric or instrumental coefficients, up to kGlobMax global columns): the
// section sizes and value-row offsets come from the system view at run time. The
// LSQR step and A x run the GEN instances of k_fused and k_aprod1; the kernel
// here is for Eq. (3) alone outside the one pass: the column norms, the start of
// a solve and lsqr_aprod2 in bucket order, and separate passes.

// Eq. (3) (SQUARE: squared coefficients, the column norms) for a general
// layout over the star-aligned wave ranges: astrometric per-star segments,
// attitude by device atomics when ATT (else left to the bucket-order pass),
// instrumental columns [0, hcols) in an FP64 LDS histogram (the rest to
// k_instr_tail), global columns as per-workgroup partials
// gpart[blockIdx.x * kGlobMax + g].
template <typename T, typename Acc, typename VU, bool SQUARE, bool ATT>
__global__ __launch_bounds__(kBlock) void k_gen_aprod2(SysView s, const VU* __restrict__ u,
                                                        Acc* __restrict__ q,
                                                        const int64_t* __restrict__ wb,
                                                        Acc* __restrict__ gpart, int64_t hcols,
                                                        const Scalars* __restrict__ sc,
                                                        const int32_t* __restrict__ inv)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* lds = reinterpret_cast<double*>(smem_raw);
    __shared__ Acc gred[kGlobMax][kWavesPerBlock];
    if (sc != nullptr && sc->done) return;
    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t m = s.m;
    const int na = s.na, ni = s.ni, ng = s.ng;
    for (int64_t j = threadIdx.x; j < hcols; j += kBlock) lds[j] = 0.0;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave;
    const int64_t rb = wb[wave], re = wb[wave + 1];
    Acc gsum[kGlobMax];
#pragma unroll
    for (int g = 0; g < kGlobMax; ++g) gsum[g] = (Acc)0;
    SegAcc<Acc, kAstro> seg;
    auto astro_emit = [q, na, lane](int64_t star, const Acc (&v)[kAstro]) {
        star_put<1>(v, lane, [&](int j, int, Acc sum) {
            if (j < na) q[(int64_t)na * star + j] += sum;
        });
    };
    for (int64_t r0 = rb < re ? (rb & ~(int64_t)(kWave - 1)) : re; r0 < re; r0 += kWave) {
        const int64_t i = r0 + lane;
        const bool ok = i >= rb && i < re;
        const int64_t ic = i < rb ? rb : (i < re ? i : re - 1);
        Acc ui = (Acc)0;
        if (!SQUARE) ui = ok ? (Acc)u[inv ? (int64_t)ldnt(&inv[ic]) : ic] : (Acc)0;
        auto contrib = [&](T a) -> Acc {
            return SQUARE ? (ok ? (Acc)a * (Acc)a : (Acc)0) : (Acc)a * ui;
        };
        if (na > 0) {  // uniform: seg_chunk is collective
            const int64_t st = i < re ? ldnt(&s.star[ic]) : kNoStar;
            Acc pa[kAstro];
#pragma unroll
            for (int j = 0; j < kAstro; ++j)
                pa[j] = j < na ? contrib(ldnt(&val[j * m + ic])) : (Acc)0;
            seg_chunk(seg, st, pa, lane, astro_emit);
        }
        if (ATT && s.natt > 0 && ok) {
            const int64_t t = ldnt(&s.att[ic]);
#pragma unroll
            for (int ax = 0; ax < kAxes; ++ax)
#pragma unroll
                for (int qq = 0; qq < kParAxis; ++qq)
                    atomicAdd(&q[s.att_base + ax * s.n_dfa + t + qq],
                              contrib(ldnt(&val[(s.off_att + ax * kParAxis + qq) * m + ic])));
        }
        for (int j = 0; j < ni; ++j) {
            const int32_t ix = ldnt(&s.instr[j * m + ic]);
            const Acc c = contrib(ldnt(&val[(s.off_instr + j) * m + ic]));
            if (ok && ix < hcols) atomicAdd(&lds[ix], (double)c);
        }
        for (int g = 0; g < ng; ++g) {
            const Acc c = contrib(ldnt(&val[(s.off_glob + g) * m + ic]));
            gsum[g] += ok ? c : (Acc)0;
        }
    }
    if (na > 0) seg_finish(seg, lane, astro_emit);
#pragma unroll
    for (int g = 0; g < kGlobMax; ++g) {
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) gsum[g] += __shfl_down(gsum[g], off);
        if (lane == 0) gred[g][threadIdx.x / kWave] = gsum[g];
    }
    __syncthreads();
    if (threadIdx.x < kGlobMax) {
        Acc t = (Acc)0;
        for (int k = 0; k < kWavesPerBlock; ++k) t += gred[threadIdx.x][k];
        gpart[(int64_t)blockIdx.x * kGlobMax + threadIdx.x] = t;
    }
    Acc* __restrict__ qins = q + s.instr_base;
    for (int64_t j = threadIdx.x; j < hcols; j += kBlock) {
        const double v = lds[j];
        if (v != 0.0) atomicAdd(&qins[j], (Acc)v);
    }
}

// --------------------------------------------------------- constraint rows
// Equations appended below the observation rows (Sect. 2): a few long sparse
// rows, in CSR form with FP64 values. One workgroup per row (grid-stride
// over rows); their vector entries sit after the observation rows, unpermuted.

// Eq. (2) on the constraint rows: dot_r = sum_e val[e] x[col[e]], then per
// MODE (as k_aprod1) y[r] += dot, y[r] = dot - coef_u y[r] or
// y[r] = b[r] - dot, and rowssq[r] = y[r]^2 (not in A1_ACCUM).
template <typename Acc, typename VX, typename VY, int MODE>
__global__ __launch_bounds__(kBlock) void k_con_aprod1(int64_t nc,
                                                        const int64_t* __restrict__ rowptr,
                                                        const int64_t* __restrict__ col,
                                                        const double* __restrict__ val,
                                                        const VX* __restrict__ x,
                                                        VY* __restrict__ y,
                                                        const double* __restrict__ b,
                                                        const Scalars* __restrict__ sc,
                                                        double* __restrict__ rowssq)
{
    __shared__ double red[kWavesPerBlock];
    if (MODE == A1_LSQR && sc->done) return;
    const Acc coef = (MODE == A1_LSQR) ? (Acc)sc->coef_u : (Acc)0;
    for (int64_t r = blockIdx.x; r < nc; r += gridDim.x) {
        const int64_t e1 = rowptr[r + 1];
        Acc d = (Acc)0;
        for (int64_t e = rowptr[r] + threadIdx.x; e < e1; e += kBlock)
            d += (Acc)val[e] * (Acc)x[col[e]];
        const double t = block_sum((double)d, red);
        if (threadIdx.x == 0) {
            const Acc dot = (Acc)t;
            if (MODE == A1_ACCUM) {
                y[r] = (VY)((Acc)y[r] + dot);
            } else {
                const VY nv = MODE == A1_LSQR ? (VY)(dot - coef * (Acc)y[r])
                                              : (VY)((Acc)b[r] - dot);
                y[r] = nv;
                rowssq[r] = (double)nv * (double)nv;
            }
        }
    }
}

// Both products of an LSQR step on the constraint rows: u_r = dot_r - coef_u u_r
// (as k_con_aprod1), rowssq[r] = u_r^2, and q[col[e]] += val[e] u_r with the
// new value, by the workgroup that holds the row (its entries are read again
// from L2).
template <typename Acc>
__global__ __launch_bounds__(kBlock) void k_con_step(int64_t nc, const int64_t* __restrict__ rowptr,
                                                      const int64_t* __restrict__ col,
                                                      const double* __restrict__ val,
                                                      const Acc* __restrict__ x,
                                                      Acc* __restrict__ u, Acc* __restrict__ q,
                                                      const Scalars* __restrict__ sc,
                                                      double* __restrict__ rowssq)
{
    __shared__ double red[kWavesPerBlock];
    __shared__ Acc nu;
    if (sc->done) return;
    const Acc coef = (Acc)sc->coef_u;
    for (int64_t r = blockIdx.x; r < nc; r += gridDim.x) {
        const int64_t e0 = rowptr[r], e1 = rowptr[r + 1];
        Acc d = (Acc)0;
        for (int64_t e = e0 + threadIdx.x; e < e1; e += kBlock) d += (Acc)val[e] * (Acc)x[col[e]];
        const double t = block_sum((double)d, red);
        if (threadIdx.x == 0) {
            const Acc nv = (Acc)((Acc)t - coef * u[r]);
            u[r] = nv;
            rowssq[r] = (double)nv * (double)nv;
            nu = nv;
        }
        __syncthreads();
        const Acc ur = nu;
        for (int64_t e = e0 + threadIdx.x; e < e1; e += kBlock)
            atomicAdd(&q[col[e]], (Acc)val[e] * ur);
        __syncthreads();  // nu is rewritten for the next row
    }
}

// part[0] = sum of rowssq[0, nc) in a fixed order: the constraint rows' share
// of ||u||^2, stored after the observation rows' partials.
__global__ __launch_bounds__(kBlock) void k_con_ssq(int64_t nc, const double* __restrict__ rowssq,
                                                     double* __restrict__ part)
{
    __shared__ double red[kWavesPerBlock];
    double v = 0.0;
    for (int64_t k = threadIdx.x; k < nc; k += kBlock) v += rowssq[k];
    const double r = block_sum(v, red);
    if (threadIdx.x == 0) part[0] = r;
}

// Eq. (3) on the constraint rows: q[col[e]] += val[e] u[r] (SQUARE: val[e]^2,
// the column norms), device atomics (a column may appear in several rows).
template <typename Acc, typename VU, bool SQUARE>
__global__ __launch_bounds__(kBlock) void k_con_aprod2(int64_t nc,
                                                        const int64_t* __restrict__ rowptr,
                                                        const int64_t* __restrict__ col,
                                                        const double* __restrict__ val,
                                                        const VU* __restrict__ u,
                                                        Acc* __restrict__ q,
                                                        const Scalars* __restrict__ sc)
{
    if (sc != nullptr && sc->done) return;
    for (int64_t r = blockIdx.x; r < nc; r += gridDim.x) {
        const Acc ur = SQUARE ? (Acc)0 : (Acc)u[r];
        const int64_t e1 = rowptr[r + 1];
        for (int64_t e = rowptr[r] + threadIdx.x; e < e1; e += kBlock) {
            const Acc a = (Acc)val[e];
            atomicAdd(&q[col[e]], SQUARE ? a * a : a * ur);
        }
    }
}

// Structure of the constraint rows: rowptr[0] = 0 and non-decreasing (bit 1),
// then, in a second launch once that holds, every column in [0, n) (bit 2).
__global__ __launch_bounds__(kBlock) void k_validate_con_rows(int64_t nc,
                                                               const int64_t* __restrict__ rowptr,
                                                               int32_t* __restrict__ flag)
{
    int32_t bad = 0;
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < nc;
         r += (int64_t)gridDim.x * kBlock) {
        if (r == 0 && rowptr[0] != 0) bad |= 1;
        if (rowptr[r + 1] < rowptr[r]) bad |= 1;
    }
    if (bad) atomicOr(flag, bad);
}

__global__ __launch_bounds__(kBlock) void k_validate_con_cols(int64_t nnz,
                                                               const int64_t* __restrict__ col,
                                                               int64_t n,
                                                               int32_t* __restrict__ flag)
{
    int32_t bad = 0;
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * kBlock)
        if (col[e] < 0 || col[e] >= n) bad |= 2;
    if (bad) atomicOr(flag, bad);
}

// ---------------------------------------------------------- column vectors
// Norm of the new row vector from its partials (part[0, npart), and the squares
// con[0, ncon) of its constraint entries); npart = 0: beta is in the state.
struct BetaView {
    const double* part;
    const double* con;
    int32_t npart, ncon;
};

// beta = ||u~||, v~ = p .* q / beta - beta v ; q = 0 ; alpha^2 partials. The
// slices and partials of the sections that the row passes left in their
// histograms are added to q on the way, so that neither they nor beta take a
// launch of their own. Every workgroup sums the same partials of beta in the
// same order; workgroup 0 stores beta, anorm and beta_zero, which the others
// do not read.
template <typename Acc>
__global__ __launch_bounds__(kBlock) void k_col_a(int64_t n, const double* __restrict__ p,
                                                   Acc* __restrict__ q, double* __restrict__ v,
                                                   Scalars* __restrict__ sc, BetaView bv,
                                                   SliceView att, SliceView ins, GlobView glob,
                                                   double* __restrict__ part)
{
    __shared__ double red[kBlock];
    __shared__ double bsh;
    double t = 0.0;  // loaded beside the flag
    for (int k = threadIdx.x; k < bv.npart; k += kBlock) t += bv.part[k];
    for (int k = threadIdx.x; k < bv.ncon; k += kBlock) t += bv.con[k];
    if (sc->done) return;
    if (bv.npart > 0) {
        const double ssq = block_sum(t, red);
        if (threadIdx.x == 0) {
            const double b = sqrt(ssq);
            bsh = b;
            if (blockIdx.x == 0) {
                sc->beta = b;
                if (b > 0.0) {
                    const double a = sc->alpha;
                    sc->anorm = sqrt(sc->anorm * sc->anorm + a * a + b * b);
                    sc->beta_zero = 0;
                } else {
                    sc->beta_zero = 1;
                }
            }
        }
    } else if (threadIdx.x == 0) {
        bsh = sc->beta;
    }
    __syncthreads();
    const double beta = bsh;
    if (!(beta > 0.0)) return;
    const double ib = 1.0 / beta;
    double ssq = 0.0;
    auto column = [&](int64_t j, double sum) {
        const double qj = (double)q[j] + sum;
        q[j] = (Acc)0;
        const double vt = p[j] * qj * ib - beta * v[j];
        v[j] = vt;
        ssq += vt * vt;
    };
    for_columns(att, ins, n - glob.ng, red, column, [&](int64_t j) { column(j, 0.0); });
    for_globals<Acc>(glob, red, column);
    const double r = block_sum(ssq, red);
    if (threadIdx.x == 0) part[blockIdx.x] = r;
}

// alpha_{i+1} = ||v~|| and the plane rotation eliminating beta_{i+1}.
__device__ __forceinline__ void rotate_update(Scalars& s, double ssq)
{
    double alpha = s.alpha;
    if (!s.beta_zero) alpha = sqrt(ssq);
    const double beta = s.beta;
    const double rhobar = s.rhobar;
    const double rho = sqrt(rhobar * rhobar + beta * beta);
    const double c = rhobar / rho;
    const double sn = beta / rho;
    const double theta = sn * alpha;
    const double phi = c * s.phibar;
    s.alpha = alpha;
    s.rho = rho;
    s.c = c;
    s.s = sn;
    s.theta = theta;
    s.rhobar = -c * alpha;
    s.phi = phi;
    s.phibar = sn * s.phibar;
    s.t1 = phi / rho;
    s.t2 = -theta / rho;
    s.inv_alpha = alpha > 0.0 ? 1.0 / alpha : 1.0;
    s.coef_u = beta > 0.0 ? alpha / beta : 0.0;
    s.rnorm = s.phibar;
    s.arnorm = alpha * fabs(c) * s.phibar;
}

// Place of column j of the attitude section in the interleaved copy vp3.
__device__ __forceinline__ int64_t att_place(int64_t c, int64_t n_dfa)
{
    const int ax = (c >= n_dfa) + (c >= 2 * n_dfa);
    return kAxes * (c - ax * n_dfa) + ax;
}

// alpha and the rotation, v = v~/alpha ; vp = p .* v (and its attitude section
// interleaved by axis, vp3, when there is one) ; y += t1 w ; w = v + t2 w ;
// partials of ||w/rho||^2 and ||y||^2 ; var (optional) += (w/rho)^2, the
// per-iteration variance term of Algorithm 1 (diagonal estimate of
// (Abar^T Abar)^-1, rescaled by p^2 after the loop). Every workgroup sums the
// same partc and makes the same rotation from the state A; workgroup 0 stores
// the new state to B, which the stopping tests read (Gate).
template <typename VP>
__global__ __launch_bounds__(kBlock) void k_col_b(int64_t n, const double* __restrict__ p,
                                                   double* __restrict__ v,
                                                   double* __restrict__ w,
                                                   double* __restrict__ y, VP* __restrict__ vp,
                                                   VP* __restrict__ vp3, int64_t att_base,
                                                   int64_t n_dfa, const Scalars* __restrict__ A,
                                                   Scalars* __restrict__ B,
                                                   const double* __restrict__ partc, int npartc,
                                                   double* __restrict__ part_dd,
                                                   double* __restrict__ part_xx,
                                                   double* __restrict__ var)
{
    __shared__ double red[kWavesPerBlock];
    __shared__ double bc[4];
    double t = 0.0;  // loaded beside the flag
    for (int k = threadIdx.x; k < npartc; k += kBlock) t += partc[k];
    if (A->done) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *B = *A;
        return;
    }
    const double ssq = block_sum(t, red);
    if (threadIdx.x == 0) {
        Scalars s = *A;
        rotate_update(s, ssq);
        bc[0] = s.beta_zero ? 1.0 : s.inv_alpha;
        bc[1] = s.t1;
        bc[2] = s.t2;
        bc[3] = 1.0 / s.rho;
        if (blockIdx.x == 0) *B = s;
    }
    __syncthreads();
    const double ia = bc[0], t1 = bc[1], t2 = bc[2], ir = bc[3];
    const int64_t natt = vp3 ? kAxes * n_dfa : 0;
    double dd = 0.0, xx = 0.0;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock) {
        const double vj = v[j] * ia;
        v[j] = vj;
        const VP vpj = (VP)(p[j] * vj);
        vp[j] = vpj;
        const int64_t ca = j - att_base;
        if (ca >= 0 && ca < natt) vp3[att_place(ca, n_dfa)] = vpj;
        const double wj = w[j];
        const double dk = wj * ir;
        dd += dk * dk;
        if (var) var[j] += dk * dk;
        const double yj = y[j] + t1 * wj;
        y[j] = yj;
        xx += yj * yj;
        w[j] = vj + t2 * wj;
    }
    double r = block_sum(dd, red);
    if (threadIdx.x == 0) part_dd[blockIdx.x] = r;
    r = block_sum(xx, red);
    if (threadIdx.x == 0) part_xx[blockIdx.x] = r;
}

// Initial v = v~/alpha_1 ; vp = p .* v (vp3 as in k_col_b) ; w = v ; y = 0.
template <typename VP>
__global__ __launch_bounds__(kBlock) void k_col_init(int64_t n, const double* __restrict__ p,
                                                      double* __restrict__ v,
                                                      double* __restrict__ w,
                                                      double* __restrict__ y,
                                                      VP* __restrict__ vp, VP* __restrict__ vp3,
                                                      int64_t att_base, int64_t n_dfa,
                                                      const Scalars* __restrict__ sc)
{
    const double ia = sc->inv_alpha;
    const int64_t natt = vp3 ? kAxes * n_dfa : 0;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock) {
        const double vj = v[j] * ia;
        v[j] = vj;
        w[j] = vj;
        const VP vpj = (VP)(p[j] * vj);
        vp[j] = vpj;
        const int64_t ca = j - att_base;
        if (ca >= 0 && ca < natt) vp3[att_place(ca, n_dfa)] = vpj;
        y[j] = 0.0;
    }
}

// u~ = b (stored as VU, row i at u[inv[i]] or u[i]) ; FP64 sum of squares of
// the stored values.
template <typename VU>
__global__ __launch_bounds__(kBlock) void k_copy_ssq(int64_t m, const double* __restrict__ b,
                                                      VU* __restrict__ u,
                                                      double* __restrict__ part,
                                                      const int32_t* __restrict__ inv)
{
    __shared__ double red[kWavesPerBlock];
    double ssq = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * kBlock) {
        const VU v = (VU)b[i];
        u[inv ? (int64_t)inv[i] : i] = v;
        ssq += (double)v * (double)v;
    }
    const double r = block_sum(ssq, red);
    if (threadIdx.x == 0) part[blockIdx.x] = r;
}

template <typename V>
__global__ __launch_bounds__(kBlock) void k_fill(int64_t n, V* __restrict__ a, V value)
{
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock)
        a[j] = value;
}

// out = p^2 .* var: the variance estimate re-multiplied by the column
// scaling (Algorithm 1 after the loop)
__global__ __launch_bounds__(kBlock) void k_unprecond_var(int64_t n,
                                                           const double* __restrict__ p,
                                                           const double* __restrict__ var,
                                                           double* __restrict__ out)
{
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock)
        out[j] = p[j] * p[j] * var[j];
}

// x = p .* y (un-preconditioning, Algorithm 1 after the loop)
__global__ __launch_bounds__(kBlock) void k_unprecond(int64_t n, const double* __restrict__ p,
                                                       const double* __restrict__ y,
                                                       double* __restrict__ x)
{
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock)
        x[j] = p[j] * y[j];
}

// Refinement: x += p .* y ; partial maxima of |p .* y| and |x|.
__global__ __launch_bounds__(kBlock) void k_refine_update(int64_t n,
                                                           const double* __restrict__ p,
                                                           const double* __restrict__ y,
                                                           double* __restrict__ x,
                                                           double* __restrict__ part_d,
                                                           double* __restrict__ part_x)
{
    __shared__ double red[kWavesPerBlock];
    double dm = 0.0, xm = 0.0;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock) {
        const double d = p[j] * y[j];
        const double xj = x[j] + d;
        x[j] = xj;
        dm = fmax(dm, fabs(d));
        xm = fmax(xm, fabs(xj));
    }
    double r = block_max(dm, red);
    if (threadIdx.x == 0) part_d[blockIdx.x] = r;
    r = block_max(xm, red);
    if (threadIdx.x == 0) part_x[blockIdx.x] = r;
}

__global__ __launch_bounds__(kBlock) void k_refine_norms(const double* __restrict__ part_d,
                                                          const double* __restrict__ part_x,
                                                          int nblk, Scalars* __restrict__ sc)
{
    __shared__ double red[kWavesPerBlock];
    const double d = max_partials(part_d, nblk, red);
    const double x = max_partials(part_x, nblk, red);
    if (threadIdx.x == 0) {
        sc->dmax = d;
        sc->xmax = x;
    }
}

// ------------------------------------------------------------ scalar kernels
// Start of a solve: beta_1 = ||b||, reset the state.
__global__ __launch_bounds__(kBlock) void k_scalar_init_beta(const double* __restrict__ part,
                                                              int nblk, Scalars* __restrict__ sc)
{
    __shared__ double red[kWavesPerBlock];
    const double ssq = sum_partials(part, nblk, red);
    if (threadIdx.x != 0) return;
    const double beta = sqrt(ssq);
    sc->beta = beta;
    sc->bnorm = beta;
    sc->alpha = 0.0;
    sc->anorm = 0.0;
    sc->ddnorm = 0.0;
    sc->acond = 0.0;
    sc->xnorm = 0.0;
    sc->rnorm = beta;
    sc->arnorm = 0.0;
    sc->itn = 0;
    sc->istop = 0;
    sc->beta_zero = 0;
    sc->done = beta > 0.0 ? 0 : 1;  // b = 0: x = 0 solves it (istop 0)
}

// alpha_1 = ||A^T u_1|| ; rhobar = alpha ; phibar = beta.
__global__ __launch_bounds__(kBlock) void k_scalar_init_alpha(const double* __restrict__ part,
                                                               int nblk, Scalars* __restrict__ sc)
{
    __shared__ double red[kWavesPerBlock];
    const double ssq = sum_partials(part, nblk, red);
    if (threadIdx.x != 0 || sc->done) return;
    const double alpha = sqrt(ssq);
    sc->alpha = alpha;
    sc->rhobar = alpha;
    sc->phibar = sc->beta;
    sc->arnorm = alpha * sc->beta;
    sc->arnorm0 = sc->arnorm;
    sc->inv_alpha = alpha > 0.0 ? 1.0 / alpha : 1.0;
    sc->coef_u = alpha / sc->beta;
    if (sc->arnorm == 0.0) sc->done = 1;  // A^T b = 0: x = 0 (istop 0)
}

// ------------------------------------------------------------------- set-up
// Index validation: bit 1 star out of range, 2 stars not sorted,
// 4 attitude start out of range, 8 instrumental index out of range.
__global__ __launch_bounds__(kBlock) void k_validate(SysView s, int32_t* __restrict__ flag)
{
    int32_t bad = 0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < s.m;
         i += (int64_t)gridDim.x * kBlock) {
        const int64_t st = s.star[i];
        if (st < 0 || st >= s.n_stars) bad |= 1;
        if (i > 0 && s.star[i - 1] > st) bad |= 2;
        if (s.natt > 0) {
            const int64_t t = s.att[i];
            if (t < 0 || t > s.n_dfa - kParAxis) bad |= 4;
        }
        for (int j = 0; j < s.ni; ++j) {
            const int32_t c = s.instr[j * s.m + i];
            if (c < 0 || (int64_t)c >= s.n_instr_cols) bad |= 8;
        }
    }
    if (bad) atomicOr(flag, bad);
}

// Compact index copies for the fused passes: star as int32, instrumental
// indices as uint16 (the caller checks that they fit).
__global__ __launch_bounds__(kBlock) void k_compact_idx(SysView s, int32_t* __restrict__ star32,
                                                         uint16_t* __restrict__ instr16)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < s.m;
         i += (int64_t)gridDim.x * kBlock) {
        star32[i] = (int32_t)s.star[i];
#pragma unroll
        for (int j = 0; j < kInstr; ++j)
            if (j < s.ni) instr16[j * s.m + i] = (uint16_t)s.instr[j * s.m + i];
    }
}

// Star-aligned row boundaries: range g starts at the first star boundary at
// or after g*m/nw, so that no star is split between two waves.
template <typename K>
__global__ __launch_bounds__(kBlock) void k_wave_bounds(const K* __restrict__ star,
                                                         int64_t m, int64_t nw,
                                                         int64_t* __restrict__ wb)
{
    const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (g > nw) return;
    if (g == nw) {
        wb[g] = m;
        return;
    }
    int64_t r = g * m / nw;  // g <= nw <= 2^20, m < 2^40: no overflow
    while (r > 0 && r < m && star[r] == star[r - 1]) ++r;
    wb[g] = r;
}

// p_j = 1/sqrt(ssq_j), 1 for an empty column (or for every column when not
// preconditioning); resets ssq.
__global__ __launch_bounds__(kBlock) void k_make_p(int64_t n, double* __restrict__ ssq,
                                                    double* __restrict__ p, int precondition)
{
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock) {
        const double s2 = ssq[j];
        p[j] = (precondition && s2 > 0.0) ? 1.0 / sqrt(s2) : 1.0;
        ssq[j] = 0.0;
    }
}

// ------------------------------------------------ attitude in bucket order
// The attitude columns of a row are 3 windows of 4 consecutive columns at the
// row's start t. Rows stably sorted by the bucket of t (t / W, W starts per
// bucket) put every bucket's rows together while keeping star order inside a
// bucket; the columns one bucket touches are 3 x (W + 3), few enough for an
// LDS histogram, so Eq. (3) for the attitude section becomes a sequential
// sweep with LDS atomics and no device atomics. The solver keeps its row
// vector u~ in this order (row i at u[inv[i]]): the attitude sweep reads it
// sequentially, and the star-order passes reach it through inv, whose targets
// form one run per bucket for any stretch of consecutive rows.
__global__ __launch_bounds__(kBlock) void k_bucket_keys(const int64_t* __restrict__ att, int64_t m,
                                                         int64_t width, int32_t* __restrict__ keys,
                                                         int32_t* __restrict__ rows)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * kBlock) {
        keys[i] = (int32_t)(att[i] / width);
        rows[i] = (int32_t)i;
    }
}

__global__ __launch_bounds__(kBlock) void k_invert_perm(const int32_t* __restrict__ perm, int64_t m,
                                                         int32_t* __restrict__ invperm)
{
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < m;
         k += (int64_t)gridDim.x * kBlock)
        invperm[perm[k]] = (int32_t)k;
}

// bstart[b] = first sorted position of bucket b (b = 0..nb; empty buckets
// included), from the sorted keys.
__global__ __launch_bounds__(kBlock) void k_bucket_starts(const int32_t* __restrict__ skeys,
                                                           int64_t m, int64_t nb,
                                                           int64_t* __restrict__ bstart)
{
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k <= m;
         k += (int64_t)gridDim.x * kBlock) {
        const int64_t prev = k > 0 ? (int64_t)skeys[k - 1] : -1;
        const int64_t cur = k < m ? (int64_t)skeys[k] : nb;
        for (int64_t b = prev + 1; b <= cur; ++b) bstart[b] = k;
    }
}

// att_sorted[c ld + k] = values[off_att + c][perm[k]], c < 12 (ld >= m: the
// column stride of the copy) ; tloc[k] = t of row perm[k] minus its bucket's
// first start.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_att_gather(const T* __restrict__ val,
                                                        const int64_t* __restrict__ att, int64_t m,
                                                        const int32_t* __restrict__ perm,
                                                        int64_t width, int off_att, int64_t ld,
                                                        T* __restrict__ att_sorted,
                                                        uint16_t* __restrict__ tloc)
{
    constexpr int kAtt = kAxes * kParAxis;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < m;
         k += (int64_t)gridDim.x * kBlock) {
        const int64_t i = perm[k];
#pragma unroll
        for (int c = 0; c < kAtt; ++c) att_sorted[c * ld + k] = val[(off_att + c) * m + i];
        const int64_t t = att[i];
        tloc[k] = (uint16_t)(t - (t / width) * width);  // width < 2^16: a window fits in LDS
    }
}

// Attitude part of Eq. (2) over the rows in bucket order, folded into the
// row vector: u~[k] <- sum_c a_c x[col_c] - coef_u u~[k] for the 12 attitude
// coefficients of row k (u~ in bucket order, coalesced), for K right-hand
// sides (u~ [m][K] row-interleaved, x3 [3 n_dfa][K]). The G workgroups of a
// bucket share its rows as in k_att_hist; the bucket's attitude columns
// [b W, b W + W + 3) of the interleaved copy x3 are staged in LDS first
// (win[j][3 c + axis], 3 (W + 3) KS Acc), so no row gathers from global
// memory. One plane per right-hand side: with the KS values of a column
// together, the random columns of a wave share 1/KS of the LDS banks (1e7 rows,
// 4 right-hand sides: 84% of the LDS cycles were conflicts). KS right-hand sides share one sweep over the rows (one window each);
// K / KS sweeps cover the tile. Frozen RHS (done) keep u~. The fused pass
// (kAttPre) then adds the other sections. SEP: u is a separate bucket-order
// vector that receives the attitude part alone (u[k] <- sum_c a_c x[col_c],
// nothing read), for the fused pass's kAttGather form. att_sorted holds
// coefficient c of bucket-order row k at c ld + k, ld a multiple of 64.
// Row blocks start at the 64-row boundary at or below the bucket's first row
// b0, so every wave reads whole 128-byte lines: a line shared by two waves
// that load at the same time is fetched from memory twice (measured: 1.15x
// the streamed bytes when the blocks started at b0). Lanes below b0 load row
// b0 and store nothing.
// PIPE: each thread issues the loads of its next row before the store of the
// current one. A wave's vector-memory counter retires loads and stores in
// issue order, so a store issued before the next row's loads would be waited
// for together with them (one store round trip per row); after them it is
// not.
// GATED (single right-hand side): the pass makes the previous iteration's
// stopping tests first (Gate); otherwise sc holds the K current states.
template <typename T, typename Acc, int K, int KS, int NT, bool SEP = false,
          bool PIPE = (KS * sizeof(Acc) <= 8), bool GATED = false, bool PLAIN = false>
__global__ __launch_bounds__(NT) void k_att_dot(int64_t ld, const T* __restrict__ att_sorted,
                                                 const uint16_t* __restrict__ tloc,
                                                 const int64_t* __restrict__ bstart,
                                                 int64_t width, int G, int64_t n_dfa,
                                                 const Acc* __restrict__ x3, Acc* __restrict__ u,
                                                 int64_t slices, const Scalars* __restrict__ sc,
                                                 Gate gate = Gate{})
{
    static_assert(K % KS == 0, "sweeps of KS right-hand sides cover the tile");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[2 * kWavesPerBlock];
    __shared__ int32_t gflag;
    GateIn gin = {};
    if constexpr (GATED) gin = gate_load(gate);
    Acc* win = reinterpret_cast<Acc*>(smem_raw);
    const int64_t span = width + kParAxis - 1;
    const SideBySide sb = side_by_side(blockIdx.x, K / KS);
    if (sb.part >= slices) return;
    const int64_t bk = sb.part / G, g = sb.part - bk * G;
    const int64_t c0 = bk * width;
    // columns past n_dfa - 1 are never referenced (t + 3 <= n_dfa - 1)
    const int64_t ncol = span < n_dfa - c0 ? span : n_dfa - c0;
    const int64_t b0 = bstart[bk], r1 = bstart[bk + 1];
    const int64_t a0 = b0 & ~(int64_t)(kWave - 1);
    {
        const int s0 = sb.side * KS;
        uint32_t live = 0;
        Acc coef[KS];
        if constexpr (!GATED) {
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                live |= (sc[s0 + j].done ? 0u : 1u) << j;
                coef[j] = (Acc)sc[s0 + j].coef_u;
            }
            if (live == 0) return;  // uniform over the workgroup
        }
        const int32_t plane = (int32_t)(kAxes * span);
        if constexpr (K == 1) {
            stage<NT>(win, x3 + kAxes * c0, kAxes * ncol);
        } else {
            for (int32_t e = threadIdx.x; e < (int32_t)(kAxes * ncol) * KS; e += NT) {
                const int32_t col = e / KS, j = e - col * KS;
                win[j * plane + col] = x3[(kAxes * c0 + col) * K + s0 + j];
            }
        }
        if constexpr (GATED) {
            if (!gate_open(gate, gin, red, &gflag)) return;
            live = 1u;
            coef[0] = (Acc)gin.coef;
        }
        __syncthreads();
        constexpr int kAtt = kAxes * kParAxis;
        // the attitude dot product of one row from the LDS window
        auto row_dot_win = [&](int64_t tl, const T (&a)[kAtt], Acc (&d)[KS]) {
#pragma unroll
            for (int j = 0; j < KS; ++j) d[j] = (Acc)0;
#pragma unroll
            for (int ax = 0; ax < kAxes; ++ax)
#pragma unroll
                for (int qq = 0; qq < kParAxis; ++qq) {
                    const Acc av = (Acc)a[ax * kParAxis + qq];
                    const Acc* w = win + (kAxes * ((int32_t)tl + qq) + ax);
#pragma unroll
                    for (int j = 0; j < KS; ++j) d[j] += av * w[j * plane];
                }
        };
        const int64_t stride = (int64_t)G * NT;
        if (PIPE) {
            // Three rows in flight, each in its own registers (no copies,
            // which would wait for the loads): a row's loads are issued two
            // rows before it is finished, so a store is only ever waited for
            // two rows after it was issued. Rows past the end repeat the
            // last row: loaded before that row's store, they store the same
            // value again.
            struct Row {
                int64_t tl;
                T a[kAtt];
                Acc uo[KS];
            };
            auto load = [&](Row& r, int64_t k) {
                const int64_t kk = k < b0 ? b0 : k;
                r.tl = ld_stream<PLAIN>(&tloc[kk]);
#pragma unroll
                for (int c = 0; c < kAtt; ++c) r.a[c] = ld_stream<PLAIN>(&att_sorted[c * ld + kk]);
#pragma unroll
                for (int j = 0; j < KS; ++j) r.uo[j] = SEP ? (Acc)0 : u[kk * K + s0 + j];
            };
            auto finish = [&](const Row& r, int64_t k) {
                if (k < b0) return;
                Acc d[KS];
                row_dot_win(r.tl, r.a, d);
#pragma unroll
                for (int j = 0; j < KS; ++j)
                    if (KS == 1 || ((live >> j) & 1u))
                        u[k * K + s0 + j] = SEP ? d[j] : d[j] - coef[j] * r.uo[j];
            };
            int64_t k0 = a0 + g * NT + threadIdx.x;
            if (b0 < r1 && k0 < r1) {
                const int64_t klast = k0 + (r1 - 1 - k0) / stride * stride;
                auto next = [&](int64_t k) { return k < klast ? k + stride : klast; };
                Row A, B, C;
                int64_t k1 = next(k0);
                load(A, k0);
                load(B, k1);
                for (;;) {
                    // scheduling fences keep the issue order of each step:
                    // the loads of the row two ahead, then this row's store
                    const int64_t k2 = next(k1);
                    load(C, k2);
                    __builtin_amdgcn_sched_barrier(0);
                    finish(A, k0);
                    __builtin_amdgcn_sched_barrier(0);
                    const int64_t k3 = next(k2);
                    load(A, k3);
                    __builtin_amdgcn_sched_barrier(0);
                    finish(B, k1);
                    __builtin_amdgcn_sched_barrier(0);
                    const int64_t k4 = next(k3);
                    load(B, k4);
                    __builtin_amdgcn_sched_barrier(0);
                    finish(C, k2);
                    __builtin_amdgcn_sched_barrier(0);
                    if (k2 >= klast) break;  // rows from k3 on repeat the last row
                    k0 = k3;
                    k1 = k4;
                }
            }
        } else {
            for (int64_t k = a0 + g * NT + threadIdx.x; k < r1; k += stride) {
                if (k < b0) continue;
                const int64_t tl = ld_stream<PLAIN>(&tloc[k]);
                T a[kAtt];
#pragma unroll
                for (int c = 0; c < kAtt; ++c) a[c] = ld_stream<PLAIN>(&att_sorted[c * ld + k]);
                Acc d[KS];
                row_dot_win(tl, a, d);
#pragma unroll
                for (int j = 0; j < KS; ++j) {
                    if (!((live >> j) & 1u)) continue;
                    Acc* up = u + k * K + s0 + j;
                    *up = SEP ? d[j] : d[j] - coef[j] * *up;
                }
            }
        }
    }
}

// Attitude part of Eq. (3) over the rows in bucket order. The G workgroups
// of bucket b share its rows in interleaved blocks of NT (workgroup w = b G +
// g takes blocks g, g + G, ..., so the G streams advance through memory
// together): an LDS histogram hist[KS][axis][W + 3] gets a * u for the 12
// coefficients of each of its rows and the KS right-hand sides of one sweep,
// then is stored as S2[w][r][axis][W + 3]; k_slice_reduce adds the slices. The
// histogram and S2 are FP64 whatever Acc is: gfx950's LDS FP64 atomic add
// runs at 7.6x the rate of the FP32 one (measured, random addresses over
// 150 KB: 1550 vs 204 G/s), and the sums are more accurate. U is in bucket
// order ([m][K]); the K / KS sweeps of a tile are workgroups side by side (one sweep
// after the other read every row from memory K / KS times; slices = nbk G).
// Frozen RHS are skipped. GATHER: U is in star order instead, and the row at
// bucket position k is read at U[perm[k]] (a read through the permutation,
// whose targets form one increasing run per bucket).
// PIPE: each thread issues the loads of its next row before the atomics of
// the current one (with GATHER, the current row's read through the
// permutation first: its index came with the previous loads).
// att_sorted and the row blocks as in k_att_dot (64-row aligned; lanes below
// the bucket's first row load that row with a zero weight).
template <typename T, typename Acc, int K, int KS, int NT, bool GATHER = false,
          bool PIPE = (KS <= 2), bool PLAIN = false>
__global__ __launch_bounds__(NT) void k_att_hist(int64_t ld, const T* __restrict__ att_sorted,
                                                  const uint16_t* __restrict__ tloc,
                                                  const int64_t* __restrict__ bstart,
                                                  int64_t width, int G, const Acc* __restrict__ U,
                                                  double* __restrict__ S2, int64_t slices,
                                                  const Scalars* __restrict__ sc,
                                                  const int32_t* __restrict__ perm = nullptr)
{
    static_assert(K % KS == 0, "sweeps of KS right-hand sides cover the tile");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* hist = reinterpret_cast<double*>(smem_raw);
    const int64_t span = width + kParAxis - 1;
    const SideBySide sb = side_by_side(blockIdx.x, K / KS);
    if (sb.part >= slices) return;
    const int64_t bk = sb.part / G, g = sb.part - bk * G;
    const int64_t b0 = bstart[bk], r1 = bstart[bk + 1];
    const int64_t a0 = b0 & ~(int64_t)(kWave - 1);
    {
        const int s0 = sb.side * KS;
        uint32_t live = 0;
#pragma unroll
        for (int j = 0; j < KS; ++j)
            live |= (sc != nullptr && sc[s0 + j].done ? 0u : 1u) << j;
        if (live == 0) return;  // uniform over the workgroup
        for (int64_t e = threadIdx.x; e < kAxes * span * KS; e += NT) hist[e] = 0.0;
        __syncthreads();
        constexpr int kAtt = kAxes * kParAxis;
        auto scatter = [&](int64_t tl, const T (&a)[kAtt], const double (&uk)[KS]) {
#pragma unroll
            for (int ax = 0; ax < kAxes; ++ax)
#pragma unroll
                for (int qq = 0; qq < kParAxis; ++qq)
#pragma unroll
                    for (int j = 0; j < KS; ++j)
                        if ((live >> j) & 1u)
                            atomicAdd(&hist[(j * kAxes + ax) * (int32_t)span + (int32_t)tl + qq],
                                      (double)a[ax * kParAxis + qq] * uk[j]);
        };
        const int64_t stride = (int64_t)G * NT;
        if (PIPE) {
            // Three rows in flight as in k_att_dot; rows past the end repeat
            // the last row with a zero weight. With GATHER a row's value is
            // read through the permutation one step before the row is
            // scattered (its index came with the row's loads).
            struct Row {
                int64_t tl, ku;
                T a[kAtt];
                double uk[KS];
            };
            auto load = [&](Row& r, int64_t k) {
                const int64_t kk = k < b0 ? b0 : k;
                r.tl = ld_stream<PLAIN>(&tloc[kk]);
                r.ku = GATHER ? (int64_t)ld_stream<PLAIN>(&perm[kk]) : kk;
#pragma unroll
                for (int c = 0; c < kAtt; ++c) r.a[c] = ld_stream<PLAIN>(&att_sorted[c * ld + kk]);
                if (!GATHER)
#pragma unroll
                    for (int j = 0; j < KS; ++j) r.uk[j] = (double)U[kk * K + s0 + j];
            };
            auto value = [&](Row& r, double w) {
#pragma unroll
                for (int j = 0; j < KS; ++j)
                    r.uk[j] = w * (GATHER ? (double)U[r.ku * K + s0 + j] : r.uk[j]);
            };
            int64_t k0 = a0 + g * NT + threadIdx.x;
            if (b0 < r1 && k0 < r1) {
                const int64_t klast = k0 + (r1 - 1 - k0) / stride * stride;
                // next row and its weight (0 for a repeat of the last row;
                // only a thread's first row can lie below b0)
                auto next = [&](int64_t k) { return k < klast ? k + stride : klast; };
                Row A, B, C;
                int64_t k1 = next(k0);
                load(A, k0);
                load(B, k1);
                value(A, k0 >= b0 ? 1.0 : 0.0);
                for (;;) {
                    const int64_t k2 = next(k1);
                    value(B, k1 > k0 ? 1.0 : 0.0);
                    load(C, k2);
                    __builtin_amdgcn_sched_barrier(0);
                    scatter(A.tl, A.a, A.uk);
                    __builtin_amdgcn_sched_barrier(0);
                    const int64_t k3 = next(k2);
                    value(C, k2 > k1 ? 1.0 : 0.0);
                    load(A, k3);
                    __builtin_amdgcn_sched_barrier(0);
                    scatter(B.tl, B.a, B.uk);
                    __builtin_amdgcn_sched_barrier(0);
                    const int64_t k4 = next(k3);
                    value(A, k3 > k2 ? 1.0 : 0.0);
                    load(B, k4);
                    __builtin_amdgcn_sched_barrier(0);
                    scatter(C.tl, C.a, C.uk);
                    __builtin_amdgcn_sched_barrier(0);
                    if (k2 >= klast) break;
                    k0 = k3;
                    k1 = k4;
                }
            }
        } else {
            for (int64_t k = a0 + g * NT + threadIdx.x; k < r1; k += stride) {
                if (k < b0) continue;
                const int64_t tl = ld_stream<PLAIN>(&tloc[k]);
                const int64_t ku = GATHER ? (int64_t)ld_stream<PLAIN>(&perm[k]) : k;
                double uk[KS];
#pragma unroll
                for (int j = 0; j < KS; ++j) uk[j] = (double)U[ku * K + s0 + j];
                T a[kAtt];  // all loads issued before the first atomic
#pragma unroll
                for (int c = 0; c < kAtt; ++c) a[c] = ld_stream<PLAIN>(&att_sorted[c * ld + k]);
                scatter(tl, a, uk);
            }
        }
        __syncthreads();
        for (int j = 0; j < KS; ++j) {
            if (!((live >> j) & 1u)) continue;
            double* out = S2 + (sb.part * K + s0 + j) * kAxes * span;
            for (int64_t e = threadIdx.x; e < kAxes * span; e += NT) out[e] = hist[j * kAxes * span + e];
        }
    }
}

// q[(base + axis len + c) K + r] += sum of the slices of every workgroup whose
// histogram holds column c (SliceView). The slices are read along the columns
// (consecutive threads, consecutive columns of one right-hand side), by V.gl
// threads per column; blockIdx.y, gridDim.y split the right-hand sides.
// Bound by the latency of the slice loads where the columns are few (256
// slices of 180 ... 30,000 columns: 44-59 -> 4-6 us), by the bytes of the
// slices otherwise.
// The last blocks (blockIdx.x == gridDim.x - 1) finish the row pass before it
// instead: beta_r = ||u~_r|| and anorm from part[npart][K] (if any), and the
// global columns' partials gpart[nblk][K] added to qglob. Nothing else of this launch reads what they store.
template <typename Acc, int K>
__global__ __launch_bounds__(kBlock) void k_slice_reduce(SliceView V, Acc* __restrict__ q,
                                                          Scalars* __restrict__ sc,
                                                          const double* __restrict__ part,
                                                          int npart,
                                                          const Acc* __restrict__ gpart, int nblk,
                                                          Acc* __restrict__ qglob)
{
    __shared__ double red[kBlock];
    if (blockIdx.x == gridDim.x - 1) {
        for (int r = blockIdx.y; r < K; r += gridDim.y) {
            if (sc[r].done) continue;  // uniform over the block
            double ssq = 0.0, g = 0.0;
            for (int k = threadIdx.x; k < npart; k += kBlock) ssq += part[(int64_t)k * K + r];
            for (int k = threadIdx.x; k < nblk; k += kBlock) g += (double)gpart[(int64_t)k * K + r];
            ssq = block_sum(ssq, red);
            g = block_sum(g, red);
            if (threadIdx.x != 0) continue;
            qglob[r] = (Acc)((double)qglob[r] + g);  // 0 with beta_r = 0
            if (npart == 0) continue;
            Scalars& s = sc[r];
            const double beta = sqrt(ssq);
            s.beta = beta;
            if (beta > 0.0) {
                s.anorm = sqrt(s.anorm * s.anorm + s.alpha * s.alpha + beta * beta);
                s.beta_zero = 0;
            } else {
                s.beta_zero = 1;
            }
        }
        return;
    }
    Acc* __restrict__ qs = q + V.base * K;
    const int64_t total = V.cols(), tiles = V.tiles();
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x - 1) {
        const int64_t col = tile * V.ct() + (threadIdx.x & (V.ct() - 1));
        for (int r = blockIdx.y; r < K; r += gridDim.y) {
            const double sum = slice_tile_sum<K>(V, col < total, col, r, red);
            if (threadIdx.x >= V.ct() || col >= total || sc[r].done) continue;
            qs[col * K + r] = (Acc)((double)qs[col * K + r] + sum);
        }
    }
}

// ====================================================== batched right-hand sides
// K right-hand sides advance together: one row per lane, K values per lane,
// so every coefficient and index of A is read once per K RHS (an SpMM).
// Layouts of one k-tile: U [m][K] (row-interleaved), column vectors [n][K].
// sc points at the tile's K Scalars; a RHS with sc[r].done set is frozen:
// no kernel changes its vectors or scalars any more.
namespace batched {

// Running masks: bit r set when RHS r is still iterating.
template <int K>
__device__ __forceinline__ uint32_t live_mask(const Scalars* __restrict__ sc)
{
    uint32_t mk = 0;
#pragma unroll
    for (int r = 0; r < K; ++r) mk |= (sc[r].done ? 0u : 1u) << r;
    return mk;
}

// K-wide gather of a column vector row [n][K].
template <typename V, int K>
__device__ __forceinline__ void load_k(const V* __restrict__ p, V (&out)[K])
{
#pragma unroll
    for (int r = 0; r < K; ++r) out[r] = p[r];
}

// Deterministic block sums of K doubles per thread into part[blk*K + r].
template <int K>
__device__ __forceinline__ void block_sums_k(double (&v)[K], double* __restrict__ part,
                                             double* lds /* >= K * kWavesPerBlock */)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
    for (int r = 0; r < K; ++r)
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) v[r] += __shfl_down(v[r], off);
    __syncthreads();
    if (lane == 0)
#pragma unroll
        for (int r = 0; r < K; ++r) lds[r * kWavesPerBlock + w] = v[r];
    __syncthreads();
    if (threadIdx.x < K) {
        double s = 0.0;
        for (int k = 0; k < kWavesPerBlock; ++k) s += lds[threadIdx.x * kWavesPerBlock + k];
        part[(int64_t)blockIdx.x * K + threadIdx.x] = s;
    }
}

// U[p(i)][r] = B[i][r] (B row stride ldb; p(i) = inv[i], or i without inv),
// FP64 sums of squares per RHS.
template <typename VU, int K>
__global__ __launch_bounds__(kBlock) void k_copy_ssq(int64_t m, const double* __restrict__ B,
                                                      int64_t ldb, VU* __restrict__ U,
                                                      double* __restrict__ part,
                                                      const int32_t* __restrict__ inv)
{
    __shared__ double red[K * kWavesPerBlock];
    double ssq[K];
#pragma unroll
    for (int r = 0; r < K; ++r) ssq[r] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * kBlock) {
        const int64_t pi = inv ? (int64_t)inv[i] : i;
#pragma unroll
        for (int r = 0; r < K; ++r) {
            const VU v = (VU)B[i * ldb + r];
            U[pi * K + r] = v;
            ssq[r] += (double)v * (double)v;
        }
    }
    block_sums_k<K>(ssq, part, red);
}

// U = A VP - coef_r U per live RHS (row i at U[inv[i]] or U[i]); sums of
// squares of the new U per RHS.
template <typename T, typename Acc, int K>
__global__ __launch_bounds__(kBlock) void k_aprod1(SysView s, const Acc* __restrict__ VP,
                                                    Acc* __restrict__ U,
                                                    const Scalars* __restrict__ sc,
                                                    double* __restrict__ part,
                                                    const int32_t* __restrict__ inv)
{
    __shared__ double red[K * kWavesPerBlock];
    const uint32_t live = live_mask<K>(sc);
    if (live == 0) return;
    Acc coef[K];
#pragma unroll
    for (int r = 0; r < K; ++r) coef[r] = (Acc)sc[r].coef_u;
    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t m = s.m;
    double ssq[K];
#pragma unroll
    for (int r = 0; r < K; ++r) ssq[r] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * kBlock) {
        const int64_t st = ldnt(&s.star[i]);
        const int64_t t = ldnt(&s.att[i]);
        T a[kPar];
#pragma unroll
        for (int c = 0; c < kPar; ++c) a[c] = ldnt(&val[c * m + i]);
        int32_t ic[kInstr];
#pragma unroll
        for (int j = 0; j < kInstr; ++j) ic[j] = ldnt(&s.instr[j * m + i]);
        Acc sum[K];
#pragma unroll
        for (int r = 0; r < K; ++r) sum[r] = (Acc)0;
        Acc xv[K];
#pragma unroll
        for (int j = 0; j < kAstro; ++j) {
            load_k<Acc, K>(VP + (kAstro * st + j) * K, xv);
#pragma unroll
            for (int r = 0; r < K; ++r) sum[r] += (Acc)a[j] * xv[r];
        }
#pragma unroll
        for (int ax = 0; ax < kAxes; ++ax)
#pragma unroll
            for (int qq = 0; qq < kParAxis; ++qq) {
                load_k<Acc, K>(VP + (s.att_base + ax * s.n_dfa + t + qq) * K, xv);
#pragma unroll
                for (int r = 0; r < K; ++r) sum[r] += (Acc)a[kOffAtt + ax * kParAxis + qq] * xv[r];
            }
#pragma unroll
        for (int j = 0; j < kInstr; ++j) {
            load_k<Acc, K>(VP + (s.instr_base + ic[j]) * K, xv);
#pragma unroll
            for (int r = 0; r < K; ++r) sum[r] += (Acc)a[kOffInstr + j] * xv[r];
        }
        load_k<Acc, K>(VP + s.glob_base * K, xv);
#pragma unroll
        for (int r = 0; r < K; ++r) sum[r] += (Acc)a[kOffGlob] * xv[r];
        Acc* u = U + (inv ? (int64_t)ldnt(&inv[i]) : i) * K;
#pragma unroll
        for (int r = 0; r < K; ++r) {
            if (!((live >> r) & 1u)) continue;
            const Acc nu = sum[r] - coef[r] * u[r];
            u[r] = nu;
            ssq[r] += (double)nu * (double)nu;
        }
    }
    block_sums_k<K>(ssq, part, red);
}

// Q += A^T U over star-aligned per-wave ranges (astrometric: accumulate-and-
// flush segments, attitude: device atomics, instrumental: LDS histogram
// [hcols][K] of columns [0, hcols), the others left to k_instr_tail, global:
// partials gpart[blk][K]). Frozen RHS contribute nothing.
template <typename T, typename Acc, int K, bool ATT = true, int NT = kBlock>
__global__ __launch_bounds__(NT) void k_aprod2(SysView s, const Acc* __restrict__ U,
                                                    Acc* __restrict__ Q,
                                                    const int64_t* __restrict__ wb,
                                                    Acc* __restrict__ gpart, int64_t hcols,
                                                    const Scalars* __restrict__ sc,
                                                    const int32_t* __restrict__ inv)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* lds = reinterpret_cast<double*>(smem_raw);
    __shared__ Acc gred[K * (NT / kWave)];
    uint32_t live = 0;
#pragma unroll
    for (int r = 0; r < K; ++r) live |= (sc[r].done ? 0u : 1u) << r;
    if (live == 0) return;
    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t m = s.m;
    for (int64_t j = threadIdx.x; j < hcols * K; j += NT) lds[j] = 0.0;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave = (int64_t)blockIdx.x * (NT / kWave) + threadIdx.x / kWave;
    const int64_t rb = wb[wave], re = wb[wave + 1];
    Acc* __restrict__ qatt = Q + s.att_base * K;
    Acc* __restrict__ qins = Q + s.instr_base * K;
    Acc gsum[K];
#pragma unroll
    for (int r = 0; r < K; ++r) gsum[r] = (Acc)0;
    SegAcc<Acc, kAstro * K> seg;
    auto astro_emit = [Q, lane](int64_t star, const Acc (&v)[kAstro * K]) {
        Acc* dst = Q + kAstro * star * K;
#pragma unroll
        for (int j = 0; j < kAstro * K; ++j) {
            const Acc tot = wave_sum(v[j]);
            if (lane == 0) dst[j] += tot;
        }
    };
    // Chunks start on 64-row boundaries so that every coefficient stream is
    // read in whole cache lines; lanes before rb (owned by the previous wave)
    // take the first row's star with zero contributions.
    for (int64_t r0 = rb < re ? (rb & ~(int64_t)(kWave - 1)) : re; r0 < re; r0 += kWave) {
        const int64_t i = r0 + lane;
        const bool ok = i >= rb && i < re;
        const int64_t ic = i < rb ? rb : (i < re ? i : re - 1);
        const int64_t st = i < re ? ldnt(&s.star[ic]) : kNoStar;
        const int64_t t = ATT ? ldnt(&s.att[ic]) : 0;
        T a[kPar];
#pragma unroll
        for (int c = 0; c < kPar; ++c)
            a[c] = (ATT || c < kOffAtt || c >= kOffInstr) ? ldnt(&val[c * m + ic]) : (T)0;
        int32_t ix[kInstr];
#pragma unroll
        for (int j = 0; j < kInstr; ++j) ix[j] = ldnt(&s.instr[j * m + ic]);
        const int64_t pu = inv ? (int64_t)ldnt(&inv[ic]) : ic;
        Acc u[K];
#pragma unroll
        for (int r = 0; r < K; ++r) u[r] = (ok && ((live >> r) & 1u)) ? U[pu * K + r] : (Acc)0;

        if (ok) {
#pragma unroll
            for (int ax = 0; ax < (ATT ? kAxes : 0); ++ax)
#pragma unroll
                for (int qq = 0; qq < kParAxis; ++qq) {
                    Acc* dst = qatt + (ax * s.n_dfa + t + qq) * K;
                    const Acc av = (Acc)a[kOffAtt + ax * kParAxis + qq];
#pragma unroll
                    for (int r = 0; r < K; ++r)
                        if ((live >> r) & 1u) atomicAdd(dst + r, av * u[r]);
                }
#pragma unroll
            for (int j = 0; j < kInstr; ++j) {
                const Acc av = (Acc)a[kOffInstr + j];
                if (ix[j] >= hcols) continue;
#pragma unroll
                for (int r = 0; r < K; ++r) {
                    if (!((live >> r) & 1u)) continue;
                    atomicAdd(&lds[ix[j] * K + r], (double)(av * u[r]));
                }
            }
        }
#pragma unroll
        for (int r = 0; r < K; ++r) gsum[r] += (Acc)a[kOffGlob] * u[r];
        Acc pa[kAstro * K];
#pragma unroll
        for (int j = 0; j < kAstro; ++j)
#pragma unroll
            for (int r = 0; r < K; ++r) pa[j * K + r] = (Acc)a[j] * u[r];
        seg_chunk(seg, st, pa, lane, astro_emit);
    }
    seg_finish(seg, lane, astro_emit);
#pragma unroll
    for (int r = 0; r < K; ++r) {
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) gsum[r] += __shfl_down(gsum[r], off);
    }
    if (lane == 0)
#pragma unroll
        for (int r = 0; r < K; ++r) gred[r * (NT / kWave) + threadIdx.x / kWave] = gsum[r];
    __syncthreads();
    if (threadIdx.x < K) {
        Acc g = (Acc)0;
        for (int k = 0; k < NT / kWave; ++k) g += gred[threadIdx.x * (NT / kWave) + k];
        gpart[(int64_t)blockIdx.x * K + threadIdx.x] = g;
    }
    for (int64_t j = threadIdx.x; j < hcols * K; j += NT) {
        const double v = lds[j];
        if (v != 0.0) atomicAdd(&qins[j], (Acc)v);
    }
}

// X3[(3 c + axis) K + r] = VP[(att_base + axis n_dfa + c) ld + r]: the
// attitude section interleaved by axis, K values per column kept together
// (ld: row stride of VP, K for a tile's own vectors).
template <typename V, int K>
__global__ __launch_bounds__(kBlock) void k_interleave_att(const V* __restrict__ VP, int64_t ld,
                                                            int64_t att_base, int64_t n_dfa,
                                                            V* __restrict__ X3)
{
    const int64_t total = (int64_t)kAxes * n_dfa * K;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < total;
         j += (int64_t)gridDim.x * kBlock) {
        const int64_t col = j / K, r = j - col * K;
        const int64_t c = col / kAxes, ax = col - c * kAxes;
        X3[j] = VP[(att_base + ax * n_dfa + c) * ld + r];
    }
}

// Refinement residual of a k-tile: U_r = B_r - A X_r for the RHS with bit r
// of `live` set (FP32-stored values widened, FP64 accumulation, stored as
// VU at row i's place inv[i] (or i)), U_r = 0 for the others; FP64 sums of
// squares of the stored values per RHS. X: [n][ldx], B: [m][ldb]; X3: the
// attitude section of X interleaved by axis, K values per column.
template <typename T, typename VU, int K>
__global__ __launch_bounds__(kBlock) void k_resid(SysView s, const double* __restrict__ X,
                                                   int64_t ldx, const double* __restrict__ X3,
                                                   const double* __restrict__ B, int64_t ldb,
                                                   VU* __restrict__ U, double* __restrict__ part,
                                                   const int32_t* __restrict__ inv, uint32_t live)
{
    __shared__ double red[K * kWavesPerBlock];
    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t m = s.m;
    double ssq[K];
#pragma unroll
    for (int r = 0; r < K; ++r) ssq[r] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * kBlock) {
        const int64_t st = ldnt(&s.star[i]);
        const int64_t t = ldnt(&s.att[i]);
        T a[kPar];
#pragma unroll
        for (int c = 0; c < kPar; ++c) a[c] = ldnt(&val[c * m + i]);
        int32_t ic[kInstr];
#pragma unroll
        for (int j = 0; j < kInstr; ++j) ic[j] = ldnt(&s.instr[j * m + i]);
        double d[K];
#pragma unroll
        for (int r = 0; r < K; ++r) d[r] = 0.0;
#pragma unroll
        for (int j = 0; j < kAstro; ++j)
#pragma unroll
            for (int r = 0; r < K; ++r) d[r] += (double)a[j] * X[(kAstro * st + j) * ldx + r];
#pragma unroll
        for (int ax = 0; ax < kAxes; ++ax)
#pragma unroll
            for (int qq = 0; qq < kParAxis; ++qq) {
                const double* xv = X3 + (kAxes * (t + qq) + ax) * K;
                const double av = (double)a[kOffAtt + ax * kParAxis + qq];
#pragma unroll
                for (int r = 0; r < K; ++r) d[r] += av * xv[r];
            }
#pragma unroll
        for (int j = 0; j < kInstr; ++j)
#pragma unroll
            for (int r = 0; r < K; ++r)
                d[r] += (double)a[kOffInstr + j] * X[(s.instr_base + ic[j]) * ldx + r];
#pragma unroll
        for (int r = 0; r < K; ++r) d[r] += (double)a[kOffGlob] * X[s.glob_base * ldx + r];
        VU* u = U + (inv ? (int64_t)ldnt(&inv[i]) : i) * K;
#pragma unroll
        for (int r = 0; r < K; ++r) {
            const VU v = ((live >> r) & 1u) ? (VU)(B[i * ldb + r] - d[r]) : (VU)0;
            u[r] = v;
            ssq[r] += (double)v * (double)v;
        }
    }
    block_sums_k<K>(ssq, part, red);
}

// Refinement step of a k-tile: X_r += p .* Y_r for the RHS with bit r of
// `live` set; per-RHS partial maxima of |p .* Y_r| and |X_r|
// (part_d/part_x [nblk][K]).
template <int K>
__global__ __launch_bounds__(kBlock) void k_refine_update(int64_t n, const double* __restrict__ p,
                                                           const double* __restrict__ Y,
                                                           double* __restrict__ X, int64_t ldx,
                                                           uint32_t live,
                                                           double* __restrict__ part_d,
                                                           double* __restrict__ part_x)
{
    __shared__ double red[kWavesPerBlock];
    double dm[K], xm[K];
#pragma unroll
    for (int r = 0; r < K; ++r) dm[r] = xm[r] = 0.0;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock) {
        const double pj = p[j];
#pragma unroll
        for (int r = 0; r < K; ++r) {
            if (!((live >> r) & 1u)) continue;
            const double d = pj * Y[j * K + r];
            const double xj = X[j * ldx + r] + d;
            X[j * ldx + r] = xj;
            dm[r] = fmax(dm[r], fabs(d));
            xm[r] = fmax(xm[r], fabs(xj));
        }
    }
#pragma unroll
    for (int r = 0; r < K; ++r) {
        double v = block_max(dm[r], red);
        if (threadIdx.x == 0) part_d[(int64_t)blockIdx.x * K + r] = v;
        v = block_max(xm[r], red);
        if (threadIdx.x == 0) part_x[(int64_t)blockIdx.x * K + r] = v;
    }
}

// sc[r].dmax, sc[r].xmax = maxima over the partials of k_refine_update.
template <int K>
__global__ __launch_bounds__(kBlock) void k_refine_norms(const double* __restrict__ part_d,
                                                          const double* __restrict__ part_x,
                                                          int nblk, Scalars* __restrict__ sc)
{
    __shared__ double red[kWavesPerBlock];
    for (int r = 0; r < K; ++r) {
        double v = 0.0, w = 0.0;
        for (int k = threadIdx.x; k < nblk; k += kBlock) {
            v = fmax(v, part_d[(int64_t)k * K + r]);
            w = fmax(w, part_x[(int64_t)k * K + r]);
        }
        const double d = block_max(v, red);
        const double x = block_max(w, red);
        if (threadIdx.x == 0) {
            sc[r].dmax = d;
            sc[r].xmax = x;
        }
    }
}

// X[j][r] = 0 (row stride ldx), r < K
template <int K>
__global__ __launch_bounds__(kBlock) void k_zero_cols(int64_t n, double* __restrict__ X,
                                                       int64_t ldx)
{
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock)
#pragma unroll
        for (int r = 0; r < K; ++r) X[j * ldx + r] = 0.0;
}

// Fused iteration pass of a K-tile (the batched form of the single-RHS fused
// pass): per row, U~_r = Abar VP_r - coef_r U_r for every live RHS r, written
// with its FP64 sum of squares per workgroup (part[blk][K]), and the same
// registers scattered into Q += A^T U~ for the astrometric, instrumental and
// global columns. Frozen RHS keep U and contribute nothing. Dynamic LDS: the
// FP64 histogram [hcols][K] of instrumental columns [0, hcols) (the others
// are left to k_instr_tail), then the instrumental slice of VP (LDSX). In
// 1024-thread workgroups (128 registers per lane) a multi-RHS tile would
// reduce its star segments chunk by chunk instead of carrying 5K running sums;
// the tiles run in 512 or 256 threads, which have the registers. AM as in the single-RHS pass (kAttPre after
// k_att_dot over the tile's K right-hand sides). us (optional): a star-order
// copy of the new U~ (us[i K + r]) for the instrumental tail passes.
template <typename T, typename Acc, int K, int NT, bool LDSX, int AM, bool CIDX>
__global__ __launch_bounds__(NT) void k_fused(SysView s, const Acc* __restrict__ VP,
                                               const Acc* __restrict__ X3, Acc* __restrict__ U,
                                               Acc* __restrict__ Q, const int64_t* __restrict__ wb,
                                               Acc* __restrict__ gpart, double* __restrict__ part,
                                               int64_t hcols, const Scalars* __restrict__ sc,
                                               const int32_t* __restrict__ inv,
                                               Acc* __restrict__ us = nullptr)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ Acc gred[K * (NT / kWave)];
    __shared__ double sred[K * (NT / kWave)];
    const uint32_t live = live_mask<K>(sc);
    if (live == 0) return;
    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t m = s.m;
    const int64_t ninst = s.n_instr_cols;
    double* hist = reinterpret_cast<double*>(smem_raw);
    const Acc* xi = VP + s.instr_base * K;
    for (int64_t j = threadIdx.x; j < hcols * K; j += NT) hist[j] = 0.0;
    if (LDSX) {
        const int64_t off = (hcols * K * 8 + 15) & ~(int64_t)15;
        Acc* xl = reinterpret_cast<Acc*>(smem_raw + off);
        for (int64_t j = threadIdx.x; j < ninst * K; j += NT) xl[j] = xi[j];
        xi = xl;
    }
    __syncthreads();

    Acc coef[K], xg[K];
#pragma unroll
    for (int r = 0; r < K; ++r) {
        coef[r] = (Acc)sc[r].coef_u;
        xg[r] = VP[s.glob_base * K + r];
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave = (int64_t)blockIdx.x * (NT / kWave) + threadIdx.x / kWave;
    const int64_t rb = wb[wave], re = wb[wave + 1];
    Acc* __restrict__ qins = Q + s.instr_base * K;
    double ssq[K];
    Acc gsum[K];
#pragma unroll
    for (int r = 0; r < K; ++r) {
        ssq[r] = 0.0;
        gsum[r] = (Acc)0;
    }
    constexpr bool kChunkFlush = NT > 512 && K > 1;
    SegAcc<Acc, kChunkFlush ? 1 : kAstro * K> seg;
    auto astro_emit = [Q, lane](int64_t star, const Acc (&v)[kAstro * K]) {
        Acc* dst = Q + kAstro * star * K;
#pragma unroll
        for (int j = 0; j < kAstro * K; ++j) {
            const Acc tot = wave_sum(v[j]);
            if (lane != 0) continue;
            if (kChunkFlush) dst[j] += tot;  // a star in several pieces
            else dst[j] = tot;
        }
    };
    for (int64_t r0 = rb < re ? (rb & ~(int64_t)(kWave - 1)) : re; r0 < re; r0 += kWave) {
        const int64_t i = r0 + lane;
        const bool ok = i >= rb && i < re;
        const int64_t ic = i < rb ? rb : (i < re ? i : re - 1);
        const int64_t stc = star_of<CIDX>(s, ic);
        const int64_t st = i < re ? stc : kNoStar;
        const int64_t t = AM == kAttPre ? 0 : ldnt(&s.att[ic]);
        T a[kPar];
#pragma unroll
        for (int c = 0; c < kPar; ++c)
            if (AM != kAttPre || c < kOffAtt || c >= kOffInstr) a[c] = ldnt(&val[c * m + ic]);
        int32_t ix[kInstr];
#pragma unroll
        for (int j = 0; j < kInstr; ++j) ix[j] = instr_of<CIDX>(s, j, ic);

        const int64_t pu = inv ? (int64_t)ldnt(&inv[ic]) : ic;
        Acc d[K];
#pragma unroll
        for (int r = 0; r < K; ++r) d[r] = (Acc)0;
        const Acc* xa = VP + kAstro * stc * K;
#pragma unroll
        for (int j = 0; j < kAstro; ++j)
#pragma unroll
            for (int r = 0; r < K; ++r) d[r] += (Acc)a[j] * xa[j * K + r];
        if (AM != kAttPre) {
#pragma unroll
            for (int ax = 0; ax < kAxes; ++ax)
#pragma unroll
                for (int qq = 0; qq < kParAxis; ++qq) {
                    const Acc* xv = AM == kAttX3 ? X3 + (kAxes * (t + qq) + ax) * K
                                                 : VP + (s.att_base + ax * s.n_dfa + t + qq) * K;
                    const Acc av = (Acc)a[kOffAtt + ax * kParAxis + qq];
#pragma unroll
                    for (int r = 0; r < K; ++r) d[r] += av * xv[r];
                }
        }
#pragma unroll
        for (int j = 0; j < kInstr; ++j)
#pragma unroll
            for (int r = 0; r < K; ++r) d[r] += (Acc)a[kOffInstr + j] * xi[ix[j] * K + r];
#pragma unroll
        for (int r = 0; r < K; ++r) {
            d[r] += (Acc)a[kOffGlob] * xg[r];
            const bool on = ok && ((live >> r) & 1u);
            // kAttPre: U already holds the attitude part minus coef U
            const Acc nu = AM == kAttPre ? d[r] + U[pu * K + r] : d[r] - coef[r] * U[pu * K + r];
            if (on) U[pu * K + r] = nu;
            if (on && us) us[ic * K + r] = nu;
            d[r] = on ? nu : (Acc)0;
            ssq[r] += (double)d[r] * (double)d[r];
        }
        if (ok) {
#pragma unroll
            for (int j = 0; j < kInstr; ++j) {
                if (ix[j] >= hcols) continue;
                const Acc av = (Acc)a[kOffInstr + j];
#pragma unroll
                for (int r = 0; r < K; ++r) {
                    if (!((live >> r) & 1u)) continue;
                    atomicAdd(&hist[ix[j] * K + r], (double)(av * d[r]));
                }
            }
        }
#pragma unroll
        for (int r = 0; r < K; ++r) gsum[r] += (Acc)a[kOffGlob] * d[r];
        Acc pa[kAstro * K];
#pragma unroll
        for (int j = 0; j < kAstro; ++j)
#pragma unroll
            for (int r = 0; r < K; ++r) pa[j * K + r] = (Acc)a[j] * d[r];
        if (kChunkFlush) {
            seg_flush(st, pa, lane, astro_emit);
        } else {
            if constexpr (!kChunkFlush) seg_chunk(seg, st, pa, lane, astro_emit);
        }
    }
    if constexpr (!kChunkFlush) seg_finish(seg, lane, astro_emit);
#pragma unroll
    for (int r = 0; r < K; ++r) {
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            gsum[r] += __shfl_down(gsum[r], off);
            ssq[r] += __shfl_down(ssq[r], off);
        }
    }
    if (lane == 0)
#pragma unroll
        for (int r = 0; r < K; ++r) {
            gred[r * (NT / kWave) + threadIdx.x / kWave] = gsum[r];
            sred[r * (NT / kWave) + threadIdx.x / kWave] = ssq[r];
        }
    __syncthreads();
    if (threadIdx.x < K) {
        Acc g = (Acc)0;
        double q2 = 0.0;
        for (int k = 0; k < NT / kWave; ++k) {
            g += gred[threadIdx.x * (NT / kWave) + k];
            q2 += sred[threadIdx.x * (NT / kWave) + k];
        }
        gpart[(int64_t)blockIdx.x * K + threadIdx.x] = g;
        part[(int64_t)blockIdx.x * K + threadIdx.x] = q2;
    }
    for (int64_t j = threadIdx.x; j < hcols * K; j += NT) {
        const double v = hist[j];
        if (v != 0.0) atomicAdd(&qins[j], (Acc)v);
    }
}

// ---- right-hand sides across lanes (k_fused_rl)
// In this layout lane l of a wave handles row slot l / K and right-hand side
// l % K, so a wave steps over R = 64 / K rows at a time and every lane holds
// one RHS value, as in the single-RHS pass (registers do not grow with K).
// Sum over the R row slots of the lanes of one RHS (lanes equal mod K); the
// result is in every lane.
template <int K, typename V>
__device__ __forceinline__ V rhs_sum(V v)
{
#pragma unroll
    for (int off = K; off < kWave; off <<= 1) v += __shfl_xor(v, off);
    return v;
}

// Per-star segmented sums (SegAcc) in the RHS-across-lanes layout: the keys
// of the K lanes of a row slot are equal, segments are runs of row slots;
// emit(key, values) runs on the whole wave once per finished segment.
template <typename Acc, int K, typename Emit>
__device__ __forceinline__ void seg_chunk_rl(SegAcc<Acc, kAstro>& S, int64_t key,
                                             const Acc (&v)[kAstro], int lane, Emit&& emit)
{
    const bool cont = key == S.key;
#pragma unroll
    for (int j = 0; j < kAstro; ++j) S.acc[j] += cont ? v[j] : (Acc)0;
    uint64_t rest = __ballot(!cont);
    if (rest == 0) return;
    if (S.key >= 0) {
        emit(S.key, S.acc);
    }
    S.key = -1;
#pragma unroll
    for (int j = 0; j < kAstro; ++j) S.acc[j] = (Acc)0;
    while (rest != 0) {
        const int l0 = __ffsll((unsigned long long)rest) - 1;
        const int64_t k2 = __shfl(key, l0);
        if (k2 == kNoStar) break;
        const bool mine = key == k2;
        const uint64_t same = __ballot(mine);
        if ((same >> (kWave - 1)) & 1ull) {  // reaches the last row slot: stays open
            S.key = k2;
#pragma unroll
            for (int j = 0; j < kAstro; ++j) S.acc[j] = mine ? v[j] : (Acc)0;
            break;
        }
        Acc t[kAstro];
#pragma unroll
        for (int j = 0; j < kAstro; ++j) t[j] = mine ? v[j] : (Acc)0;
        emit(k2, t);
        rest &= ~same;
    }
}

template <typename Acc, int K, typename Emit>
__device__ __forceinline__ void seg_finish_rl(SegAcc<Acc, kAstro>& S, int lane, Emit&& emit)
{
    if (S.key < 0) return;
    emit(S.key, S.acc);
    S.key = -1;
}

// Lane q of each group of K in {2, 4} lanes broadcast to the group (a quad
// permutation: lane p of a quad reads lane (p & ~(K - 1)) + q), in VALU
// cross-lane moves, without LDS. Every lane of the wave must be active.
template <int K, int Q>
__device__ __forceinline__ int32_t group_bcast(int32_t v)
{
    static_assert((K == 2 || K == 4) && Q < K, "groups of 2 or 4 lanes");
    constexpr int s0 = Q, s1 = Q, s2 = (K == 4 ? 0 : 2) + Q, s3 = s2;
    constexpr int ctrl = s0 | (s1 << 2) | (s2 << 4) | (s3 << 6);
    return __builtin_amdgcn_mov_dpp(v, ctrl, 0xf, 0xf, false);
}
template <int K, int Q, typename V>
__device__ __forceinline__ V group_bcast_v(V v)
{
    if constexpr (sizeof(V) == 8) {
        const int64_t b = __builtin_bit_cast(int64_t, v);
        const int32_t lo = group_bcast<K, Q>((int32_t)(b & 0xffffffff));
        const int32_t hi = group_bcast<K, Q>((int32_t)(b >> 32));
        return __builtin_bit_cast(V, (int64_t)(uint32_t)lo | ((int64_t)hi << 32));
    } else if constexpr (sizeof(V) == 4) {
        return __builtin_bit_cast(V, group_bcast<K, Q>(__builtin_bit_cast(int32_t, v)));
    } else {
        return (V)group_bcast<K, Q>((int32_t)v);
    }
}

constexpr int kNaRl = kAstro + kInstr + 1;  // coefficients outside the attitude section
template <int K>
constexpr int rl_nv() { return kNaRl / K; }                // value loads per lane (K = 2, 4)
template <int K>
constexpr int rl_ni() { return (kInstr + K - 1) / K; }     // index loads per lane
__device__ __forceinline__ constexpr int rl_col(int e)
{
    return e < kAstro ? e : kOffInstr + (e - kAstro);
}

// A step reads 64 / K entries of BYTES of a column. Where that is less than a line
// of 128 bytes the next step reads on in it: loaded plain it is then still in L2,
// nontemporal it may be gone (2e7 rows, FP32, 4 right-hand
// sides, a refined solve: 223.3 -> 220.8 ms).
// PL: all loads plain, for a matrix that the last-level cache holds (1.2e6 rows,
// FP64, 4 right-hand sides: 9.05 -> 8.69 ms; 1e7 rows 286.5 -> 290.0 ms).
template <bool PL, int K, int BYTES>
constexpr bool rl_plain()
{
    return PL || kWave / K * BYTES < 128;
}

// The loads of load_row_rl for K in {2, 4}, before the broadcast: lane r of a
// row slot loads entries r, r + K, ... of the 12 coefficients and 6 indices.
template <typename T, int K, bool CIDX, bool PL>
__device__ __forceinline__ void load_raw_rl(const SysView& s, const T* __restrict__ val,
                                            int64_t ic, int rj, T (&tv)[rl_nv<K>()],
                                            int32_t (&ti)[rl_ni<K>()])
{
    static_assert(K == 2 || K == 4, "row slots of 2 or 4 lanes");
    const int64_t m = s.m;
#pragma unroll
    for (int t = 0; t < rl_nv<K>(); ++t) tv[t] =
        ld_stream<rl_plain<PL, K, sizeof(T)>()>(&val[rl_col(t * K + rj) * m + ic]);
#pragma unroll
    for (int t = 0; t < rl_ni<K>(); ++t) {
        const int j = t * K + rj < kInstr ? t * K + rj : kInstr - 1;
        ti[t] = instr_of<CIDX, rl_plain<PL, K, CIDX ? 2 : 4>()>(s, j, ic);
    }
}

// The broadcast of load_row_rl: each loaded entry to the K lanes of its slot.
template <typename T, int K>
__device__ __forceinline__ void bcast_row_rl(const T (&tv)[rl_nv<K>()],
                                             const int32_t (&ti)[rl_ni<K>()], T (&a)[kPar],
                                             int32_t (&ix)[kInstr])
{
    constexpr int nv = rl_nv<K>(), ni = rl_ni<K>();
    auto col = [](int e) { return rl_col(e); };
#pragma unroll
    for (int t = 0; t < nv; ++t) {
        a[col(t * K + 0)] = group_bcast_v<K, 0>(tv[t]);
        a[col(t * K + 1)] = group_bcast_v<K, 1>(tv[t]);
        if constexpr (K == 4) {
            a[col(t * K + 2)] = group_bcast_v<K, 2>(tv[t]);
            a[col(t * K + 3)] = group_bcast_v<K, 3>(tv[t]);
        }
    }
#pragma unroll
    for (int t = 0; t < ni; ++t) {
        if (t * K + 0 < kInstr) ix[t * K + 0] = group_bcast<K, 0>(ti[t]);
        if (t * K + 1 < kInstr) ix[t * K + 1] = group_bcast<K, 1>(ti[t]);
        if constexpr (K == 4) {
            if (t * K + 2 < kInstr) ix[t * K + 2] = group_bcast<K, 2>(ti[t]);
            if (t * K + 3 < kInstr) ix[t * K + 3] = group_bcast<K, 3>(ti[t]);
        }
    }
}

// The 12 coefficients of row ic outside the attitude section (astrometric,
// instrumental, global) and its 6 instrumental indices, loaded by the K lanes
// of its row slot together: lane r of the slot loads entries r, r + K, ...
// and each entry is then broadcast to the K lanes (K in {2, 4}); for other
// K every lane loads all of them.
template <typename T, int K, bool CIDX, bool PL>
__device__ __forceinline__ void load_row_rl(const SysView& s, const T* __restrict__ val,
                                            int64_t ic, int rj, T (&a)[kPar],
                                            int32_t (&ix)[kInstr])
{
    if constexpr (K == 2 || K == 4) {
        T tv[rl_nv<K>()];
        int32_t ti[rl_ni<K>()];
        load_raw_rl<T, K, CIDX, PL>(s, val, ic, rj, tv, ti);
        bcast_row_rl<T, K>(tv, ti, a, ix);
    } else {
        const int64_t m = s.m;
#pragma unroll
        for (int e = 0; e < kNaRl; ++e)
            a[rl_col(e)] = ld_stream<rl_plain<PL, K, sizeof(T)>()>(&val[rl_col(e) * m + ic]);
#pragma unroll
        for (int j = 0; j < kInstr; ++j) ix[j] = instr_of<CIDX, rl_plain<PL, K, CIDX ? 2 : 4>()>(s, j, ic);
    }
}

// The fused pass of a K-tile after the attitude pre-pass (fused modes 2 and
// 3) with the K right-hand sides of a row in K lanes: per row and live RHS r,
// U~_r = (attitude part already in U) + the other sections' products with
// VP_r, written with its FP64 sum of squares, and the same value scattered
// into Q += A^T U~ for the astrometric (per-star segments), instrumental (LDS
// histogram [hcols][K], the rest to k_instr_tail) and global (partials
// gpart[blk][K]) columns. A2: aprod2 alone (Q += A^T U, U not changed, no
// sums of squares), the start of a tile's solve. U row i at U[inv[i] K + r].
// PIPE (K in {2, 4}, not A2): two row steps in flight per wave. A step waits
// for its coefficient, index, star and permutation loads, then for the
// gathers they address (U through inv, the astrometric and instrumental
// values of VP); the loads of the next step are issued before the gathers of
// the current one, so each step waits one round trip instead of two. Each
// step keeps its loads in its own registers (no copies, which would wait).
template <typename T, typename Acc, int K, int NT, bool LDSX, bool CIDX, bool A2,
          bool PIPE = false, bool PL = false>
__global__ __launch_bounds__(NT) void k_fused_rl(SysView s, const Acc* __restrict__ VP,
                                                  Acc* __restrict__ U, Acc* __restrict__ Q,
                                                  const int64_t* __restrict__ wb,
                                                  Acc* __restrict__ gpart,
                                                  double* __restrict__ part, int64_t hcols,
                                                  const Scalars* __restrict__ sc,
                                                  const int32_t* __restrict__ inv)
{
    constexpr int R = kWave / K;  // row slots of a wave
    constexpr int W = NT / kWave;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ Acc gred[W * K];
    __shared__ double sred[W * K];
    uint32_t live = 0;
#pragma unroll
    for (int r = 0; r < K; ++r)
        live |= (sc[r].done ? 0u : 1u) << r;
    if (live == 0) return;
    const T* __restrict__ val = static_cast<const T*>(s.val);
    const int64_t ninst = s.n_instr_cols;
    double* hist = reinterpret_cast<double*>(smem_raw);
    const Acc* xi = VP + s.instr_base * K;
    for (int64_t e = threadIdx.x; e < hcols * K; e += NT) hist[e] = 0.0;
    if (LDSX && !A2) {
        const int64_t off = (hcols * K * 8 + 15) & ~(int64_t)15;
        Acc* xl = reinterpret_cast<Acc*>(smem_raw + off);
        for (int64_t e = threadIdx.x; e < ninst * K; e += NT) xl[e] = xi[e];
        xi = xl;
    }
    __syncthreads();

    const int lane = threadIdx.x & (kWave - 1);
    const int rj = lane & (K - 1);    // this lane's right-hand side
    const int slot = lane / K;        // and row slot
    const bool lj = (live >> rj) & 1u;
    const Acc xg = A2 ? (Acc)0 : VP[s.glob_base * K + rj];
    // The wave's rows (a bucket order has fewer than 2^31), in scalar registers where
    // the instrumental slice is in LDS; where it is not, that makes the compiler
    // spill two registers a step at K = 4 (FP64: 15% slower).
    uint32_t rb, re;
    if constexpr (LDSX) {
        const int32_t wave = uniform((int32_t)(blockIdx.x * W + threadIdx.x / kWave));
        rb = (uint32_t)uniform((int32_t)wb[wave]);
        re = (uint32_t)uniform((int32_t)wb[wave + 1]);
    } else {
        const int64_t wave = (int64_t)blockIdx.x * W + threadIdx.x / kWave;
        rb = (uint32_t)wb[wave];
        re = (uint32_t)wb[wave + 1];
    }
    Acc* __restrict__ qins = Q + s.instr_base * K;
    double ssq = 0.0;
    Acc gsum = (Acc)0;
    SegAcc<Acc, kAstro> seg;
    auto astro_emit = [Q, lane](int64_t star, const Acc (&v)[kAstro]) {
        star_put<K>(v, lane, [&](int j, int r, Acc sum) {
            Acc* dst = Q + (kAstro * star + j) * K + r;
            if (A2) *dst += sum;
            else *dst = sum;  // as in the single-RHS pass
        });
    };
    // one R-row step: the row of slot `slot` (clamped), its coefficients,
    // indices, star and place in U already loaded
    auto step = [&](uint32_t r0, int64_t stc, const T (&a)[kPar], const int32_t (&ix)[kInstr],
                    int64_t pu) {
        const uint32_t i = r0 + slot;
        const bool ok = i >= rb && i < re;
        const int64_t st = i < re ? stc : kNoStar;
        const Acc uo = U[pu * K + rj];
        const bool on = ok && lj;
        Acc d;
        if (A2) {
            d = on ? uo : (Acc)0;
        } else {
            // Eq. (2): the row's non-attitude products with VP_r, added to
            // the attitude part the pre-pass left in U
            Acc dot = (Acc)0;
            const Acc* xa = VP + kAstro * stc * K + rj;
#pragma unroll
            for (int j = 0; j < kAstro; ++j) dot += (Acc)a[j] * xa[j * K];
#pragma unroll
            for (int j = 0; j < kInstr; ++j) {
                // compact indices: offsets below 65536 x 16 x 8 bytes
                const Acc x = !LDSX && CIDX ? ld_off<true>(xi, (uint32_t)(ix[j] * K + rj))
                                            : xi[ix[j] * K + rj];
                dot += (Acc)a[kOffInstr + j] * x;
            }
            dot += (Acc)a[kOffGlob] * xg;
            const Acc nu = dot + uo;
            if (on) U[pu * K + rj] = nu;
            d = on ? nu : (Acc)0;
            ssq += (double)d * (double)d;
        }
        // Eq. (3) with the new value, attitude columns excluded
        if (on) {
#pragma unroll
            for (int j = 0; j < kInstr; ++j)
                if (ix[j] < hcols)
                    atomicAdd(&hist[ix[j] * K + rj], (double)((Acc)a[kOffInstr + j] * d));
        }
        gsum += (Acc)a[kOffGlob] * d;
        Acc pa[kAstro];
#pragma unroll
        for (int j = 0; j < kAstro; ++j) pa[j] = (Acc)a[j] * d;
        seg_chunk_rl<Acc, K>(seg, st, pa, lane, astro_emit);
    };
    // R-row steps aligned to R rows (every coefficient stream read in whole
    // R-row pieces); slots outside [rb, re) use a clamped row and contribute
    // nothing
    auto row_of = [&](uint32_t r0) -> int64_t {
        const uint32_t i = r0 + slot;
        return i < rb ? rb : (i < re ? i : re - 1);
    };
    const uint32_t rstart = rb < re ? (rb & ~(uint32_t)(R - 1)) : re;
    if constexpr (PIPE && (K == 2 || K == 4) && !A2) {
        struct Raw {
            T tv[rl_nv<K>()];
            int32_t ti[rl_ni<K>()];
            std::conditional_t<CIDX, int32_t, int64_t> stc;
            int32_t pu;
        };
        auto load = [&](Raw& w, uint32_t r0) {
            const int64_t ic = row_of(r0);
            w.stc = (decltype(w.stc))star_of<CIDX, rl_plain<PL, K, 4>()>(s, ic);
            load_raw_rl<T, K, CIDX, PL>(s, val, ic, rj, w.tv, w.ti);
            w.pu = inv ? ld_stream<rl_plain<PL, K, 4>()>(&inv[ic]) : (int32_t)ic;
        };
        auto run = [&](const Raw& w, uint32_t r0) {
            T a[kPar];
            int32_t ix[kInstr];
            bcast_row_rl<T, K>(w.tv, w.ti, a, ix);
            step(r0, w.stc, a, ix, w.pu);
        };
        // r0, re and R are uniform over the wave, so are the branches
        if (rstart < re) {
            Raw A, B;
            uint32_t r0 = rstart;
            load(A, r0);
            for (;;) {
                const uint32_t r1 = r0 + R;
                if (r1 < re) load(B, r1);
                __builtin_amdgcn_sched_barrier(0);
                run(A, r0);
                __builtin_amdgcn_sched_barrier(0);
                if (r1 >= re) break;
                const uint32_t r2 = r1 + R;
                if (r2 < re) load(A, r2);
                __builtin_amdgcn_sched_barrier(0);
                run(B, r1);
                __builtin_amdgcn_sched_barrier(0);
                if (r2 >= re) break;
                r0 = r2;
            }
        }
    } else {
        for (uint32_t r0 = rstart; r0 < re; r0 += R) {
            const int64_t ic = row_of(r0);
            const int64_t stc = star_of<CIDX, rl_plain<PL, K, 4>()>(s, ic);
            T a[kPar];
            int32_t ix[kInstr];
            load_row_rl<T, K, CIDX, PL>(s, val, ic, rj, a, ix);
            const int64_t pu = inv ? (int64_t)ld_stream<rl_plain<PL, K, 4>()>(&inv[ic]) : ic;
            step(r0, stc, a, ix, pu);
        }
    }
    seg_finish_rl<Acc, K>(seg, lane, astro_emit);
    gsum = rhs_sum<K>(gsum);
    ssq = rhs_sum<K>(ssq);
    if (lane < K) {
        gred[(threadIdx.x / kWave) * K + lane] = gsum;
        sred[(threadIdx.x / kWave) * K + lane] = ssq;
    }
    __syncthreads();
    if (threadIdx.x < K) {
        Acc g = (Acc)0;
        double q2 = 0.0;
        for (int w = 0; w < W; ++w) {
            g += gred[w * K + threadIdx.x];
            q2 += sred[w * K + threadIdx.x];
        }
        gpart[(int64_t)blockIdx.x * K + threadIdx.x] = g;
        if (!A2) part[(int64_t)blockIdx.x * K + threadIdx.x] = q2;
    }
    for (int64_t e = threadIdx.x; e < hcols * K; e += NT) {
        const double v = hist[e];
        if (v != 0.0) atomicAdd(&qins[e], (Acc)v);
    }
}

// V~ = p Q / beta_r - beta_r V ; Q = 0 ; alpha^2 partials per RHS.
template <typename Acc, int K>
__global__ __launch_bounds__(kBlock) void k_col_a(int64_t n, const double* __restrict__ p,
                                                   Acc* __restrict__ Q, double* __restrict__ V,
                                                   const Scalars* __restrict__ sc,
                                                   double* __restrict__ part)
{
    __shared__ double red[K * kWavesPerBlock];
    double beta[K], ib[K], ssq[K];
    uint32_t act = 0;
#pragma unroll
    for (int r = 0; r < K; ++r) {
        beta[r] = sc[r].beta;
        ib[r] = beta[r] > 0.0 ? 1.0 / beta[r] : 0.0;
        ssq[r] = 0.0;
        act |= ((sc[r].done || sc[r].beta_zero) ? 0u : 1u) << r;
    }
    if (act == 0) return;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock) {
        const double pj = p[j];
#pragma unroll
        for (int r = 0; r < K; ++r) {
            if (!((act >> r) & 1u)) continue;
            const double qj = (double)Q[j * K + r];
            Q[j * K + r] = (Acc)0;
            const double vt = pj * qj * ib[r] - beta[r] * V[j * K + r];
            V[j * K + r] = vt;
            ssq[r] += vt * vt;
        }
    }
    block_sums_k<K>(ssq, part, red);
}

// FOLD: the attitude section of VP is also kept interleaved by axis, X3.
template <typename VP, int K, bool FOLD>
__global__ __launch_bounds__(kBlock) void k_col_b(int64_t n, const double* __restrict__ p,
                                                   double* __restrict__ V, double* __restrict__ W,
                                                   double* __restrict__ Y, VP* __restrict__ VPv,
                                                   VP* __restrict__ X3, int64_t att_base,
                                                   int64_t n_dfa, const Scalars* __restrict__ sc,
                                                   double* __restrict__ part_dd,
                                                   double* __restrict__ part_xx)
{
    __shared__ double red[K * kWavesPerBlock];
    double ia[K], t1[K], t2[K], ir[K], dd[K], xx[K];
    uint32_t act = 0;
#pragma unroll
    for (int r = 0; r < K; ++r) {
        ia[r] = sc[r].beta_zero ? 1.0 : sc[r].inv_alpha;
        t1[r] = sc[r].t1;
        t2[r] = sc[r].t2;
        ir[r] = 1.0 / sc[r].rho;
        dd[r] = 0.0;
        xx[r] = 0.0;
        act |= (sc[r].done ? 0u : 1u) << r;
    }
    if (act == 0) return;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock) {
        const double pj = p[j];
        const int64_t ca = j - att_base;
        const int64_t o3 = ca >= 0 && ca < kAxes * n_dfa ? att_place(ca, n_dfa) * K : -1;
#pragma unroll
        for (int r = 0; r < K; ++r) {
            if (!((act >> r) & 1u)) continue;
            const int64_t o = j * K + r;
            const double vj = V[o] * ia[r];
            V[o] = vj;
            const VP vpj = (VP)(pj * vj);
            VPv[o] = vpj;
            if (FOLD && o3 >= 0) X3[o3 + r] = vpj;
            const double wj = W[o];
            const double dk = wj * ir[r];
            dd[r] += dk * dk;
            const double yj = Y[o] + t1[r] * wj;
            Y[o] = yj;
            xx[r] += yj * yj;
            W[o] = vj + t2[r] * wj;
        }
    }
    block_sums_k<K>(dd, part_dd, red);
    block_sums_k<K>(xx, part_xx, red);
}

template <typename VP, int K, bool FOLD>
__global__ __launch_bounds__(kBlock) void k_col_init(int64_t n, const double* __restrict__ p,
                                                      double* __restrict__ V,
                                                      double* __restrict__ W,
                                                      double* __restrict__ Y,
                                                      VP* __restrict__ VPv, VP* __restrict__ X3,
                                                      int64_t att_base, int64_t n_dfa,
                                                      const Scalars* __restrict__ sc)
{
    double ia[K];
#pragma unroll
    for (int r = 0; r < K; ++r) ia[r] = sc[r].inv_alpha;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock) {
        const double pj = p[j];
        const int64_t ca = j - att_base;
        const int64_t o3 = ca >= 0 && ca < kAxes * n_dfa ? att_place(ca, n_dfa) * K : -1;
#pragma unroll
        for (int r = 0; r < K; ++r) {
            const int64_t o = j * K + r;
            const double vj = V[o] * ia[r];
            V[o] = vj;
            W[o] = vj;
            const VP vpj = (VP)(pj * vj);
            VPv[o] = vpj;
            if (FOLD && o3 >= 0) X3[o3 + r] = vpj;
            Y[o] = 0.0;
        }
    }
}

// X[j][r] (row stride ldx) = p_j Y[j][r]
template <int K>
__global__ __launch_bounds__(kBlock) void k_unprecond(int64_t n, const double* __restrict__ p,
                                                       const double* __restrict__ Y,
                                                       double* __restrict__ X, int64_t ldx)
{
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * kBlock) {
        const double pj = p[j];
#pragma unroll
        for (int r = 0; r < K; ++r) X[j * ldx + r] = pj * Y[j * K + r];
    }
}

// Sum of column r of part[nblk][K], one block, fixed order; thread 0.
template <int K>
__device__ __forceinline__ double sum_col(const double* part, int nblk, int r, double* lds)
{
    double v = 0.0;
    for (int k = threadIdx.x; k < nblk; k += kBlock) v += part[(int64_t)k * K + r];
    return block_sum(v, lds);
}

// The single-RHS scalar steps applied per RHS, a block each (K blocks); frozen
// ones are skipped.
template <int K>
__global__ __launch_bounds__(kBlock) void k_scalar_init_beta(const double* __restrict__ part,
                                                              int nblk, Scalars* __restrict__ sc)
{
    __shared__ double red[kWavesPerBlock];
    const int r = blockIdx.x;
    {
        const double ssq = sum_col<K>(part, nblk, r, red);
        if (threadIdx.x == 0) {
            Scalars& s = sc[r];
            const double beta = sqrt(ssq);
            s.beta = beta;
            s.bnorm = beta;
            s.alpha = s.anorm = s.ddnorm = s.acond = s.xnorm = s.arnorm = 0.0;
            s.rnorm = beta;
            s.inv_alpha = 1.0;
            s.itn = 0;
            s.istop = 0;
            s.beta_zero = 0;
            s.done = beta > 0.0 ? 0 : 1;
        }
    }
}

template <int K>
__global__ __launch_bounds__(kBlock) void k_scalar_init_alpha(const double* __restrict__ part,
                                                               int nblk, Scalars* __restrict__ sc)
{
    __shared__ double red[kWavesPerBlock];
    const int r = blockIdx.x;
    {
        const double ssq = sum_col<K>(part, nblk, r, red);
        if (threadIdx.x == 0 && !sc[r].done) {
            Scalars& s = sc[r];
            const double alpha = sqrt(ssq);
            s.alpha = alpha;
            s.rhobar = alpha;
            s.phibar = s.beta;
            s.arnorm = alpha * s.beta;
            s.arnorm0 = s.arnorm;
            s.inv_alpha = alpha > 0.0 ? 1.0 / alpha : 1.0;
            s.coef_u = alpha / s.beta;
            if (s.arnorm == 0.0) s.done = 1;
        }
    }
}

template <int K>
__global__ __launch_bounds__(kBlock) void k_scalar_alpha(const double* __restrict__ part,
                                                          int nblk, Scalars* __restrict__ sc)
{
    __shared__ double red[kWavesPerBlock];
    const int r = blockIdx.x;
    {
        if (sc[r].done) return;
        const double ssq = sum_col<K>(part, nblk, r, red);
        if (threadIdx.x == 0) {
            Scalars& s = sc[r];
            double alpha = s.alpha;
            if (!s.beta_zero) alpha = sqrt(ssq);
            const double beta = s.beta;
            const double rho = sqrt(s.rhobar * s.rhobar + beta * beta);
            const double c = s.rhobar / rho;
            const double sn = beta / rho;
            const double theta = sn * alpha;
            const double phi = c * s.phibar;
            s.alpha = alpha;
            s.rho = rho;
            s.c = c;
            s.s = sn;
            s.theta = theta;
            s.rhobar = -c * alpha;
            s.phi = phi;
            s.phibar = sn * s.phibar;
            s.t1 = phi / rho;
            s.t2 = -theta / rho;
            s.inv_alpha = alpha > 0.0 ? 1.0 / alpha : 1.0;
            s.coef_u = beta > 0.0 ? alpha / beta : 0.0;
            s.rnorm = s.phibar;
            s.arnorm = alpha * fabs(c) * s.phibar;
        }
    }
}

template <int K>
__global__ __launch_bounds__(kBlock) void k_scalar_stop(const double* __restrict__ part_dd,
                                                         const double* __restrict__ part_xx,
                                                         int nblk, Scalars* __restrict__ sc)
{
    __shared__ double red[kWavesPerBlock];
    const int r = blockIdx.x;
    {
        if (sc[r].done) return;
        const double dd = sum_col<K>(part_dd, nblk, r, red);
        const double xx = sum_col<K>(part_xx, nblk, r, red);
        if (threadIdx.x == 0) {
            Scalars& s = sc[r];
            const double ddnorm = s.ddnorm + dd;
            const double xnorm = sqrt(xx);
            const double anorm = s.anorm;
            const double acond = anorm * sqrt(ddnorm);
            const double rnorm = s.rnorm, arnorm = s.arnorm, bnorm = s.bnorm;
            s.ddnorm = ddnorm;
            s.xnorm = xnorm;
            s.acond = acond;
            const int32_t itn = s.itn + 1;
            s.itn = itn;
            const double test1 = rnorm / bnorm;
            const double test2 = (anorm * rnorm) > 0.0 ? arnorm / (anorm * rnorm) : 0.0;
            const double test3 = acond > 0.0 ? 1.0 / acond : 0.0;
            const double t1 = test1 / (1.0 + anorm * xnorm / bnorm);
            const double rtol = s.btol + s.atol * anorm * xnorm / bnorm;
            int32_t istop = 0;
            if (itn >= s.itn_limit) istop = 7;
            if (s.tests) {
                if (1.0 + test3 <= 1.0) istop = 6;
                if (1.0 + test2 <= 1.0) istop = 5;
                if (1.0 + t1 <= 1.0) istop = 4;
                if (test3 <= s.ctol) istop = 3;
                if (test2 <= s.atol) istop = 2;
                if (test1 <= rtol) istop = 1;
            }
            // relative normal-equation test of a refinement's inner solve
            if (s.rel_ar > 0.0 && arnorm <= s.rel_ar * s.arnorm0) istop = 2;
            s.istop = istop;
            if (istop != 0) s.done = 1;
        }
    }
}

}  // namespace batched
}  // namespace avugsr
