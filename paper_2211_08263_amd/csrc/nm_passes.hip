// FFT pass kernels of the operator of eq. (Fourier_ND_A) and of the
// reference-medium preconditioner of eqs. (precond)-(acous), for gfx950.
//
// Data layout.  Real fields are SoA [component][z][y][x] with x fastest and are read as pairs of
// neighbouring voxels, V = (x, x + 1).  A transform along y or z of a pair is one complex transform
// that carries two real columns, so the derivatives D_y and D_z (forward transform, i xi / n,
// inverse transform) need no real-to-complex unpacking.  Along x, two neighbouring rows (y, y + 1)
// form one complex line.  Forward transforms are unnormalized.
//
// Passes of one operator apply q = A p.  Every pass is one axis; the derivatives stay in real
// space, and the x pass holds all six strains of its voxels, so D_x never goes to memory:
//   y: D_y p_j (3 -> 3) | z: D_z p_j, joined with D_y p_3 to g23 (4 -> 3) |
//   x: D_x p, strain, sigma = C : eps, Q_j = rho p_j - bdt2 D_x sigma_1j (8 -> 8) |
//   z: Q_j -= bdt2 D_z sigma_3j (6 -> 3) | y: q_j = Q_j - bdt2 D_y sigma_2j (6 -> 3):
// 47 fields moved.  (Taking D_x on x half-spectra instead, with the y and z derivatives between an
// x-forward and an x-inverse pass, moves 62 in seven passes; at 256^3 that took 0.80 ms in FP32 and
// 1.63 ms in FP64.)
// The x pass also leaves p . A p = sum rho p.p + bdt2 eps : sigma (D is antisymmetric), so the step
// length is known before the last pass, which then updates the residual instead of storing q.
// The residual lives as its y spectrum R: the preconditioner z = M r goes on from there with
//   z-forward | x: x-forward, (beta dt^2 K + rhobar I)^-1, x-inverse | z-inverse,
// and its y-inverse is the next iteration's first pass (YS_PCG).  One iteration: eight passes, 80
// fields (eleven passes and 104 fields before).
// In 2D (n3 == 1) the z passes drop out: D_z = 0.  The reductions that ride on them in 3D are then done
// by the passes that need them, every block for itself (a few hundred partials at most), and that of
// r.r rides on the preconditioner's x pass: four launches an iteration.  (With a launch for each of the
// three sums, as before: FP64, 64^2, 35.3 us an iteration, 29.4 with these.)
#include "nm_common.h"
#include "nm_fft.h"
#include "nm_passes.h"

#include <type_traits>

// Nontemporal (streaming) loads (bit 0) and stores (bit 1), per pass and precision: what a whole solve
// runs fastest with, as a pass's setting also moves the pass that reads its output.  Measured at
// 256^3 (FP32: mixed step; FP64: PCG iteration): all plain 19.2 ms / 2.14 ms, all streaming 19.5 / 2.08,
// stores only 19.2 / 2.14, loads only 18.6 / 2.09, these settings 17.7 / 1.96.
#ifndef NM_NT_YS64
#define NM_NT_YS64 3
#endif
#ifndef NM_NT_YS32
#define NM_NT_YS32 3
#endif
#ifndef NM_NT_ZS64
#define NM_NT_ZS64 1
#endif
#ifndef NM_NT_ZS32
#define NM_NT_ZS32 1
#endif
#ifndef NM_NT_XS64
#define NM_NT_XS64 3
#endif
#ifndef NM_NT_XS32
#define NM_NT_XS32 3
#endif
#ifndef NM_NT_ZD64
#define NM_NT_ZD64 1
#endif
#ifndef NM_NT_ZD32
#define NM_NT_ZD32 1
#endif
#ifndef NM_NT_YE64
#define NM_NT_YE64 3
#endif
#ifndef NM_NT_YE32
#define NM_NT_YE32 3
#endif
#ifndef NM_NT_CF64
#define NM_NT_CF64 1
#endif
#ifndef NM_NT_CF32
#define NM_NT_CF32 1
#endif
#ifndef NM_NT_XP64
#define NM_NT_XP64 2
#endif
#ifndef NM_NT_XP32
#define NM_NT_XP32 0
#endif
// Those are for grids whose fields pass through the last-level cache.  Where a solve's fields about fit it
// (kPlainBytes), nothing streams: FP64 PCG iteration at 128^3 270.9 us with the settings above, 260.7 all
// plain.  Blocks of small grids (see kColSmallBlocks, kXSmallBlocks) stream everything, as stores that
// wait in the L2 are written back at the kernel's end, where nothing covers them: 64^3 66.2 us with the
// settings above, 69.5 all plain, 59.8 all streaming.  The smallest grids would be 5-10% faster plain
// (streaming / plain: 16^3 44.0 / 39.3 us, 32^3 43.4 / 41.1, 512x8x8 51.7 / 49.5); there is one setting
// for all that take those blocks.
enum Mem { MEM_PLAIN = 0, MEM_STREAM = 1 };
#define NM_NT(FAM, T) (SMALL ? 3 : MEM == MEM_PLAIN ? 0 : sizeof(T) == 8 ? NM_NT_##FAM##64 : NM_NT_##FAM##32)

namespace nm {

// Wavefronts per SIMD that the register allocation of a pass aims at.
constexpr int kXStressWaves64 = 2, kXStressWaves32 = 3, kXPrecondWaves64 = 2, kXPrecondWaves32 = 3, kColWaves64 = 2,
              kColWaves32 = 3;

// Early exit of a guarded kernel once the Krylov loop has stopped: a uniform branch, as no launch writes the
// flag that guards it (see ScalarSlot).
__device__ __forceinline__ bool stopped(const double* stop) { return stop && *stop != 0.0; }

// ---------------------------------------------------------------------------
// Deterministic reductions (fixed shuffle tree per wave, fixed order across waves)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Block sum, valid in thread 0 (blocks of BLK threads, whole wavefronts).
template <int BLK> __device__ __forceinline__ double block_sum(double v)
{
    if constexpr (BLK == 64) return wave_sum(v);
    __shared__ double sh[16];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < BLK / 64; i++) s += sh[i];
    return s;
}

// Sum over the block of n partials, to every thread.
template <int BLK> __device__ __forceinline__ double block_total(const double* part, int n)
{
    constexpr int U = 4;
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += U * BLK) {
        double w[U];
#pragma unroll
        for (int k = 0; k < U; k++) w[k] = i + k * BLK < n ? part[i + k * BLK] : 0.0;
#pragma unroll
        for (int k = 0; k < U; k++) v += w[k];
    }
    v = wave_sum(v);
    if constexpr (BLK == 64) return v;
    __shared__ double sh[BLK / 64];
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < BLK / 64; i++) s += sh[i];
    return s;
}

// The reduction a pass carries (see Carry): run by the first block of every field, beside the
// pass's own blocks, so that it costs no launch of its own.
template <int BLK> __device__ __forceinline__ void carry_reduce(const Carry& c, int field)
{
    const double* part = c.part + (long)field * c.n;
    double* scal = c.scal + (long)field * S_COUNT;
    double v = 0.0;
    constexpr int U = 8; // partials in flight per thread
    for (int i = threadIdx.x; i < c.n; i += U * BLK) {
        double w[U];
#pragma unroll
        for (int k = 0; k < U; k++) w[k] = i + k * BLK < c.n ? part[i + k * BLK] : 0.0;
#pragma unroll
        for (int k = 0; k < U; k++) v += w[k];
    }
    const double s = block_sum<BLK>(v);
    if (threadIdx.x != 0) return;
    const bool frozen = c.multi && scal[S_STOP] != 0.0;
    switch (c.action) {
    case RED_RR_CHECK: {
        if (frozen) break;
        scal[S_RR] = s;
        const double it = scal[S_ITER] + 1.0;
        scal[S_ITER] = it;
        const bool done = scal[S_MODE] != 0.0 ? it >= scal[S_LIMIT]
                                              : (s <= scal[S_THR2] || it >= scal[S_LIMIT] || !(s < 1e300));
        if (done) scal[S_STOP] = 1.0;
        break;
    }
    case RED_ALPHA:
        scal[S_PQ] = s;
        scal[S_ALPHA] = frozen ? 0.0 : scal[S_RZ] / s;
        break;
    case RED_RZ_INIT:
        scal[S_RZ] = s;
        scal[S_FIRST] = 1.0;
        break;
    case RED_BETA:
        scal[S_BETA] = frozen ? 0.0 : s / scal[S_RZ];
        scal[S_RZ] = s;
        scal[S_FIRST] = 0.0;
        break;
    default: break;
    }
}

// The twiddle table of length L on its way to LDS: fetched to registers first thing in a kernel, so
// that the fetch overlaps the check of the stop flag and the operands' loads, and stored behind
// them (the caller synchronizes the block before use).
template <int L, int BLK, typename V> struct TwStage {
    static constexpr int N = (L + BLK - 1) / BLK;
    V r[N];
    __device__ __forceinline__ void fetch(const V* __restrict__ tw)
    {
#pragma unroll
        for (int k = 0; k < N; k++) {
            const int i = (int)threadIdx.x + k * BLK;
            r[k] = tw[tw_offset(L) + (i < L ? i : 0)];
        }
    }
    __device__ __forceinline__ void store(V* dst) const
    {
#pragma unroll
        for (int k = 0; k < N; k++) {
            const int i = (int)threadIdx.x + k * BLK;
            if (i < L) dst[i] = r[k];
        }
    }
};

// Frequency (times 1/n, the round trip's normalization) of the bins of one axis.
struct AxisFreq {
    const double* mf; // table of the finite-difference rules, or null
    double k, inv_n;
    int n;
    __device__ __forceinline__ double at(int b) const { return (mf ? mf[b] : k * freq_index(b, n)) * inv_n; }
};

// The axis frequencies in LDS, beside the twiddles: computed per point in registers they would put a
// branch (table or formula) and a conversion in front of every multiplication.
template <int L, int BLK, typename T> __device__ __forceinline__ void stage_freq(T* dst, const AxisFreq& f)
{
    for (int i = threadIdx.x; i < L; i += BLK) dst[i] = (T)f.at(i);
}

// multiply by i s
template <typename V, typename S> __device__ __forceinline__ V iscale(V a, S s) { return V{-a.y * s, a.x * s}; }

// ---------------------------------------------------------------------------
// y and z directions: tiles of TX consecutive columns of L points, one component per block.
// A thread holds R points of one column and the block L / R threads per column, so that every row
// of a tile is TX elements (128 bytes in FP32, 256 in FP64) wide.  Bound by HBM: 256^3 FP32 / FP64, us
// and TB/s: y start (6 fields) 78 / 149, 5.2 / 5.4; z strain (7) 96 / 157, 4.9 / 6.0; z divergence (9)
// 109 / 202, 5.5 / 6.0; y end (9) 98 / 204, 6.2 / 5.9; transforms alone (6) 66 / 150, 6.1 / 5.4.
// One component per block keeps two operands in registers at most, so that the loads of other
// blocks cover a block's transforms.  Rows half as wide (radix 8 or 128 threads): FP32 y start 106-113,
// z divergence 157-162 us, FP64 1.30 against 1.24 ms for the operator.  Radix 8 with 512 threads is no
// different from radix 16 with 256.
// ---------------------------------------------------------------------------
// Columns of an axis: column c starts at (c >> sh) * hi + (c & mask), its points lie step apart.
struct Cols {
    int ncols, sh, mask;
    long hi, step;
};

// Points per thread.
template <typename T, int L> constexpr int col_radix()
{
    // (128-long columns in FP64: radix 16 takes 67 KB of LDS, two blocks per compute unit and 1.5 rounds of
    // blocks at 128^3; radix 8 half of that: PCG iteration 279 -> 273 us)
    return L <= 16 ? L : (L <= (sizeof(T) == 8 ? 128 : 64) ? 8 : 16);
}
// Threads per block, and on grids too small to give every compute unit a block of those: a wavefront, or
// what keeps the rows of a tile eight elements wide, with every operand fetched ahead of the first
// transform.  FP64, 32^3: operator 49.5 -> 39.5 us, PCG iteration 47.8 -> 43.1; 512x8x8 54.4 -> 51.3.
constexpr int kColSmallBlocks = 512;
template <typename T, int L> constexpr int col_block() { return L == 512 && sizeof(T) == 4 ? 512 : 256; }
template <typename T, int L> constexpr int col_small_block()
{
    const int b = 8 * (L / col_radix<T, L>());
    return b > 64 ? b : 64;
}

template <typename T, int L, int BLK> struct ColShape {
    static constexpr int R = col_radix<T, L>(), G = L / R;
    static constexpr int W = sizeof(T) == 8 ? kColWaves64 : kColWaves32; // wavefronts per SIMD
    static constexpr int TX = BLK / G;
};

template <typename T, int L, int BLK> struct ColTile {
    using V = cx_t<T>;
    using Sh = ColShape<T, L, BLK>;
    static constexpr int R = Sh::R, G = Sh::G, TX = Sh::TX;
    int t;
    bool valid;
    uint32_t lane, mstep; // byte offsets: of the thread's first point; between its points (uniform)
    ColAddr<TX> addr;
    __device__ __forceinline__ ColTile(const Cols& g, int tile)
    {
        const int c = threadIdx.x % TX;
        t = threadIdx.x / TX;
        addr.c = c;
        const int col = tile * TX + c;
        valid = col < g.ncols;
        const int cc = valid ? col : 0; // surplus lanes read column 0 and store nothing
        const long off = (long)(cc >> g.sh) * g.hi + (cc & g.mask) + (long)t * g.step;
        lane = (uint32_t)(off * sizeof(V));
        mstep = (uint32_t)(G * g.step * sizeof(V));
    }
    // element index of point m within the component
    __device__ __forceinline__ uint32_t elem(int m) const { return (lane + (uint32_t)m * mstep) / (uint32_t)sizeof(V); }
    // point m of the column (a scalar base, the thread's offset and nothing else per lane)
    template <typename P> __device__ __forceinline__ P* at(P* base, int m) const
    {
        using C = std::conditional_t<std::is_const_v<P>, const char, char>;
        return (P*)((C*)base + (uint64_t)m * mstep + lane);
    }
    template <int NT> __device__ __forceinline__ void ld(const V* base, V (&v)[R]) const
    {
#pragma unroll
        for (int m = 0; m < R; m++) v[m] = ld_nt<NT>(at(base, m));
    }
    template <int NT> __device__ __forceinline__ void st(V* base, const V (&v)[R]) const
    {
        if (!valid) return;
#pragma unroll
        for (int m = 0; m < R; m++) st_nt<NT>(at(base, m), v[m]);
    }
    template <int DIR> __device__ __forceinline__ void fft(V (&v)[R], V* lds, const V* tw) const
    {
        group_fft<L, R, DIR, false, FFT_PLAIN, 1>((V(&)[1][R])v, t, lds, addr, tw);
    }
    // v <- D v
    __device__ __forceinline__ void deriv(V (&v)[R], V* lds, const V* tw, const T* fr) const
    {
        fft<-1>(v, lds, tw);
#pragma unroll
        for (int m = 0; m < R; m++) v[m] = iscale(v[m], fr[t + m * G]);
        fft<+1>(v, lds, tw);
    }
    // the Gamma mask (null: none) of the thread's points
    __device__ __forceinline__ void ld_mask(const uint8_t* mask, uint16_t (&k)[R]) const
    {
#pragma unroll
        for (int m = 0; m < R; m++) k[m] = mask ? ((const uint16_t*)mask)[elem(m)] : (uint16_t)0;
    }
    __device__ __forceinline__ void masked(const uint16_t (&k)[R], V (&v)[R]) const
    {
#pragma unroll
        for (int m = 0; m < R; m++) {
            if (k[m] & 0x00ffu) v[m].x = 0;
            if (k[m] & 0xff00u) v[m].y = 0;
        }
    }
    __device__ __forceinline__ void masked(const uint8_t* mask, V (&v)[R]) const
    {
        if (!mask) return;
        uint16_t k[R];
        ld_mask(mask, k);
        masked(k, v);
    }
};
// Component and tile of a block: in FP32 the three components of a tile are neighbours, in FP64 one
// component follows the other (256^3: FP32 mixed step 18.2 -> 17.9 ms, FP64 iteration 1.96 against
// 1.99 ms with the FP32 order).
template <typename T> __device__ __forceinline__ int col_comp(int blk, int ntiles)
{
    return sizeof(T) == 4 ? blk % 3 : blk / ntiles;
}
template <typename T> __device__ __forceinline__ int col_tile(int blk, int ntiles)
{
    return sizeof(T) == 4 ? blk / 3 : blk % ntiles;
}
// Prologue of a column kernel: the twiddles' fetch, the stop flag (and what is done where it is set) ...
#define NM_COL_BEGIN(L, ...)                                                                                           \
    [[maybe_unused]] constexpr bool SMALL = BLK < col_block<T, L>();                                                   \
    __shared__ V lds[ColShape<T, L, BLK>::G > 1 ? BLK * ColShape<T, L, BLK>::R : 1];                             \
    __shared__ V tws[L];                                                                                               \
    TwStage<L, BLK, V> tst;                                                                            \
    if constexpr (ColShape<T, L, BLK>::G > 1) tst.fetch(tw);                                                                \
    if (stopped(a.lay.stop)) {                                                                                         \
        __VA_ARGS__;                                                                                                   \
        return;                                                                                                        \
    }
// ... and, behind the operands' loads, the tables published to the block.
#define NM_COL_TABLES(L)                                                                                               \
    if constexpr (ColShape<T, L, BLK>::G > 1) tst.store(tws);
#define NM_COL_READY(L)                                                                                                \
    NM_COL_TABLES(L)                                                                                                   \
    __syncthreads();
#define NM_COL_READY_FREQ(L)                                                                                           \
    __shared__ T frs[L];                                                                                               \
    NM_COL_TABLES(L)                                                                                                   \
    stage_freq<L, BLK>(frs, f);                                                                                             \
    __syncthreads();

template <typename T, int L, int BLK, int MEM, int MODE>
__global__ __launch_bounds__(BLK, (ColShape<T, L, BLK>::W)) void k_ystart(PassArgs a, Cols g, AxisFreq f, int ntiles,
                                                                  const cx_t<T>* __restrict__ tw)
{
    using V = cx_t<T>;
    NM_COL_BEGIN(L, if (MODE == YS_PCG && blockIdx.x == 0 && threadIdx.x == 0) a.scal[S_HALT] = 1.0)
    constexpr int R = ColShape<T, L, BLK>::R, NT = NM_NT(YS, T);
    const int fld = blockIdx.z, j = col_comp<T>(blockIdx.x, ntiles);
    const ColTile<T, L, BLK> c(g, col_tile<T>(blockIdx.x, ntiles));
    const long fo = (long)fld * a.lay.bf + j * a.lay.ns;
    V* const dst = (V*)a.S + (long)fld * a.lay.bs + j * a.lay.cs;
    const bool zero_comp = a.lay.dim == 2 && j == 2;
    V v[R];
    if constexpr (MODE == YS_APPLY) {
        c.template ld<NT>((const V*)a.u + fo, v);
        NM_COL_READY_FREQ(L)
        c.deriv(v, lds, tws, frs);
    } else if constexpr (MODE == YS_EXPLICIT) {
        const T dt = (T)a.dt, hdt = (T)(0.5 * a.dt);
        V vo[R], ao[R];
        c.template ld<NT>((const V*)a.u + fo, v);
        c.template ld<NT>((const V*)a.v + fo, vo);
        c.template ld<NT>((const V*)a.a + fo, ao);
#pragma unroll
        for (int m = 0; m < R; m++) {
            vo[m] = V{vo[m].x + hdt * ao[m].x, vo[m].y + hdt * ao[m].y};
            v[m] = V{v[m].x + dt * vo[m].x, v[m].y + dt * vo[m].y};
        }
        c.template st<NT>((V*)a.v + fo, vo);
        c.template st<NT>((V*)a.u + fo, v);
        NM_COL_READY_FREQ(L)
        c.deriv(v, lds, tws, frs);
    } else {
        const double* sc = a.scal + (long)fld * S_COUNT;
        const bool first = sc[S_FIRST] != 0.0;
        T beta = (T)sc[S_BETA];
        const T alpha = (T)sc[S_ALPHA];
        c.template ld<NT>((const V*)a.S2 + (long)fld * a.lay.bs + j * a.lay.cs, v);
        V po[R];
        if (!first) {
            // the deferred x += alpha p_old goes first, so that its operand is not held over the transform
            V xo[R];
            c.template ld<NT>((const V*)a.p + fo, po);
            c.template ld<NT>((const V*)a.x + fo, xo);
#pragma unroll
            for (int m = 0; m < R; m++) xo[m] = V{xo[m].x + alpha * po[m].x, xo[m].y + alpha * po[m].y};
            c.template st<NT>((V*)a.x + fo, xo);
        } else {
#pragma unroll
            for (int m = 0; m < R; m++) po[m] = V{0, 0};
        }
        uint16_t mk[R];
        if constexpr (SMALL) c.ld_mask(a.mask, mk);
        if (a.carry.action == RED_BETA) {
            // S_RZ still holds the last iteration's r.z; YE_UPDATE moves the new one there
            const double rz = block_total<BLK>(a.carry.part + (long)fld * a.carry.n, a.carry.n);
            beta = (T)(a.carry.multi && sc[S_STOP] != 0.0 ? 0.0 : rz / sc[S_RZ]);
            if (blockIdx.x == 0 && threadIdx.x == 0) a.scal[(long)fld * S_COUNT + S_RZ2] = rz;
        }
        NM_COL_READY_FREQ(L)
        c.template fft<+1>(v, lds, tws);
        if constexpr (!SMALL) c.masked(a.mask, v);
        else c.masked(mk, v);
        if (!first) {
#pragma unroll
            for (int m = 0; m < R; m++) v[m] = V{v[m].x + beta * po[m].x, v[m].y + beta * po[m].y};
        }
        if (zero_comp) {
#pragma unroll
            for (int m = 0; m < R; m++) v[m] = V{0, 0};
        }
        c.template st<NT>((V*)a.p + fo, v);
        c.deriv(v, lds, tws, frs);
    }
    c.template st<NT>(dst, v);
}

template <typename T, int L, int BLK, int MEM>
__global__ __launch_bounds__(BLK, (ColShape<T, L, BLK>::W)) void k_zstrain(PassArgs a, Cols g, AxisFreq f, int ntiles,
                                                                   const cx_t<T>* __restrict__ tw)
{
    using V = cx_t<T>;
    NM_COL_BEGIN(L)
    constexpr int R = ColShape<T, L, BLK>::R, NT = NM_NT(ZS, T);
    const int fld = blockIdx.z, j = col_comp<T>(blockIdx.x, ntiles);
    const ColTile<T, L, BLK> c(g, col_tile<T>(blockIdx.x, ntiles));
    V* const S = (V*)a.S + (long)fld * a.lay.bs;
    V* const dst = S + (j == 0 ? 3 : j == 1 ? 2 : 4) * a.lay.cs;
    V v[R], w[R];
    c.template ld<NT>((const V*)a.p + (long)fld * a.lay.bf + j * a.lay.ns, v);
    if (j == 1) c.template ld<NT>(dst, w); // D_y p_3
    NM_COL_READY_FREQ(L)
    c.deriv(v, lds, tws, frs);
    if (j == 1) {
        // g23 = D_z p_2 + D_y p_3
#pragma unroll
        for (int m = 0; m < R; m++) v[m] = cadd(v[m], w[m]);
    }
    c.template st<NT>(dst, v);
}

template <typename T, int L, int BLK, int MEM>
__global__ __launch_bounds__(BLK, (ColShape<T, L, BLK>::W)) void k_zdiv(PassArgs a, Cols g, AxisFreq f, int ntiles,
                                                                const cx_t<T>* __restrict__ tw)
{
    using V = cx_t<T>;
    NM_COL_BEGIN(L)
    constexpr int R = ColShape<T, L, BLK>::R, NT = NM_NT(ZD, T);
    const int fld = blockIdx.z;
    int blk = blockIdx.x;
    if (a.carry.action != RED_NONE) {
        if (blk == 0) {
            carry_reduce<BLK>(a.carry, fld);
            return;
        }
        blk--;
    }
    const int j = col_comp<T>(blk, ntiles);
    const ColTile<T, L, BLK> c(g, col_tile<T>(blk, ntiles));
    // sigma_31, sigma_32, sigma_33
    const V* src = (const V*)a.S + (long)fld * a.lay.bs + (j == 0 ? 3 : j == 1 ? 2 : 4) * a.lay.cs;
    V* const Q = (V*)a.S2 + (long)fld * a.lay.bs + j * a.lay.cs;
    V v[R], w[R];
    c.template ld<NT>(src, v);
    c.template ld<NT>(Q, w);
    NM_COL_READY_FREQ(L)
    c.deriv(v, lds, tws, frs);
    const T cd = (T)-a.bdt2;
#pragma unroll
    for (int m = 0; m < R; m++) v[m] = V{w[m].x + cd * v[m].x, w[m].y + cd * v[m].y};
    c.template st<NT>(Q, v);
}

template <typename T, int L, int BLK, int MEM, int MODE>
__global__ __launch_bounds__(BLK, (ColShape<T, L, BLK>::W)) void k_yend(PassArgs a, Cols g, AxisFreq f, int ntiles,
                                                                const cx_t<T>* __restrict__ tw)
{
    using V = cx_t<T>;
    NM_COL_BEGIN(L)
    constexpr int R = ColShape<T, L, BLK>::R, NT = NM_NT(YE, T);
    const int fld = blockIdx.z, j = col_comp<T>(blockIdx.x, ntiles);
    const ColTile<T, L, BLK> c(g, col_tile<T>(blockIdx.x, ntiles));
    const long fo = (long)fld * a.lay.bf + j * a.lay.ns;
    // sigma_21, sigma_22, sigma_23
    V* const src = (V*)a.S + (long)fld * a.lay.bs + j * a.lay.cs;
    const V* Q = (const V*)a.S2 + (long)fld * a.lay.bs + j * a.lay.cs;
    const bool zero_comp = a.lay.dim == 2 && j == 2;
    V v[R], w[R];
    c.template ld<NT>(src, v);
    V ro[R];
    uint16_t mk[R];
    if constexpr (SMALL || MODE != YE_UPDATE) c.template ld<NT>(Q, w);
    if constexpr (MODE == YE_UPDATE) c.template ld<NT>((const V*)a.r + fo, ro);
    if constexpr (SMALL && MODE == YE_RESIDUAL) c.template ld<NT>((const V*)a.b + fo, ro);
    if constexpr (SMALL && (MODE == YE_UPDATE || MODE == YE_OUT || MODE == YE_RESIDUAL)) c.ld_mask(a.mask, mk);
    double pq = 0.0;
    if constexpr (MODE == YE_UPDATE) {
        if (a.carry.action == RED_ALPHA) pq = block_total<BLK>(a.carry.part + (long)fld * a.carry.n, a.carry.n);
    }
    NM_COL_READY_FREQ(L)
    const T cd = (T)-a.bdt2;
    if constexpr (MODE == YE_UPDATE) {
        // r = mask(y-inverse(R / n - alpha cd i xi / n y-forward(sigma)) - alpha Q): three transforms, like the
        // update R -= alpha y-forward(mask q) of the spectrum alone.  That one leaves R's rounding on the Gamma
        // voxels, where the masked q is zero, and there it stays, until the free residual is the smaller one
        // (FP64: from some eps |r_0| on) and the iteration grows without bound.  A y line all Gamma shares its
        // transform with the next one, so whole planes are no exception.  FP64 iteration with a Gamma plane, that
        // update / this one: 64^3 61.7 / 61.6 us, 128^3 260.5 / 265.2, 256^3 1924 / 1933 (Q is read late instead
        // of R); R transformed back on its own, in the tiles that have Gamma: 128^3 266.7, 256^3 1943.
        double* const sc = a.scal + (long)fld * S_COUNT;
        T alpha;
        if (a.carry.action == RED_ALPHA) {
            const double rz = sc[S_RZ2], al = a.carry.multi && sc[S_STOP] != 0.0 ? 0.0 : rz / pq;
            alpha = (T)al;
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                sc[S_PQ] = pq;
                sc[S_ALPHA] = al;
                sc[S_RZ] = rz;
                sc[S_FIRST] = 0.0;
            }
        } else {
            alpha = (T)sc[S_ALPHA];
        }
        if (zero_comp) alpha = 0; // q is zero
        const T inv_n = (T)f.inv_n, ac = alpha * cd;
        c.template fft<-1>(v, lds, tws);
#pragma unroll
        for (int m = 0; m < R; m++) {
            const T s = ac * frs[c.t + m * ColTile<T, L, BLK>::G];
            v[m] = V{inv_n * ro[m].x + s * v[m].y, inv_n * ro[m].y - s * v[m].x};
        }
        if constexpr (!SMALL) c.template ld<NT>(Q, w);
        c.template fft<+1>(v, lds, tws);
#pragma unroll
        for (int m = 0; m < R; m++) v[m] = V{v[m].x - alpha * w[m].x, v[m].y - alpha * w[m].y};
        if constexpr (!SMALL) c.masked(a.mask, v);
        else c.masked(mk, v);
        double part = 0.0;
#pragma unroll
        for (int m = 0; m < R; m++) part += (double)v[m].x * (double)v[m].x + (double)v[m].y * (double)v[m].y;
        c.template fft<-1>(v, lds, tws);
        c.template st<NT>((V*)a.r + fo, v);
        const double s = block_sum<BLK>(c.valid ? part : 0.0);
        if (threadIdx.x == 0) a.partials[(long)fld * (3 * ntiles) + blockIdx.x] = s;
        return;
    }
    c.deriv(v, lds, tws, frs);
#pragma unroll
    for (int m = 0; m < R; m++) {
        v[m] = V{w[m].x + cd * v[m].x, w[m].y + cd * v[m].y};
        if (zero_comp) v[m] = V{0, 0};
    }
    if constexpr (MODE == YE_EXPLICIT || MODE == YE_EXPLICIT_NEXT) {
        // o = dt/2 div sigma.  The last step of a batch: v <- v + o / rho, a <- (2/dt) o / rho.  Between two
        // steps: v <- v + 2 o / rho, u <- u + dt v and its D_y, 21 fields where an end that leaves v and a and a
        // start that reads them back move 33 (FP64, 256^3, 3 steps: 4.92 ms, 4.45 with this).
        constexpr bool NEXT = MODE == YE_EXPLICIT_NEXT;
        const T* rho = (const T*)a.rho;
        const T dt = (T)a.dt, idt2 = (T)(2.0 / a.dt);
        // (fetched here and a few points at a time: held over the transforms they would spill)
        constexpr int H = NEXT ? 2 : R < 4 ? R : 4;
#pragma unroll
        for (int q = 0; q < R; q += H) {
            ColTile<T, L, BLK> e = c; // the offset hidden: kept per array and chunk, the addresses would spill
            asm("" : "+v"(e.lane));
            V vo[H], ao[H]; // ao: acceleration, or the next displacement
            uint32_t ph[H];
            uint16_t mk[H];
#pragma unroll
            for (int m = 0; m < H; m++) {
                vo[m] = ld_nt<NT>(e.at((const V*)a.v + fo, q + m));
                if constexpr (NEXT) {
                    ao[m] = ld_nt<NT>(e.at((const V*)a.u + fo, q + m));
                    mk[m] = a.mask ? ((const uint16_t*)a.mask)[e.elem(q + m)] : (uint16_t)0;
                }
                ph[m] = ((const uint32_t*)a.phase)[e.elem(q + m)];
            }
#pragma unroll
            for (int m = 0; m < H; m++) {
                V o = V{v[q + m].x / rho[ph[m] & 0xffffu], v[q + m].y / rho[ph[m] >> 16]};
                if constexpr (NEXT) {
                    o = V{mk[m] & 0x00ffu ? (T)0 : 2 * o.x, mk[m] & 0xff00u ? (T)0 : 2 * o.y};
                } else {
                    ao[m] = V{idt2 * o.x, idt2 * o.y};
                }
                vo[m] = V{vo[m].x + o.x, vo[m].y + o.y};
                if (zero_comp) vo[m] = V{0, 0};
                if constexpr (NEXT) {
                    ao[m] = V{ao[m].x + dt * vo[m].x, ao[m].y + dt * vo[m].y};
                    v[q + m] = ao[m];
                } else if (zero_comp) {
                    ao[m] = V{0, 0};
                }
            }
            if (c.valid) {
                V* const second = NEXT ? (V*)a.u : (V*)a.a;
#pragma unroll
                for (int m = 0; m < H; m++) {
                    st_nt<NT>(e.at((V*)a.v + fo, q + m), vo[m]);
                    st_nt<NT>(e.at(second + fo, q + m), ao[m]);
                }
            }
            if constexpr (NEXT) {
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (NEXT) {
            c.deriv(v, lds, tws, frs);
            c.template st<NT>(src, v);
        }
    } else if constexpr (MODE == YE_RESIDUAL) {
        // b - q here rather than q to memory and a kernel that reads it back (6 fields: FP64, 256^3, this
        // pass and that kernel 191 + 253 us, 295 in one)
        if constexpr (!SMALL) c.template ld<NT>((const V*)a.b + fo, ro);
#pragma unroll
        for (int m = 0; m < R; m++) v[m] = V{ro[m].x - v[m].x, ro[m].y - v[m].y};
        if constexpr (!SMALL) c.masked(a.mask, v);
        else c.masked(mk, v);
        c.template st<NT>((V*)a.out + fo, v);
        double part = 0.0;
#pragma unroll
        for (int m = 0; m < R; m++) part += (double)v[m].x * (double)v[m].x + (double)v[m].y * (double)v[m].y;
        if (a.r32 && c.valid) {
            float2* const r32 = (float2*)a.r32 + fo;
#pragma unroll
            for (int m = 0; m < R; m++) r32[c.elem(m)] = float2{(float)v[m].x, (float)v[m].y};
        }
        const double s = block_sum<BLK>(c.valid ? part : 0.0);
        if (threadIdx.x == 0) a.partials[(long)fld * (3 * ntiles) + blockIdx.x] = s;
    } else {
        if constexpr (!SMALL) c.masked(a.mask, v);
        else c.masked(mk, v);
        c.template st<NT>((V*)a.out + fo, v);
    }
}

template <typename T, int L, int BLK, int MEM, int DIR>
__global__ __launch_bounds__(BLK, (ColShape<T, L, BLK>::W)) void k_colfft(ColFft a, Cols g, int ntiles,
                                                                  const cx_t<T>* __restrict__ tw)
{
    using V = cx_t<T>;
    NM_COL_BEGIN(L)
    constexpr int R = ColShape<T, L, BLK>::R, NT = NM_NT(CF, T);
    const int fld = blockIdx.z;
    int blk = blockIdx.x;
    if (a.carry.action != RED_NONE) {
        if (blk == 0) {
            carry_reduce<BLK>(a.carry, fld);
            return;
        }
        blk--;
    }
    const int j = col_comp<T>(blk, ntiles);
    const ColTile<T, L, BLK> c(g, col_tile<T>(blk, ntiles));
    V v[R];
    uint16_t mk[R];
    c.template ld<NT>((const V*)a.src + (long)fld * a.sb + j * a.sc, v);
    if constexpr (SMALL && DIR > 0) c.ld_mask(a.mask, mk);
    NM_COL_READY(L)
    c.template fft<DIR>(v, lds, tws);
    if constexpr (DIR > 0) {
        if constexpr (!SMALL) c.masked(a.mask, v);
        else c.masked(mk, v);
        if (a.zero3 && j == 2) {
#pragma unroll
            for (int m = 0; m < R; m++) v[m] = V{0, 0};
        }
    }
    c.template st<NT>((V*)a.dst + (long)fld * a.db + j * a.dc, v);
}

// ---------------------------------------------------------------------------
// x direction
// ---------------------------------------------------------------------------
// sigma_v = C_v eps_v for one voxel (Voigt, engineering shear; 21 = upper triangle).
template <typename T> __device__ __forceinline__ void voigt_stress(const T* __restrict__ c, const T e[6], T s[6])
{
    // row-major upper triangle offsets: row a starts at a*6 - a*(a-1)/2
    s[0] = c[0] * e[0] + c[1] * e[1] + c[2] * e[2] + c[3] * e[3] + c[4] * e[4] + c[5] * e[5];
    s[1] = c[1] * e[0] + c[6] * e[1] + c[7] * e[2] + c[8] * e[3] + c[9] * e[4] + c[10] * e[5];
    s[2] = c[2] * e[0] + c[7] * e[1] + c[11] * e[2] + c[12] * e[3] + c[13] * e[4] + c[14] * e[5];
    s[3] = c[3] * e[0] + c[8] * e[1] + c[12] * e[2] + c[15] * e[3] + c[16] * e[4] + c[17] * e[5];
    s[4] = c[4] * e[0] + c[9] * e[1] + c[13] * e[2] + c[16] * e[3] + c[18] * e[4] + c[19] * e[5];
    s[5] = c[5] * e[0] + c[10] * e[1] + c[14] * e[2] + c[17] * e[3] + c[19] * e[4] + c[20] * e[5];
}

// Streaming access of one real.
template <int NT, typename T> __device__ __forceinline__ T ld_s(const T* p)
{
    if constexpr ((NT & 1) != 0) return __builtin_nontemporal_load(p);
    else return *p;
}
template <int NT, typename T> __device__ __forceinline__ void st_s(T* p, T v)
{
    if constexpr ((NT & 2) != 0) __builtin_nontemporal_store(v, p);
    else *p = v;
}

constexpr int kXR = 4; // elements per thread of a pair of x lines in the stress pass

// Threads per block of the x passes.  On small grids a wavefront (two where a line spans two) per
// block: the passes are then one chain of instructions per wavefront, in which four wavefronts on one
// compute unit wait for each other's memory and LDS instructions while other units stand idle.  From
// two blocks of 256 per compute unit on, 256 threads share the staging of the tables.  FP64 PCG
// iteration with 256 threads and with these: 64^3 73.9 / 67.4 us, 32^3 56.5 / 48.1, 512x8x8 64.8 / 54.6,
// 64^2 42.3 / 36.5.
constexpr int kXSmallBlocks = 512;
template <int N1, int R> constexpr int x_small_block() { return N1 / R > 64 ? N1 / R : 64; }
// (small blocks are alone on their SIMD: all its registers, and every operand fetched at once)
template <typename T, int BLK> constexpr int x_waves(int w64, int w32)
{
    return BLK != kBlock ? 1 : sizeof(T) == 8 ? w64 : w32;
}

// The stress pass: 16 fields and the grain ids, 256^3: 0.204 ms in FP32 (5.4 TB/s), 0.442 in FP64
// (4.9); the x pass it replaces moved 12 fields in 0.20 and 0.36 ms.  HBM bounds it in FP32, and in FP64
// the registers too (two wavefronts per SIMD).  A group of N1 / 4 lanes holds the rows (y, y + 1) of one z plane as a complex
// line of N1 points, in all three components at once (one synchronisation per stage for the three).
template <typename T, int N1, int BLK, int MEM>
__global__ __launch_bounds__(BLK, (x_waves<T, BLK>(kXStressWaves64, kXStressWaves32)))
    void k_xstress(PassArgs a, AxisFreq f, int npairs, const cx_t<T>* __restrict__ tw)
{
    using V = cx_t<T>;
    constexpr bool SMALL = BLK != kBlock;
    constexpr int R = kXR, G = N1 / R, LPB = BLK / G, NT = NM_NT(XS, T);
    // p is needed again for the inertia term.  FP32 holds it over the transforms (three wavefronts per SIMD
    // instead of four, 256^3: 221 -> 204 us; the counters showed every second read to leave the compute die).
    // FP64 has no registers for that and reads it again, the first time without the streaming hint (459 -> 442).
    constexpr bool HOLD_P = SMALL || sizeof(T) == 4;
    // strains fetched ahead of the first transform
    constexpr int EARLY = SMALL ? 5 : sizeof(T) == 8 ? 0 : 3;
    constexpr bool WAVE = G <= 64;
    constexpr int LP = line_elems(N1), AREA = LPB * LP;
    __shared__ V lds[3 * AREA];
    __shared__ V tws[N1];
    __shared__ T frs[N1];
    TwStage<N1, BLK, V> tst;
    tst.fetch(tw);
    if (stopped(a.lay.stop)) return;
    const int ll = threadIdx.x / G, t = threadIdx.x % G, fld = blockIdx.z;
    const int pr = blockIdx.x * LPB + ll;
    const bool valid = pr < npairs;
    // the two rows are neighbours in memory: reals [2 N1 pr, 2 N1 (pr + 1))
    const uint32_t base = (uint32_t)(valid ? pr : 0) * (2u * N1) + t, bb = base * (uint32_t)sizeof(T);
    const LineAddr<AREA> addr{ll * LP};
    const T* const p = (const T*)((const V*)a.p + (long)fld * a.lay.bf);
    T* const S = (T*)((V*)a.S + (long)fld * a.lay.bs);
    T* const Q = (T*)((V*)a.S2 + (long)fld * a.lay.bs);
    const long ps = 2 * a.lay.ns, cs = 2 * a.lay.cs;
    const bool has_z = a.lay.n3 > 1;
    // the lane's byte offset, hidden from the optimizer at each use: otherwise it keeps one 64-bit
    // address per buffer in registers instead of scalar bases
    auto lane_off = [&]() {
        uint32_t o = bb;
        asm("" : "+v"(o));
        return o;
    };
    auto ld = [&](const T* q, V (&v)[R]) {
        const uint32_t o = lane_off();
#pragma unroll
        for (int m = 0; m < R; m++) {
            v[m].x = ld_s<NT>((const T*)((const char*)q + o) + m * G);
            v[m].y = ld_s<NT>((const T*)((const char*)q + o) + (m * G + N1));
        }
    };
    // p: where it is read twice, the first read stays in the caches for the second
    auto ld_p = [&](const T* q, V (&v)[R]) {
        constexpr int NP = HOLD_P ? NT : NT & ~1;
        const uint32_t o = lane_off();
#pragma unroll
        for (int m = 0; m < R; m++) {
            v[m].x = ld_s<NP>((const T*)((const char*)q + o) + m * G);
            v[m].y = ld_s<NP>((const T*)((const char*)q + o) + (m * G + N1));
        }
    };
    auto st = [&](T* q, const V (&v)[R]) {
        const uint32_t o = lane_off();
#pragma unroll
        for (int m = 0; m < R; m++) {
            st_s<NT>((T*)((char*)q + o) + m * G, v[m].x);
            st_s<NT>((T*)((char*)q + o) + (m * G + N1), v[m].y);
        }
    };
    V d[3][R], w[5][R]; // displacement and its x derivative; D_y p1, D_y p2, g23, D_z p1, D_z p3
#pragma unroll
    for (int j = 0; j < 3; j++) ld_p(p + j * ps, d[j]);
#pragma unroll
    for (int c = 0; c < EARLY; c++) {
        if (c < 3 || has_z) {
            ld(S + c * cs, w[c]);
        } else {
#pragma unroll
            for (int m = 0; m < R; m++) w[c][m] = V{0, 0};
        }
    }
    V po[3][R];
    if constexpr (HOLD_P) {
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int m = 0; m < R; m++) po[j][m] = d[j][m];
    }
    uint32_t ph[R];
#pragma unroll
    for (int m = 0; m < R; m++)
        ph[m] = (uint32_t)a.phase[base + m * G] | ((uint32_t)a.phase[base + m * G + N1] << 16);
    tst.store(tws);
    stage_freq<N1, BLK>(frs, f);
    __syncthreads();
    auto deriv3 = [&](V (&v)[3][R], auto between) {
        group_fft<N1, R, -1, WAVE, FFT_PLAIN, 3>(v, t, lds, addr, tws);
        between();
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int m = 0; m < R; m++) v[j][m] = iscale(v[j][m], frs[t + m * G]);
        group_fft<N1, R, +1, WAVE, FFT_PLAIN, 3>(v, t, lds, addr, tws);
    };
    // the remaining strains are fetched between the two transforms: all of them ahead of the first
    // would take more registers than the occupancy leaves
    deriv3(d, [&]() {
#pragma unroll
        for (int c = EARLY; c < 5; c++) {
            if (c < 3 || has_z) {
                ld(S + c * cs, w[c]);
            } else {
#pragma unroll
                for (int m = 0; m < R; m++) w[c][m] = V{0, 0};
            }
        }
    });
    double part = 0.0;
    const T b2 = (T)a.bdt2;
#pragma unroll
    for (int m = 0; m < R; m++) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            auto at = [h](const V& q) { return h ? q.y : q.x; };
            auto put = [h](V& q, T x) { (h ? q.y : q.x) = x; };
            const T* cg = (const T*)a.C21 + 21 * (h ? (ph[m] >> 16) : (ph[m] & 0xffffu));
            // Voigt order 11 22 33 23 13 12
            T e[6] = {at(d[0][m]), at(w[1][m]), at(w[4][m]), at(w[2][m]), at(w[3][m]) + at(d[2][m]),
                      at(w[0][m]) + at(d[1][m])};
            T s[6];
            voigt_stress(cg, e, s);
            // (widened before the products: strain times stress can leave FP32's range where neither does)
            double es = 0.0;
#pragma unroll
            for (int q = 0; q < 6; q++) es += (double)e[q] * (double)s[q];
            part += a.bdt2 * es;
            put(d[0][m], s[0]);
            put(d[1][m], s[5]);
            put(d[2][m], s[4]);
            put(w[0][m], s[5]);
            put(w[1][m], s[1]);
            put(w[2][m], s[3]);
            put(w[3][m], s[4]);
            put(w[4][m], s[2]);
        }
        // the sum is due here: sunk to its only use, it would keep every strain and stress in registers
        asm volatile("" : "+v"(part));
        __builtin_amdgcn_sched_barrier(0); // one element's stiffness at a time in registers
    }
    if (valid) { // (surplus pairs read row 0)
#pragma unroll
        for (int c = 0; c < 3; c++) st(S + c * cs, w[c]); // s12 s22 s23
        if (has_z) {
            st(S + 3 * cs, w[3]); // s13
            st(S + 4 * cs, w[4]); // s33
        }
    }
    deriv3(d, [&]() {
        if constexpr (!HOLD_P) {
#pragma unroll
            for (int j = 0; j < 3; j++) ld(p + j * ps, po[j]);
        }
    });
    T rh[R][2];
#pragma unroll
    for (int m = 0; m < R; m++) rh[m][0] = rh[m][1] = (T)0;
    if (a.rho) {
#pragma unroll
        for (int m = 0; m < R; m++) {
            rh[m][0] = ((const T*)a.rho)[ph[m] & 0xffffu];
            rh[m][1] = ((const T*)a.rho)[ph[m] >> 16];
        }
    }
#pragma unroll
    for (int j = 0; j < 3; j++) {
#pragma unroll
        for (int m = 0; m < R; m++) {
            const V q = V{rh[m][0] * po[j][m].x, rh[m][1] * po[j][m].y};
            part += (double)q.x * (double)po[j][m].x + (double)q.y * (double)po[j][m].y;
            d[j][m] = V{q.x - b2 * d[j][m].x, q.y - b2 * d[j][m].y};
        }
        asm volatile("" : "+v"(part));
        if (valid) st(Q + j * cs, d[j]);
    }
    if (a.partials) {
        const double s = block_sum<BLK>(valid ? part : 0.0);
        if (threadIdx.x == 0) a.partials[(long)fld * ((npairs + LPB - 1) / LPB) + blockIdx.x] = s;
    }
}

// The preconditioner's middle pass on the (y, z) spectrum C of the packed pairs.  The spectra of
// the even and odd voxels of a row come apart with the mirrored row,
//   r^(2x', k) = (C(x', k) + conj C(x', -k)) / 2,  r^(2x'+1, k) = (C(x', k) - conj C(x', -k)) / (2 i),
// so a group takes the rows k = (ky, kz) and -k together: one complex line of N1 points whose
// x transform, multiplier and inverse serve both rows (z^(-k) = conj z^(k) in real space).  Rows
// that are their own mirror are done once.
// The multiplier beta dt^2 K(xi) + rhobar I: K[q][v] xi xi sums entry q (00 01 02 11 12 22) over the
// products v = 11 22 33 23 13 12 of the frequencies.  It and its inverse are formed in FP64 for FP32
// fields too, as its cofactors cancel: error of the FP32 preconditioner against 64 bits with an FP32
// inverse / with this, copper 256^3 2.91e-7 / 2.79e-7, 64^3 2.42e-7 / 2.32e-7, a Poisson ratio of 0.49999
// 16^3 2.3 / 2.1e-7.  x pass at 256^3 89 / 91 us, mixed step 29.86 / 30.00 ms.
struct PrecondParams {
    double K[6][6];
    double rhobar, inv_ntot;
    double k1, k2, k3;
    const double* mfreq;
    int n1, n2, n3, dim;
};

static PrecondParams precond_params(const SpecParams& sp)
{
    PrecondParams p;
    double C[6][6];
    for (int a = 0, o = 0; a < 6; a++)
        for (int b = a; b < 6; b++, o++) C[a][b] = C[b][a] = sp.Cbar[o];
    static const int V[3][3] = {{0, 5, 4}, {5, 1, 3}, {4, 3, 2}}; // Voigt index of a pair
    static const int P[6][2] = {{0, 0}, {1, 1}, {2, 2}, {1, 2}, {0, 2}, {0, 1}};
    for (int i = 0, q = 0; i < 3; i++)
        for (int j = i; j < 3; j++, q++)
            for (int v = 0; v < 6; v++) {
                // K_ij = Cbar_ikjm xi_k xi_m (eq. acous)
                const int k = P[v][0], m = P[v][1];
                const double c = C[V[i][k]][V[j][m]] + (k != m ? C[V[i][m]][V[j][k]] : 0.0);
                p.K[q][v] = sp.bdt2 * c;
            }
    p.rhobar = sp.rhobar;
    p.inv_ntot = sp.inv_ntot;
    p.k1 = sp.k1;
    p.k2 = sp.k2;
    p.k3 = sp.k3;
    p.mfreq = sp.mfreq;
    p.n1 = sp.n1;
    p.n2 = sp.n2;
    p.n3 = sp.n3;
    p.dim = sp.dim;
    return p;
}

template <typename T, int N1> struct XPShape {
    static constexpr int R = 8, G = N1 / R;
};

template <typename T, int N1, int BLK, int MEM>
__global__ __launch_bounds__(BLK, (x_waves<T, BLK>(kXPrecondWaves64, kXPrecondWaves32)))
    void k_xprecond(PrecondParams sp, Layout lay, const cx_t<T>* __restrict__ src,
                                                                    long sc, long sb, cx_t<T>* __restrict__ dst, int nlines,
                                                                    int nfull, const cx_t<T>* __restrict__ tw,
                                                                    double* __restrict__ partials, Carry carry)
{
    using V = cx_t<T>;
    using Sh = XPShape<T, N1>;
    constexpr bool SMALL = BLK != kBlock;
    constexpr int R = Sh::R, G = Sh::G, LPB = BLK / G, M = N1 / 2, NT = NM_NT(XP, T);
    constexpr int LP = line_elems(N1), AREA = LPB * LP;
    __shared__ V lds[AREA];
    __shared__ V tws[N1];
    TwStage<N1, BLK, V> tst;
    if constexpr (SMALL) tst.fetch(tw);
    if (stopped(lay.stop)) return;
    const int fld = blockIdx.z;
    int blk = blockIdx.x;
    if (carry.action != RED_NONE) {
        if (blk == 0) {
            carry_reduce<BLK>(carry, fld);
            return;
        }
        blk--;
    }
    if constexpr (!SMALL) {
        // (tables ahead of the operands here: held over their store, the operands spill in FP64)
        tst.fetch(tw);
        tst.store(tws);
        __syncthreads();
    }
    const int ll = threadIdx.x / G, t = threadIdx.x % G;
    const int ln = blk * LPB + ll;
    const bool valid = ln < nlines;
    // kz in (0, n3/2): every ky; kz = 0 and n3/2: ky <= n2/2
    int ky, kz;
    if (ln < nfull) {
        kz = 1 + ln / lay.n2;
        ky = ln & (lay.n2 - 1);
    } else {
        const int i = valid ? ln - nfull : 0, half = lay.n2 / 2 + 1;
        kz = i < half ? 0 : lay.n3 / 2;
        ky = i < half ? i : i - half;
    }
    const int my = (lay.n2 - ky) & (lay.n2 - 1), mz = (lay.n3 - kz) & (lay.n3 - 1);
    const bool self = my == ky && mz == kz;
    const uint32_t o1 = ((uint32_t)kz * lay.n2 + ky) * M + t, o2 = ((uint32_t)mz * lay.n2 + my) * M + t;
    const V* const in = src + (long)fld * sb;
    V* const out = dst + (long)fld * lay.bs;
    const LineAddr<AREA> addr{ll * LP};
    V v[3][R];
    {
        V ca[3][R / 2], cb[3][R / 2];
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int m = 0; m < R / 2; m++) {
                ca[j][m] = ld_nt<NT>(in + j * sc + (o1 + m * G));
                cb[j][m] = ld_nt<NT>(in + j * sc + (o2 + m * G));
            }
        if constexpr (SMALL) {
            tst.store(tws);
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int m = 0; m < R / 2; m++) {
                const V x = ca[j][m], y = cb[j][m];
                v[j][2 * m] = V{(T)0.5 * (x.x + y.x), (T)0.5 * (x.y - y.y)};
                v[j][2 * m + 1] = V{(T)0.5 * (x.y + y.y), (T)-0.5 * (x.x - y.x)};
            }
    }
    // one component at a time: three together (one synchronisation per stage) need 64 KB of LDS per
    // block, which left two blocks per compute unit (FP32, 256^3: 0.0857 against 0.0718 ms)
#pragma unroll
    for (int j = 0; j < 3; j++) group_fft<N1, R, -1, true, FFT_PAIR_IN, 1>((V(&)[1][R])v[j], t, lds, addr, tws);
    // beta dt^2 K(xi) + rhobar I at fixed (xi2, xi3) is quadratic in xi1: A0 + xi1 (A1 + xi1 A2), formed
    // once per thread (symmetric; upper triangles kept, order 00 01 02 11 12 22)
    double A0[6], A1[6];
    {
        const double x2 = sp.mfreq ? sp.mfreq[sp.n1 + ky] : sp.k2 * freq_index(ky, sp.n2);
        const double x3 = sp.mfreq ? sp.mfreq[sp.n1 + sp.n2 + kz] : sp.k3 * freq_index(kz, sp.n3);
#pragma unroll
        for (int q = 0; q < 6; q++) {
            A0[q] = x2 * (sp.K[q][1] * x2 + sp.K[q][3] * x3) + sp.K[q][2] * x3 * x3;
            A1[q] = sp.K[q][5] * x2 + sp.K[q][4] * x3;
        }
        A0[0] += sp.rhobar;
        A0[3] += sp.rhobar;
        A0[5] += sp.rhobar;
    }
    // per-thread part of r . z: products of one bin in the working precision, summed in FP64
    double part = 0.0;
#pragma unroll
    for (int m = 0; m < R; m++) {
        const int kx = t + m * G;
        const double x1 = sp.mfreq ? sp.mfreq[kx] : sp.k1 * freq_index(kx, N1);
        double Kx[6];
#pragma unroll
        for (int q = 0; q < 6; q++) Kx[q] = A0[q] + x1 * (A1[q] + x1 * sp.K[q][0]);
        const double k00 = Kx[0], k01 = Kx[1], k02 = Kx[2], k11 = Kx[3], k12 = Kx[4], k22 = Kx[5];
        const V r0 = v[0][m], r1 = v[1][m], r2 = v[2][m];
        V z0, z1, z2;
        if (sp.dim == 2) {
            const double id = sp.inv_ntot / (k00 * k11 - k01 * k01);
            const T d00 = (T)(k11 * id), d01 = (T)(k01 * id), d11 = (T)(k00 * id);
            z0 = csub(cscale(r0, d00), cscale(r1, d01));
            z1 = csub(cscale(r1, d11), cscale(r0, d01));
            z2 = V{0, 0};
        } else {
            // inverse of the symmetric 3x3 by cofactors
            const double c00 = k11 * k22 - k12 * k12;
            const double c01 = k02 * k12 - k01 * k22;
            const double c02 = k01 * k12 - k02 * k11;
            const double c11 = k00 * k22 - k02 * k02;
            const double c12 = k02 * k01 - k00 * k12;
            const double c22 = k00 * k11 - k01 * k01;
            const double id = sp.inv_ntot / (k00 * c00 + k01 * c01 + k02 * c02);
            const T d00 = (T)(c00 * id), d01 = (T)(c01 * id), d02 = (T)(c02 * id), d11 = (T)(c11 * id),
                    d12 = (T)(c12 * id), d22 = (T)(c22 * id);
            z0 = cadd(cadd(cscale(r0, d00), cscale(r1, d01)), cscale(r2, d02));
            z1 = cadd(cadd(cscale(r0, d01), cscale(r1, d11)), cscale(r2, d12));
            z2 = cadd(cadd(cscale(r0, d02), cscale(r1, d12)), cscale(r2, d22));
        }
        part += (double)(r0.x * z0.x + r0.y * z0.y + r1.x * z1.x + r1.y * z1.y + r2.x * z2.x + r2.y * z2.y);
        asm volatile("" : "+v"(part)); // due here, not where it is used
        __builtin_amdgcn_sched_barrier(0);
        v[0][m] = z0;
        v[1][m] = z1;
        v[2][m] = z2;
    }
#pragma unroll
    for (int j = 0; j < 3; j++) group_fft<N1, R, +1, true, FFT_PAIR_OUT, 1>((V(&)[1][R])v[j], t, lds, addr, tws);
    if (valid) {
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int m = 0; m < R / 2; m++) {
                const V x = v[j][2 * m], y = v[j][2 * m + 1];
                st_nt<NT>(out + j * lay.cs + (o1 + m * G), V{x.x - y.y, x.y + y.x});
                if (!self) st_nt<NT>(out + j * lay.cs + (o2 + m * G), V{x.x + y.y, y.x - x.y});
            }
    }
    if (partials) {
        // a row and its mirror contribute the same
        const double tot = block_sum<BLK>(valid ? (self ? 1.0 : 2.0) * part : 0.0);
        if (threadIdx.x == 0) partials[(long)fld * ((nlines + LPB - 1) / LPB) + blk] = tot;
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
#define NM_SIZE_SWITCH(n, ...)                                                                                         \
    switch (n) {                                                                                                       \
    case 8: { constexpr int NN = 8; __VA_ARGS__; } break;                                                              \
    case 16: { constexpr int NN = 16; __VA_ARGS__; } break;                                                            \
    case 32: { constexpr int NN = 32; __VA_ARGS__; } break;                                                            \
    case 64: { constexpr int NN = 64; __VA_ARGS__; } break;                                                            \
    case 128: { constexpr int NN = 128; __VA_ARGS__; } break;                                                          \
    case 256: { constexpr int NN = 256; __VA_ARGS__; } break;                                                          \
    case 512: { constexpr int NN = 512; __VA_ARGS__; } break;                                                          \
    default: return -1;                                                                                                \
    }

static Cols y_cols(const Layout& l)
{
    return Cols{l.M * l.n3, l.log2M, l.M - 1, (long)l.n2 * l.M, (long)l.M};
}
static Cols z_cols(const Layout& l) { return Cols{l.M * l.n2, 31, 0x7fffffff, 0, (long)l.n2 * l.M}; }
static AxisFreq axis_freq(const SpecParams& sp, int axis)
{
    const double k[3] = {sp.k1, sp.k2, sp.k3}, in[3] = {sp.inv_n1, sp.inv_n2, sp.inv_n3};
    const int n[3] = {sp.n1, sp.n2, sp.n3}, off[3] = {0, sp.n1, sp.n1 + sp.n2};
    return AxisFreq{sp.mfreq ? sp.mfreq + off[axis] : nullptr, k[axis], in[axis], n[axis]};
}
// Whether the fields of a conjugate-gradient iteration (work buffers 8, direction, iterate, residual) about fit
// the 256 MB last-level cache.
// FP64 iteration plain / streaming: 285 MB 258.5 / 264.5 us, 570 MB (256x128x128) 489.8 / 481.5,
// 1.14 GB 1049 / 933; mixed step 285 MB 4.70 / 4.80 ms, 570 MB 8.96 / 8.69.
constexpr long kPlainBytes = 320L << 20;
template <typename T> static bool plain_memory(const Layout& l)
{
    return 17 * l.ns * l.nb * (long)sizeof(cx_t<T>) <= kPlainBytes;
}

// fn(threads per block and memory setting as constants, tiles) for the columns g of L points.
template <typename T, int L, typename F> static void col_shape(const Layout& l, const Cols& g, F&& fn)
{
    using Plain = std::integral_constant<int, MEM_PLAIN>;
    using Stream = std::integral_constant<int, MEM_STREAM>;
    constexpr int G = L / col_radix<T, L>(), BIG = col_block<T, L>(), SM = col_small_block<T, L>();
    auto tiles = [&](int blk) { return (g.ncols + blk / G - 1) / (blk / G); };
    if constexpr (SM < BIG) {
        if (3 * tiles(BIG) < kColSmallBlocks) {
            fn(std::integral_constant<int, SM>{}, Stream{}, tiles(SM));
            return;
        }
    }
    if (plain_memory<T>(l)) fn(std::integral_constant<int, BIG>{}, Plain{}, tiles(BIG));
    else fn(std::integral_constant<int, BIG>{}, Stream{}, tiles(BIG));
}
static int ok() { return hipGetLastError() == hipSuccess ? 0 : -2; }

// Launch K<T, NN, BLK, MEM, ...> on the columns of `n` points; extra: blocks ahead of the tiles'.
#define NM_COL_LAUNCH(n, l, g, extra, s, K, ...)                                                                       \
    NM_SIZE_SWITCH(n, (col_shape<T, NN>(l, g, [&](auto blk, auto mem, int nt) {                                        \
                       constexpr int BLK = decltype(blk)::value, MEM = decltype(mem)::value;                           \
                       hipLaunchKernelGGL(K, dim3(3 * nt + (extra), 1, (l).nb), dim3(BLK), 0, s, __VA_ARGS__, nt,      \
                                          (const cx_t<T>*)tw);                                                         \
                   })))

template <typename T> int launch_ystart(int mode, const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s)
{
    const Cols g = y_cols(a.lay);
    const AxisFreq f = axis_freq(sp, 1);
    if (mode == YS_APPLY) {
        NM_COL_LAUNCH(a.lay.n2, a.lay, g, 0, s, (k_ystart<T, NN, BLK, MEM, YS_APPLY>), a, g, f)
    } else if (mode == YS_PCG) {
        NM_COL_LAUNCH(a.lay.n2, a.lay, g, 0, s, (k_ystart<T, NN, BLK, MEM, YS_PCG>), a, g, f)
    } else if constexpr (sizeof(T) == 8) { // the explicit scheme runs in FP64
        NM_COL_LAUNCH(a.lay.n2, a.lay, g, 0, s, (k_ystart<T, NN, BLK, MEM, YS_EXPLICIT>), a, g, f)
    } else {
        return -1;
    }
    return ok();
}

template <typename T> int launch_zstrain(const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s)
{
    const Cols g = z_cols(a.lay);
    const AxisFreq f = axis_freq(sp, 2);
    NM_COL_LAUNCH(a.lay.n3, a.lay, g, 0, s, (k_zstrain<T, NN, BLK, MEM>), a, g, f)
    return ok();
}

template <typename T> int launch_zdiv(const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s)
{
    const Cols g = z_cols(a.lay);
    const AxisFreq f = axis_freq(sp, 2);
    NM_COL_LAUNCH(a.lay.n3, a.lay, g, a.carry.action != RED_NONE, s, (k_zdiv<T, NN, BLK, MEM>), a, g, f)
    return ok();
}

template <typename T> int yend_blocks(const Layout& l)
{
    int nb = 0;
    auto count = [&]() -> int {
        NM_SIZE_SWITCH(l.n2, (col_shape<T, NN>(l, y_cols(l), [&](auto, auto, int nt) { nb = 3 * nt; })))
        return 0;
    };
    count();
    return nb;
}

template <typename T> int launch_yend(int mode, const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s)
{
    const Cols g = y_cols(a.lay);
    const AxisFreq f = axis_freq(sp, 1);
    if (mode == YE_OUT) {
        NM_COL_LAUNCH(a.lay.n2, a.lay, g, 0, s, (k_yend<T, NN, BLK, MEM, YE_OUT>), a, g, f)
    } else if (mode == YE_UPDATE) {
        NM_COL_LAUNCH(a.lay.n2, a.lay, g, 0, s, (k_yend<T, NN, BLK, MEM, YE_UPDATE>), a, g, f)
    } else if (mode == YE_RESIDUAL) {
        NM_COL_LAUNCH(a.lay.n2, a.lay, g, 0, s, (k_yend<T, NN, BLK, MEM, YE_RESIDUAL>), a, g, f)
    } else if constexpr (sizeof(T) == 8) {
        if (mode == YE_EXPLICIT) {
            NM_COL_LAUNCH(a.lay.n2, a.lay, g, 0, s, (k_yend<T, NN, BLK, MEM, YE_EXPLICIT>), a, g, f)
        } else {
            NM_COL_LAUNCH(a.lay.n2, a.lay, g, 0, s, (k_yend<T, NN, BLK, MEM, YE_EXPLICIT_NEXT>), a, g, f)
        }
    } else {
        return -1;
    }
    return ok();
}

template <typename T> int launch_colfft(const ColFft& f, const void* tw, hipStream_t s)
{
    const Cols g = f.axis == 1 ? y_cols(f.lay) : z_cols(f.lay);
    const int n = f.axis == 1 ? f.lay.n2 : f.lay.n3, extra = f.carry.action != RED_NONE;
    if (f.dir < 0) {
        NM_COL_LAUNCH(n, f.lay, g, extra, s, (k_colfft<T, NN, BLK, MEM, -1>), f, g)
    } else {
        NM_COL_LAUNCH(n, f.lay, g, extra, s, (k_colfft<T, NN, BLK, MEM, +1>), f, g)
    }
    return ok();
}

// Blocks of an x pass over `lines` groups of n1 / R lanes, and their threads (see kXSmallBlocks).
static int x_blocks(int n1, int R, int lines, int* threads)
{
    const int G = n1 / R, small = G > 64 ? G : 64;
    int blk = kBlock, nb = (lines + blk / G - 1) / (blk / G);
    if (nb < kXSmallBlocks) {
        blk = small;
        nb = (lines + blk / G - 1) / (blk / G);
    }
    *threads = blk;
    return nb;
}

// Launch an x pass K<T, NN, BLK, MEM> of R elements per thread on `grid` blocks of `threads` threads.
#define NM_X_LAUNCH(K, R, l, ...)                                                                                      \
    if (threads != kBlock) {                                                                                           \
        constexpr int BLK = x_small_block<NN, R>(), MEM = MEM_STREAM;                                                  \
        hipLaunchKernelGGL(K, grid, dim3(BLK), 0, s, __VA_ARGS__);                                                     \
    } else if (plain_memory<T>(l)) {                                                                                   \
        constexpr int BLK = kBlock, MEM = MEM_PLAIN;                                                                   \
        hipLaunchKernelGGL(K, grid, dim3(BLK), 0, s, __VA_ARGS__);                                                     \
    } else {                                                                                                           \
        constexpr int BLK = kBlock, MEM = MEM_STREAM;                                                                  \
        hipLaunchKernelGGL(K, grid, dim3(BLK), 0, s, __VA_ARGS__);                                                     \
    }

template <typename T> int xstress_blocks(const Layout& l)
{
    int threads;
    return x_blocks(l.n1, kXR, l.n2 / 2 * l.n3, &threads);
}

template <typename T> int launch_xstress(const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s)
{
    const AxisFreq f = axis_freq(sp, 0);
    const int np = a.lay.n2 / 2 * a.lay.n3;
    int threads;
    const dim3 grid(x_blocks(a.lay.n1, kXR, np, &threads), 1, a.lay.nb);
    NM_SIZE_SWITCH(a.lay.n1, {
        NM_X_LAUNCH((k_xstress<T, NN, BLK, MEM>), kXR, a.lay, a, f, np, (const cx_t<T>*)tw);
    })
    return ok();
}

// Rows (ky, kz) of which one of each mirrored couple is taken; `full` of them belong to 0 < kz < n3/2.
static int mirror_rows(const Layout& l, int* full)
{
    *full = l.n3 > 1 ? (l.n3 / 2 - 1) * l.n2 : 0;
    return *full + (l.n2 / 2 + 1) * (l.n3 > 1 ? 2 : 1);
}

template <typename T> int xprecond_blocks(const Layout& l)
{
    int full, threads;
    return x_blocks(l.n1, XPShape<T, 8>::R, mirror_rows(l, &full), &threads);
}

template <typename T>
int launch_xprecond(const SpecParams& sp, const Layout& lay, const void* src, long sc, long sb, void* S2, const void* tw,
                    hipStream_t s, double* partials, const Carry& carry)
{
    int full, threads;
    const int rows = mirror_rows(lay, &full);
    const dim3 grid(x_blocks(lay.n1, XPShape<T, 8>::R, rows, &threads) + (carry.action != RED_NONE), 1, lay.nb);
    const PrecondParams pp = precond_params(sp);
    NM_SIZE_SWITCH(lay.n1, {
        NM_X_LAUNCH((k_xprecond<T, NN, BLK, MEM>), (XPShape<T, NN>::R), lay, pp, lay, (const cx_t<T>*)src, sc, sb,
                    (cx_t<T>*)S2, rows, full, (const cx_t<T>*)tw, partials, carry);
    })
    return ok();
}

#define NM_INST(T)                                                                                                     \
    template int xstress_blocks<T>(const Layout&);                                                                     \
    template int yend_blocks<T>(const Layout&);                                                                        \
    template int xprecond_blocks<T>(const Layout&);                                                                    \
    template int launch_ystart<T>(int, const SpecParams&, const PassArgs&, const void*, hipStream_t);                  \
    template int launch_zstrain<T>(const SpecParams&, const PassArgs&, const void*, hipStream_t);                      \
    template int launch_xstress<T>(const SpecParams&, const PassArgs&, const void*, hipStream_t);                      \
    template int launch_zdiv<T>(const SpecParams&, const PassArgs&, const void*, hipStream_t);                         \
    template int launch_yend<T>(int, const SpecParams&, const PassArgs&, const void*, hipStream_t);                    \
    template int launch_colfft<T>(const ColFft&, const void*, hipStream_t);                                            \
    template int launch_xprecond<T>(const SpecParams&, const Layout&, const void*, long, long, void*, const void*,     \
                                    hipStream_t, double*, const Carry&);
NM_INST(double)
NM_INST(float)

} // namespace nm
