// Host-side launchers of the FFT pass kernels (implemented in nm_passes.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nm {

// Spectral constants of the operator and of the reference-medium preconditioner.
struct SpecParams {
    double L1, L2, L3;
    double k1, k2, k3; // 2 pi / L_i
    int n1, n2, n3;
    int dim;          // 2 (plane strain, n3 == 1, z components held at zero) or 3
    double inv_ntot;  // 1 / (n1 n2 n3): normalization of one forward/inverse round trip
    double inv_n1, inv_n2, inv_n3;
    double bdt2;      // beta dt^2
    double rhobar;    // volume-averaged density
    double Cbar[21];  // volume-averaged Voigt stiffness (upper triangle, row major)
    // Finite-difference differentiation rules: device table of the frequency each bin's
    // derivative uses in place of the spectral xi (n1 + n2 + n3 entries, axis after axis, indexed
    // by bin), or null for the spectral derivative.
    const double* mfreq = nullptr;
};

// Geometry of one launch.  Every buffer is a set of components of n3 x n2 rows of M = n1/2
// elements; an element V is a pair of neighbouring voxels (x, x + 1) in real space, or what the y
// and z transforms make of it (the transforms of a pair run as one complex transform).
// Several fields at once (multi-right-hand-side solves): nb fields, the real ones bf elements
// apart, the work buffers bs elements apart, device scalars S_COUNT apart.
struct Layout {
    int M = 0, log2M = 0;
    int n1 = 0, n2 = 0, n3 = 0;
    int dim = 3;
    long ns = 0; // component stride of the real fields (n1 n2 n3 / 2 elements)
    long cs = 0; // component stride of the work buffers, >= ns (padded off powers of two)
    long bf = 0, bs = 0;
    int nb = 1;
    const double* stop = nullptr; // device flag: when non-zero, kernels given this layout exit at once
};

// Device scalar block shared by the Krylov kernels (all double).
// S_STOP .. S_MODE drive a Krylov loop that runs several iterations between host checks:
// the residual reduction counts iterations (S_ITER) and raises S_STOP once r.r <= S_THR2
// (S_MODE 0) or the count reaches S_LIMIT; every guarded kernel after that returns at once.
// The pass that carries that reduction is guarded by S_HALT instead, which the first pass of an iteration
// raises when it finds S_STOP set: no launch reads the flag that it raises, so that a block's
// wavefronts always take the same side of the guard.
enum ScalarSlot {
    S_ALPHA = 0, S_BETA = 1, S_FIRST = 2, S_RZ = 3, S_PQ = 4, S_RR = 5,
    S_RZ2 = 7, // r.z of the iteration under way (2D, see PassArgs::carry)
    S_STOP = 8, S_ITER = 9, S_THR2 = 10, S_LIMIT = 11, S_MODE = 12, S_HALT = 13, S_COUNT = 16
};

// What a sum of per-block partials does to the scalar block.
enum ReduceAction {
    RED_NONE = -1, RED_STORE_RR = 0, RED_ALPHA = 1, RED_RZ_INIT = 2, RED_BETA = 3, RED_STORE_SLOT = 4, RED_RR_CHECK = 5
};

// A reduction carried by a pass: its first block (one per field) sums n partials of the
// pass before, field b's at part + b n, into scal + b S_COUNT.  multi: a loop whose S_STOP is set
// is frozen (alpha = beta = 0) instead of skipped.
struct Carry {
    const double* part = nullptr;
    int n = 0;
    double* scal = nullptr;
    int action = RED_NONE;
    int multi = 0;
};

// First pass of the operator, y columns: D_y of the three components into work components 0..2.
//   YS_APPLY    the field u as it is
//   YS_EXPLICIT v <- v + dt/2 a (the velocity half a step on), u <- u + dt v first (central differences,
//               eq. Central_diff_rule)
//   YS_PCG      z = mask(y-inverse of Z), p = z + beta p, x += alpha p_old (p = z, x untouched while
//               S_FIRST is set), then D_y p: the preconditioner's last pass, the direction update
//               and the operator's first pass in one
enum YStartMode { YS_APPLY = 0, YS_EXPLICIT = 1, YS_PCG = 2 };
// Last pass of the operator, y columns: q_j = Q_j - beta dt^2 D_y sigma_2j.
//   YE_OUT      q (masked) to out
//   YE_UPDATE   r_j <- mask(r_j - alpha q_j), held and left as its y spectrum R_j, with the partial sums of r.r
//   YE_EXPLICIT o = q, the last step of a batch: v <- v + o / rho, a <- 2 o / (dt rho)
//   YE_EXPLICIT_NEXT a step with a next one behind it: this step's end and the next one's YS_EXPLICIT
//               in one, v <- v + 2 o / rho (Gamma voxels, whose v is already the next half step's: v as it
//               is), u <- u + dt v, D_y u into work components 0..2; a is not needed in between
//   YE_RESIDUAL r = mask(b - q), also rounded to FP32 (r32, or null), with the partial sums of r.r
enum YEndMode { YE_OUT = 0, YE_UPDATE = 1, YE_EXPLICIT = 2, YE_EXPLICIT_NEXT = 3, YE_RESIDUAL = 4 };

struct PassArgs {
    Layout lay;
    void* S = nullptr;         // work buffer (5 components): derivatives, then stresses
    void* S2 = nullptr;        // work buffer (3 components): the preconditioner's spectrum between its first
                               // pass and YS_PCG, Q (inertia and divergence) between the stress pass and the last
    void* u = nullptr;         // YS_APPLY: field (in); explicit scheme: displacement (in/out)
    void* p = nullptr;         // YS_PCG: search direction (in/out); z and x passes: the field derived
    void* x = nullptr;         // YS_PCG: iterate (in/out)
    void* v = nullptr;         // explicit scheme: velocity
    void* a = nullptr;         // explicit scheme: acceleration
    void* r = nullptr;         // YE_UPDATE: y spectrum of the residual (in/out)
    void* out = nullptr;       // YE_OUT: result; YE_RESIDUAL: the residual (real space)
    const void* b = nullptr;   // YE_RESIDUAL: right-hand side
    float* r32 = nullptr;      // YE_RESIDUAL
    const uint8_t* mask = nullptr;   // Gamma voxel mask or null
    const uint16_t* phase = nullptr; // grain ids
    const void* C21 = nullptr;       // per-grain stiffness
    const void* rho = nullptr;       // per-grain density, or null (no inertia term)
    double bdt2 = 0.0;               // the divergence is scaled by -bdt2
    double dt = 0.0;                 // explicit scheme
    double* scal = nullptr;          // device scalars
    double* partials = nullptr;      // per-block partial sums or null
    // z passes: the reduction they carry.  YS_PCG with RED_BETA and YE_UPDATE with RED_ALPHA (2D, where no z
    // pass lies between): every block sums the partials for itself.
    Carry carry;
};

// One transform along a column axis, component by component: src (component stride sc, field stride
// sb) to dst (dc, db), possibly in place; axis 1 = y, 2 = z; dir -1 forward, +1 inverse.  mask and
// zero3 (the third component becomes zero) apply to real results.
struct ColFft {
    Layout lay;
    const void* src = nullptr;
    void* dst = nullptr;
    long sc = 0, sb = 0, dc = 0, db = 0;
    int axis = 1, dir = -1;
    const uint8_t* mask = nullptr;
    int zero3 = 0;
    Carry carry;
};

// Number of partial sums per field that a pass leaves.
template <typename T> int xstress_blocks(const Layout& lay);
template <typename T> int yend_blocks(const Layout& lay);
template <typename T> int xprecond_blocks(const Layout& lay);

template <typename T> int launch_ystart(int mode, const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s);
// z columns (3D only): S3 = D_z p_1, S2 <- D_z p_2 + S2, S4 = D_z p_3 (components of S).
template <typename T> int launch_zstrain(const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s);
// x lines: D_x p, strain, sigma = C : eps (in place on S), Q_j = rho p_j - bdt2 D_x sigma_1j;
// partials: p . A p = sum rho p.p + bdt2 eps:sigma.
template <typename T> int launch_xstress(const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s);
// z columns (3D only): Q_j -= bdt2 D_z sigma_3j.
template <typename T> int launch_zdiv(const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s);
template <typename T> int launch_yend(int mode, const SpecParams& sp, const PassArgs& a, const void* tw, hipStream_t s);
template <typename T> int launch_colfft(const ColFft& f, const void* tw, hipStream_t s);
// x lines of the preconditioner on the (y, z) spectrum src (component stride sc, field stride sb),
// result to S2 components 0..2: x-forward, (beta dt^2 K + rhobar I)^-1 / (n1 n2 n3), x-inverse;
// partials (or null): per-block sums of r . z (Parseval); carry: a reduction on the way (2D).
template <typename T>
int launch_xprecond(const SpecParams& sp, const Layout& lay, const void* src, long sc, long sb, void* S2, const void* tw,
                    hipStream_t s, double* partials, const Carry& carry);

} // namespace nm
