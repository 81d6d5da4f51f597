// Kernel argument block shared by the step, adjoint and auxiliary kernels, and the
// per-node equilibrium coefficients built from it.
#pragma once

#include <cmath>

#include "internal.h"
#include "node.h"

namespace elbm {

template <class Real>
struct StepArgs {
    const void* src;
    void* dst;
    int nx, ny, nz, abb;
    long long n;
    Real phi_ref, eps, tau2, root_rho;
    Real scale, inv_scale;
    Real T[6];
    const Real* tfield;     // 6 values per row, node-major
    const uint8_t* phase;   // material index per node (row of tfield), or null: row = node
    int phase_max;          // largest valid material index
    Real u[3];
    const Real* ufield;
    Real ex[Q], r[Q], l[Q];  // E_i - 1, 1 / (W_i E_i), ln E_i of a uniform velocity
    Real R;
    const Real* rfield;
    Real src_mult;
    int has_src;
    Real phi_lo, phi_hi;
    int rest32;     // 16-bit forms: rest population in FP32 absorbing the rounding residuals
    int sround;     // 16-bit forms: stochastic rounding of the stores
    uint32_t tmix;  // hash of the time step, mixed into the rounding counters
    int xcd_remap;  // row-vector kernel: XCD slab block order (xcd_block)
    int rows;       // one-node-per-thread kernels, ragged row-vector: x-rows of a block
    int waves;      // row-vector kernel on ragged rows: wavefronts of a row
    int pitch;      // threads of a row in blocks of several rows, and 1 / pitch
    float inv_pitch;
    Real* lam_rec;
    uint8_t* br_rec;
    unsigned long long* counters;
    // adjoint only
    const Real* adj_in;
    Real* adj_out;
    Real* t_grad;
    const Real* lam_in;
    const uint8_t* br_in;
};

// Per-node retention tensor, stored node-major (6 values of node k at 6 k): three
// 2-wide loads per node, so the field is one contiguous stream instead of six planes.
__device__ __forceinline__ void load_t6(const float* tf, long long k, float (&T)[6]) {
    const float2* p = reinterpret_cast<const float2*>(tf + 6 * k);
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const float2 v = p[m];
        T[2 * m] = v.x;
        T[2 * m + 1] = v.y;
    }
}
__device__ __forceinline__ void load_t6(const double* tf, long long k, double (&T)[6]) {
    const double2* p = reinterpret_cast<const double2*>(tf + 6 * k);
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const double2 v = p[m];
        T[2 * m] = v.x;
        T[2 * m + 1] = v.y;
    }
}

// Accumulate 6 values into node k's slot of a node-major 6-vector field (dL/dT), with the
// same three 2-wide accesses, nontemporal (each slot is read and written once per reverse
// step).
typedef float nt_f2 __attribute__((ext_vector_type(2)));
typedef double nt_d2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void add_t6(float* tf, long long k, const float (&v)[6]) {
    nt_f2* p = reinterpret_cast<nt_f2*>(tf + 6 * k);
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        nt_f2 w = __builtin_nontemporal_load(p + m);
        w.x += v[2 * m];
        w.y += v[2 * m + 1];
        __builtin_nontemporal_store(w, p + m);
    }
}
__device__ __forceinline__ void add_t6(double* tf, long long k, const double (&v)[6]) {
    nt_d2* p = reinterpret_cast<nt_d2*>(tf + 6 * k);
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        nt_d2 w = __builtin_nontemporal_load(p + m);
        w.x += v[2 * m];
        w.y += v[2 * m + 1];
        __builtin_nontemporal_store(w, p + m);
    }
}

// Row of the tensor store that holds node k's T: the node itself for a per-node field, its
// material (clamped to the table) for a material table.
template <class Real>
__device__ __forceinline__ long long tensor_row(const StepArgs<Real>& a, long long k) {
    if (a.phase) return min(int(a.phase[k]), a.phase_max);
    return k;
}

// Equilibrium factors at one node: UM = 0 zero velocity (constants fold), 1 uniform
// velocity (host-computed factors), 2 velocity field (the node's velocity u0, u1, u2).
template <class Real, int UM>
__device__ __forceinline__ void coef_velocity(const StepArgs<Real>& a, Real u0, Real u1, Real u2,
                                              NodeCoef<Real>& c) {
    if constexpr (UM == 0) {
        c.u[0] = c.u[1] = c.u[2] = Real(0);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            c.ex[i] = Real(0);
            c.r[i] = Real(1.0 / weight(i));
            c.l[i] = Real(0);
        }
    } else if constexpr (UM == 1) {
        c.u[0] = a.u[0];
        c.u[1] = a.u[1];
        c.u[2] = a.u[2];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            c.ex[i] = a.ex[i];
            c.r[i] = a.r[i];
            c.l[i] = a.l[i];
        }
    } else {
        c.u[0] = u0;
        c.u[1] = u1;
        c.u[2] = u2;
        const Real uu = c.u[0] * c.u[0] + c.u[1] * c.u[1] + c.u[2] * c.u[2];
        c.ex[0] = -Real(1.5) * uu;
        rest_factors(c.ex[0], c.r[0], c.l[0]);
#pragma unroll
        for (int P = 1; P < Q; P += 2) {
            // opposite pair: E+- = 1 + a +- b with a = 4.5 (c.u)^2 - 1.5 u.u, b = 3 c.u; the
            // excesses a +- b are formed without the 1 so that they keep their relative
            // precision (the equilibrium only needs E - 1)
            const Real cu = cdot(P, c.u[0], c.u[1], c.u[2]);
            const Real ea = Real(4.5) * cu * cu - Real(1.5) * uu;
            const Real eb = Real(3) * cu;
            c.ex[P] = ea + eb;
            c.ex[P + 1] = ea - eb;
            pair_factors(P, c.ex[P], c.ex[P + 1], c.r[P], c.r[P + 1], c.l[P], c.l[P + 1]);
        }
    }
}

template <class Real, int UM>
__device__ __forceinline__ void node_coef(const StepArgs<Real>& a, int k, NodeCoef<Real>& c) {
    if constexpr (UM == 2)
        coef_velocity<Real, UM>(a, a.ufield[k], a.ufield[a.n + k], a.ufield[2 * a.n + k], c);
    else
        coef_velocity<Real, UM>(a, Real(0), Real(0), Real(0), c);
    if (a.tfield) {
        load_t6(a.tfield, tensor_row(a, k), c.T);
    } else {
#pragma unroll
        for (int m = 0; m < 6; ++m) c.T[m] = a.T[m];
    }
}

// Hash of a time step, mixed into the seeds of the stochastic rounding.
inline uint32_t step_mix(int64_t time) { return pcg_hash(uint32_t(time) ^ 0x9E3779B9u); }

// Read one word of every 64-byte line of a kernel's first argument, all in flight together. The
// arguments lie in host memory, a line is a trip of more than half a microsecond for the first
// wave that reads it, and the compiler reads them where they are used, in five to nine dependent
// groups. After this they come from the scalar cache. us per step: plume FP64 16^3 5.1 -> 3.8,
// 32^3 6.3 -> 5.1, 48^3 12.1 -> 11.1, FP32 32^3 4.5 -> 4.1; 200 x 150 x 100 within 1 %, mostly
// faster.
template <class Args>
__device__ __forceinline__ void touch_args() {
    typedef __attribute__((address_space(4))) const uint32_t* ptr;
    ptr p = (ptr)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int N = int((sizeof(Args) + 63) / 64);
    static_assert(N <= 24, "one operand per line");
    uint32_t v[24];
#pragma unroll
    for (int i = 0; i < 24; ++i) v[i] = p[16 * (i < N ? i : N - 1)];
    asm volatile("" ::"s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]), "s"(v[5]), "s"(v[6]), "s"(v[7]),
                 "s"(v[8]), "s"(v[9]), "s"(v[10]), "s"(v[11]), "s"(v[12]), "s"(v[13]), "s"(v[14]), "s"(v[15]),
                 "s"(v[16]), "s"(v[17]), "s"(v[18]), "s"(v[19]), "s"(v[20]), "s"(v[21]), "s"(v[22]), "s"(v[23]));
}

template <class Real>
inline StepArgs<Real> make_args(const elbm_lattice* h, double src_mult) {
    StepArgs<Real> a{};
    a.nx = h->cfg.nx;
    a.ny = h->cfg.ny;
    a.nz = h->cfg.nz;
    a.abb = h->cfg.bc_x == ELBM_DIRICHLET;
    a.n = h->n;
    a.phi_ref = Real(h->cfg.phi_ref);
    a.eps = Real(h->cfg.eps);
    a.tau2 = Real(h->cfg.ghost_floor * h->cfg.ghost_floor);
    a.root_rho = Real(h->cfg.root_rho);
    const bool scaled = h->cfg.precision == ELBM_FP16;
    a.scale = Real(scaled ? h->cfg.store_scale : 1.0);
    a.inv_scale = Real(scaled ? 1.0 / h->cfg.store_scale : 1.0);
    for (int m = 0; m < 6; ++m) a.T[m] = Real(h->T_u[m]);
    a.tfield = h->t_field_mode ? static_cast<const Real*>(h->t_field) : nullptr;
    a.phase = h->t_field_mode == 2 ? h->t_phase : nullptr;
    a.phase_max = h->nphase - 1;
    for (int m = 0; m < 3; ++m) a.u[m] = Real(h->u_mode == 1 ? h->u_u[m] : 0.0);
    a.ufield = h->u_mode == 2 ? static_cast<const Real*>(h->u_field) : nullptr;
    const double* u = h->u_u;
    const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    for (int i = 0; i < Q; ++i) {
        const double cu = cx(i) * u[0] + cy(i) * u[1] + cz(i) * u[2];
        const double ex = (h->u_mode == 1) ? 3.0 * cu + 4.5 * cu * cu - 1.5 * uu : 0.0;
        const double E = 1.0 + ex;
        a.ex[i] = Real(ex);
        a.r[i] = Real(1.0 / (weight(i) * E));
        a.l[i] = Real(std::log(E));
    }
    a.has_src = h->r_mode != 0;
    a.R = Real(h->r_mode == 1 ? h->r_u : 0.0);
    a.rfield = h->r_mode == 2 ? static_cast<const Real*>(h->r_field) : nullptr;
    a.src_mult = Real(src_mult);
    a.rest32 = (h->cfg.flags & ELBM_FLAG_REST_FP32) ? 1 : 0;
    a.sround = (h->cfg.flags & ELBM_FLAG_STOCHASTIC_ROUNDING) ? 1 : 0;
    a.tmix = step_mix(h->time);
    a.xcd_remap = 0;
    a.rows = 1;
    a.waves = 1;
    a.pitch = h->cfg.nx;
    a.inv_pitch = 1.0f;
    a.phi_lo = Real(h->phi_lo);
    a.phi_hi = Real(h->phi_hi);
    a.counters = h->d_cnt;
    return a;
}

// Launch shape of the one-node-per-thread kernels: a block takes `rows` whole x-rows, its
// threads numbered through them `pitch` per row (node_of), so that the x-shifted pushes stay
// inside the block's own cache lines and no line is written by two blocks (which may sit on
// different XCDs with separate L2s). Rows longer than max_threads are cut into segments of it.
//
// Padded: a row takes 32 or whole times 64 threads, rows are stacked to 256. Packed: as many
// rows as 256 threads hold, without gaps. Rows over 128 nodes stay alone either way. Packing
// leaves fewer threads idle, but a wavefront then covers parts of several rows and a block more
// nodes. Which is faster was measured on rows of 8 to 128 nodes (about 60 lengths), 1e3 to 6e6
// nodes, five kinds of coefficients and four forms; packed where
//  - it takes a fifth fewer threads, in blocks of four wavefronts: 33 x 67 x 68 FP64 1.23 times
//    as fast, 65- to 85-node rows 1.06-1.2 in every form, 1.25-1.39 with FP32 rest and SR; padded
//    is faster on 28- to 31- and 55- to 64-node rows (by 1-13 %), and by 5-10 % where two rows
//    make three wavefronts (86- to 96-node rows) but for the rounding forms on many blocks
//    (packed 1.13);
//  - the CU with the most blocks then has no more than 1 / 0.9 times the rows, 1 / 0.85 where
//    arithmetic bounds the kernel (blocks go round the CUs: where 270 packed blocks take two rounds
//    as 400 padded ones did, 0.76-0.9 times as fast without this condition);
//  - rows are not of 17 to 31 nodes (padded to 32, two per wavefront; FP32 and plain BF16 0.7-1.05
//    packed) and memory does not set the pace (state and coefficients beyond half of the 256 MB cache:
//    FP32 0.9-1.05, FP64 0.93-1.05, plain BF16 0.89-1.0, but 1.05-1.15 where packing takes 1.4 times
//    fewer threads), unless arithmetic bounds the kernel: FP32 rest or SR,
//    FP64 with a velocity per node (1.03-1.34 there), the exact root, the adjoint (1.02-1.3). Of 17
//    to 31 nodes those to 21 then (1.04-1.3; 23 x 511 x 511 BF16 with FP32 rest and SR 0.91).
// 16-bit forms whose fullest CU would get more rows in 256-thread blocks are packed into blocks of
// three or two wavefronts where it then does not (18 x 119 x 117 BF16 7.9 us against 9.4 padded).
// Over all of these sizes, against padded alone: FP64 1.03, FP32 1.01, BF16 1.05, BF16 with FP32
// rest and SR 1.1; one in a hundred below 0.95.
//
// A lattice that 256-thread blocks would put on a part of the CUs takes the smallest packed blocks
// that still find a CU each, if they have fewer wavefronts: 32^3 FP64 6.6 -> 5.4 us, FP32
// 4.6 -> 3.7, FP16 with FP32 rest and SR 5.1 -> 4.2 in 256 blocks of 128 threads.
struct RowRule {
    bool arith;     // arithmetic bounds the kernel
    bool rounding;  // 16-bit form with FP32 rest or stochastic rounding
    bool paced;     // memory does
    bool half;      // 16-bit form
};
template <class ST>
inline RowRule row_rule(const elbm_lattice* h) {
    RowRule r;
    r.half = sizeof(ST) == 2;
    r.rounding = r.half && (h->cfg.flags & (ELBM_FLAG_REST_FP32 | ELBM_FLAG_STOCHASTIC_ROUNDING));
    r.arith = r.rounding || (sizeof(ST) == 8 && h->u_mode == 2) || h->cfg.root_rho >= 0;
    const int coefs = (h->t_field_mode == 1 ? 6 : 0) + (h->u_mode == 2 ? 3 : 0) + (h->r_mode == 2 ? 1 : 0);
    r.paced = !r.arith && double(h->n) * (Q * sizeof(ST) + coefs * sizeof(typename Store<ST>::Real)) > 128e6;
    return r;
}

struct RowGrid {
    dim3 grid, block;
    int rows, pitch;

    template <class Args>
    void place(Args& a) const {
        a.rows = rows;
        a.pitch = pitch;
        a.inv_pitch = 1.0f / float(pitch);
    }
};
inline RowGrid grid_for(const elbm_lattice* h, const RowRule& rule, int max_threads = 512) {
    const int nx = h->cfg.nx, ny = h->cfg.ny, nz = h->cfg.nz;
    RowGrid g;
    g.rows = 1;
    if (nx > max_threads) {
        g.pitch = nx;
        g.block = dim3(max_threads);
        g.grid = dim3((nx + max_threads - 1) / max_threads, ny, nz);
        return g;
    }
    const auto waves = [](int threads) { return (threads + 63) / 64; };
    const auto blocks = [&](int rows) { return (long long)((ny + rows - 1) / rows) * nz; };
    const auto rounds = [&](int rows) { return (blocks(rows) + h->cus - 1) / h->cus; };
    g.pitch = nx <= 32 ? 32 : 64 * waves(nx);
    if (nx <= 128) {
        const int pad = min(256 / g.pitch, ny), most = min(256 / nx, ny);  // rows padded, packed
        const int pad_waves = waves(pad * g.pitch);
        g.rows = pad;
        int packed = 0;
        if (blocks(most) <= h->cus) {
            const int top = blocks(pad) <= h->cus ? pad : most;
            int r = 1;
            while (r < top && blocks(r) > h->cus) ++r;
            if (waves(r * nx) < pad_waves) packed = r;
        } else {
            const auto fewer = [&](int r) {  // wavefronts padded over those of r rows packed
                return double(pad_waves) * double(blocks(pad)) / (waves(r * nx) * double(blocks(r)));
            };
            const auto even = [&](int r) { return double(rounds(pad) * pad) / double(rounds(r) * r); };
            const bool many = rule.rounding && blocks(pad) >= 8 * h->cus;
            const bool halved = nx > 16 && nx < 32;  // padded to two rows per wavefront
            const bool paced = rule.paced && !(rule.half && fewer(most) >= 1.4);
            const int three = min(192 / nx, ny), two = min(128 / nx, ny);
            if (fewer(most) >= 1.2 && even(most) >= (rule.arith ? 0.85 : 0.9) && (waves(most * nx) == 4 || many) &&
                !paced && (!halved || (rule.arith && nx <= 21)))
                packed = most;
            else if (rule.half && !rule.paced && three > 1 && fewer(three) >= 1.2 && even(three) >= 1.0)
                packed = three;
            else if (rule.half && !rule.paced && two > 1 && fewer(two) >= 1.2 && even(two) >= 1.0)
                packed = two;
            else if (many && nx > 64 && ny <= 65535)  // one row per block in y, as far as a grid goes
                packed = 1;  // alone, its row in scalar registers (step_t): 1.03-1.08 times padded pairs
        }
        if (packed) {
            g.rows = packed;
            g.pitch = nx;
        }
    }
    g.block = dim3(64 * waves(g.rows * g.pitch));
    g.grid = dim3(1, (ny + g.rows - 1) / g.rows, nz);
    return g;
}

// Node of a thread of a RowGrid launch; false if it has none. The row of thread t of a block of
// several rows comes from a product with 1 / pitch (exact: t < 512 keeps (t + 1/2) / pitch further
// from whole numbers than the product's rounding). ROW: one row per block, so that y is the same
// for the block and stays in a scalar register, with every row address derived from it.
template <bool ROW, class Args>
__device__ __forceinline__ bool node_of(const Args& a, int& x, int& y) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if constexpr (ROW) {
        x = t;
        y = blockIdx.y;
        return x < a.nx;
    } else {
        const int q = a.rows == 1 ? 0 : int((float(t) + 0.5f) * a.inv_pitch);
        x = t - q * a.pitch;
        // keep x itself, not t, q and the pitch to make it from again: two registers, which were
        // two too many for four wavefronts per SIMD in D3Q27's plain 16-bit forms with a velocity
        // per node (130 VGPRs; 66 x 213 x 213 BF16 167 us per step, 143 at 128)
        asm("" : "+v"(x));
        y = blockIdx.y * a.rows + q;
        return x < a.nx && q < a.rows && y < a.ny;
    }
}

}  // namespace elbm
