// Two time steps in one launch (D3Q19, u = 0, FP64 and FP32 storage), the state between them
// kept on chip.
//
// A single step is bound by memory: every population is read once and written once
// (step_kernels.h). The state between two steps need not go to memory. A block owns a tile of
// bx x by columns and sweeps it along z, one plane per iteration:
//
//   - its threads own the tile and a halo of one column around it (rows only when a tile spans
//     the whole x-row, which closes periodic rows itself);
//   - iteration z collides the populations of plane z (first step) and puts the post-collision
//     values into LDS;
//   - with planes z - 2, z - 1 and z there, every node of plane z - 1 in the tile finds its Q
//     populations after the first step, collides again and pushes the result to the
//     destination buffer (second step).
//
// The populations of the next plane are loaded during the second step. Halo columns and the
// two planes around a sweep are collided by the neighbouring tiles too. The node arithmetic
// is that of the single-step kernels, so the state after the launch is bitwise that of two
// single steps.
//
// What bounds it on MI355X: not HBM, the counters read 2-11 % over one pass per two steps at
// 3.8-4.5 TB/s. Over all tilings an iteration of a full chip takes 1.2 us + 0.075 us per cache line
// and run of a block (pair_plan), which is why whole rows and wide tiles win although they
// recompute more. On the 256^3 decay in FP32, with tiles of two whole rows and as many halo rows,
// VALU issue is as busy (1.02 of SIMD cycles, 623 instructions per node and step against 373 in a
// single step; 150 us per step without memory accesses, 36 of that for the halo); elsewhere it is
// at 0.31-0.61. Per step, single steps against this kernel, same box: decay 256^3 FP32 429 -> 306
// us, FP64 893 -> 707; 384^3 FP32 1531 -> 1072, FP64 3516 -> 1913; porous 384^3 (walls, material
// table) FP32 1543 -> 1181, FP64 3017 -> 2263; 200 x 150 x 100 FP32 87 -> 63; 128^3 FP32 53 -> 42,
// FP64 105 -> 84; 96^3 FP32 21.9 -> 19.1.
// Not taken elsewhere, where it measured slower: with a velocity (256^3 plume FP32 428 -> 500,
// FP64 880 -> 945; 512^3 field FP64 8.6 -> 18.6 ms, spilled registers) and for the 16-bit
// forms (decay 256^3 BF16 216 -> 280), whose single steps are bound by VALU issue or close to
// it, so that a tile's recomputation costs more than the traffic saved. D3Q27 has no room: its
// exchange takes 48 LDS values per column.
#pragma once

#include "step_kernels.h"

namespace elbm {

// Tiling of a two-step launch, and what its second step has of its own.
template <class Real>
struct PairArgs : PairPlan {
    Real src_mult;   // source multiplier of the second step
    Real* lam_rec;   // its records
    uint8_t* br_rec;
};

// LDS planes of the exchange: the post-collision values of the directions with an x or y
// component. Those with c_z > 0 are read two planes after they were written, c_z = 0 one plane
// after, c_z < 0 in the same iteration; at a Dirichlet plane a reflected value is read by its
// own column one plane after. Rings of three, two and one (two with walls) planes: 32 (36)
// values per column. Held in registers instead, they made the kernel spill.
__host__ __device__ constexpr bool shared_dir(int i) { return cx(i) != 0 || cy(i) != 0; }
__host__ __device__ constexpr int group_dirs(int czv) {
    int n = 0;
    for (int k = 0; k < Q; ++k) n += (shared_dir(k) && cz(k) == czv) ? 1 : 0;
    return n;
}
__host__ __device__ constexpr int slot_in_group(int i) {
    int n = 0;
    for (int k = 0; k < i; ++k) n += (shared_dir(k) && cz(k) == cz(i)) ? 1 : 0;
    return n;
}
constexpr int kUp = group_dirs(1), kFlat = group_dirs(0), kDown = group_dirs(-1);
template <bool ABB>
constexpr int pair_slots() {
    return 3 * kUp + 2 * kFlat + (ABB ? 2 : 1) * kDown;
}

template <class Real>
__device__ inline void count_events(const StepArgs<Real>& a, const NodeOut<Real>& o, unsigned slot) {
    if (!a.counters) return;
    if (o.branch != 255) atomicAdd(a.counters + cnt_index(0, slot), 1ull);
    if (!isfinite(o.dphi)) atomicAdd(a.counters + cnt_index(2, slot), 1ull);
    if (o.guard) atomicAdd(a.counters + cnt_index(3, slot), 1ull);
}

// A barrier that orders LDS accesses only: the next plane's loads and the last one's stores
// stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The kernel's first argument, read again from the kernel argument segment: hidden from the
// optimiser, so that values that depend on arguments alone are not hoisted out of the sweep
// into registers that the collisions need.
template <class Real>
__device__ __forceinline__ const StepArgs<Real>& fresh_args() {
    typedef __attribute__((address_space(4))) const StepArgs<Real>* ptr;
    uintptr_t p = reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr());
    asm volatile("" : "+s"(p));
    return *(const StepArgs<Real>*)(ptr)p;
}

// Tensor of node k (TF: a field or a material table; otherwise uniform); the velocity is zero.
template <class Real, bool TF>
__device__ __forceinline__ void pair_coef(const StepArgs<Real>& a, int k, NodeCoef<Real>& c) {
    coef_velocity<Real, 0>(a, Real(0), Real(0), Real(0), c);
    if constexpr (TF) {
        load_t6(a.tfield, tensor_row(a, k), c.T);
    } else {
#pragma unroll
        for (int m = 0; m < 6; ++m) c.T[m] = a.T[m];
    }
}

// Every thread runs every iteration, those without a column or outside the tile on values that
// nobody reads: branches around the collisions cost 50-700 bytes of spilled registers.
template <class Real, bool TF, bool ABB, int NT>
__global__ __launch_bounds__(NT, sizeof(Real) == 4 ? 4 : 2) void k_step_pair(const StepArgs<Real> a_in,
                                                                             const PairArgs<Real> g) {
    constexpr int SB = int(sizeof(Real));
    constexpr bool CM = sizeof(Real) == 4;  // compensated mass sum (FP32 storage)
    // one value more at each end: the columns beside a Dirichlet plane at a row's end are read
    // before the wall node's own value replaces them
    __shared__ Real lds_all[pair_slots<ABB>() * NT + 2];
    Real(*const lds)[NT] = reinterpret_cast<Real(*)[NT]>(lds_all + 1);

    // Blocks go to the eight XCDs in turn: each XCD takes a contiguous eighth of the tiles, so
    // that neighbours share the halo's lines in its L2.
    const unsigned tiles = unsigned(g.tx) * unsigned(g.ty) * unsigned(g.tz);
    const unsigned tile = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (tile >= tiles) return;
    const unsigned tyz = tile / unsigned(g.tx);
    const int x0 = int(tile - tyz * unsigned(g.tx)) * g.bx;
    const int y0 = int(tyz % unsigned(g.ty)) * g.by;
    const int z0 = int(tyz / unsigned(g.ty)) * g.len;
    const int nx = a_in.nx, ny = a_in.ny, nz = a_in.nz;
    const int ox = min(g.bx, nx - x0), oy = min(g.by, ny - y0), planes = min(g.len, nz - z0);

    const int hx = g.tx == 1 ? 0 : 1;  // halo columns in x
    const int t = threadIdx.x, cw = g.bx + 2 * hx;
    const int ly = t / cw, lx = t - ly * cw;
    int gx = x0 - hx + lx, gy = y0 - 1 + ly;
    bool comp = lx < ox + 2 * hx && ly <= oy + 1;
    if (ABB && (gx < 0 || gx >= nx)) comp = false;  // no node beyond a Dirichlet plane
    gx = gx < 0 ? gx + nx : (gx >= nx ? gx - nx : gx);
    gy = gy < 0 ? gy + ny : (gy >= ny ? gy - ny : gy);
    const bool inner = comp && lx >= hx && lx < ox + hx && ly >= 1 && ly <= oy;
    if (!comp) gx = gy = 0;
    // the column whose neighbours this thread reads, and where they are in x
    const int tc = inner ? t : cw + hx;
    const int lc = inner ? lx : hx;
    const bool lo = ABB && gx == 0, hi = ABB && gx == nx - 1;
    const int xl = !ABB && lc == 0 ? cw - 1 : -1, xr = !ABB && lc == cw - 1 ? 1 - cw : 1;

    // Every access is a scalar base (plane and run) plus one of the thread's byte offsets
    // within a plane, which pair_plan keeps below 2^31.
    const size_t plane_bytes = size_t(ny) * Q * nx * SB;
    const uint32_t run_bytes = uint32_t(nx) * SB, row_bytes = Q * run_bytes;
    const char* src = static_cast<const char*>(a_in.src);
    char* dst = static_cast<char*>(a_in.dst);
    const uint32_t xs = uint32_t(gx) * SB, ys = uint32_t(gy) * row_bytes;
    const uint32_t xm = uint32_t(gx == 0 ? nx - 1 : gx - 1) * SB, xp = uint32_t(gx == nx - 1 ? 0 : gx + 1) * SB;
    const uint32_t ym = uint32_t(gy == 0 ? ny - 1 : gy - 1) * row_bytes;
    const uint32_t yp = uint32_t(gy == ny - 1 ? 0 : gy + 1) * row_bytes;
    const int col = gy * nx + gx, nxy = nx * ny;

    Real d[Q];
    auto load_plane = [&](int z) {
        const char* p = src + size_t(z) * plane_bytes;
#pragma unroll
        for (int i = 0; i < Q; ++i) d[i] = *reinterpret_cast<const Real*>(p + size_t(i) * run_bytes + (xs + ys));
    };

    int z = z0 == 0 ? nz - 1 : z0 - 1;
    load_plane(z);
    // post-collision values that stay in the column: rest and +z of the plane before, +z of two before
    static_assert(cx(5) == 0 && cy(5) == 0 && cz(5) == 1, "direction 5 is +z");
    Real rest1 = Real(0), up1 = Real(0), up2 = Real(0);
    // first LDS plane of each group: this plane (0), the one before (1), two before (2)
    int u0 = 0, u1 = kUp, u2 = 2 * kUp, f0 = 3 * kUp, f1 = 3 * kUp + kFlat;
    int w0 = 3 * kUp + 2 * kFlat, w1 = w0 + (ABB ? kDown : 0);
    for (int s = 0; s < planes + 2; ++s) {
        // first step: plane z
        Real post[Q];
        {
            const StepArgs<Real>& a = fresh_args<Real>();
            const int k = z * nxy + col;
            NodeCoef<Real> c;
            pair_coef<Real, TF>(a, k, c);
            if (a.has_src) {
                const Real R = (a.rfield ? a.rfield[k] : a.R) * a.src_mult;
#pragma unroll
                for (int i = 0; i < Q; ++i) d[i] += R * Real(weight(i)) * (Real(1) + c.ex[i]);
            }
            NodeOut<Real> o;
            collide<Real, 0, false, CM>(d, c, a.phi_ref, a.eps, a.tau2, a.root_rho, post, o);
            if (inner && s >= 1 && s <= planes) {
                if (a.lam_rec) {
                    a.lam_rec[k] = o.lam;
                    a.br_rec[k] = uint8_t(o.branch);
                }
                count_events(a, o, blockIdx.x);
            }
            if (ABB && (lo || hi)) reflect_at_walls(post, lo, hi, a.phi_lo, a.phi_hi, a.phi_ref, o.dphi);
        }
        lds_barrier();  // every thread has read the last iteration's planes
#pragma unroll
        for (int i = 0; i < Q; ++i)
            if (shared_dir(i)) lds[(cz(i) > 0 ? u0 : (cz(i) == 0 ? f0 : w0)) + slot_in_group(i)][t] = post[i];
        lds_barrier();
        // The second step's coefficients before the next plane's populations: loads return in
        // order, so a wait for a later one would wait for those too.
        const StepArgs<Real>& a = fresh_args<Real>();
        const int zn = z == nz - 1 ? 0 : z + 1;
        const int z1 = z0 + s - 2, k1 = max(z1, 0) * nxy + col;
        NodeCoef<Real> c1;
        Real R1 = Real(0);
        if (s >= 2) {
            pair_coef<Real, TF>(a, k1, c1);
            if (a.has_src) R1 = (a.rfield ? a.rfield[k1] : a.R) * g.src_mult;
        }
        if (s + 1 < planes + 2) load_plane(zn);
        if (s >= 2) {
            // second step: plane z - 1
            Real in[Q], out[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                if (shared_dir(i)) {
                    const int from = (cz(i) > 0 ? u2 : (cz(i) == 0 ? f1 : w0)) + slot_in_group(i);
                    in[i] = lds[from][tc + (cx(i) > 0 ? xl : (cx(i) < 0 ? xr : 0)) - cy(i) * cw];
                    if (ABB && cx(i)) {
                        // a wall node's own reflected value, of the same plane
                        const int own = (cz(i) > 0 ? w1 : (cz(i) == 0 ? f1 : u1)) + slot_in_group(opp(i));
                        if ((cx(i) > 0 && lo) || (cx(i) < 0 && hi)) in[i] = lds[own][t];
                    }
                } else {
                    in[i] = cz(i) > 0 ? up2 : (cz(i) == 0 ? rest1 : post[i]);
                }
            }
            if (a.has_src) {
#pragma unroll
                for (int i = 0; i < Q; ++i) in[i] += R1 * Real(weight(i)) * (Real(1) + c1.ex[i]);
            }
            NodeOut<Real> o;
            collide<Real, 0, false, CM>(in, c1, a.phi_ref, a.eps, a.tau2, a.root_rho, out, o);
            if (inner) {
                if (g.lam_rec) {
                    g.lam_rec[k1] = o.lam;
                    g.br_rec[k1] = uint8_t(o.branch);
                }
                count_events(a, o, blockIdx.x);
            }
            if (ABB && (lo || hi)) reflect_at_walls(out, lo, hi, a.phi_lo, a.phi_hi, a.phi_ref, o.dphi);
            if (inner) {
                // push streaming (periodic in y and z; periodic or reflected in x)
                char* const zp[3] = {dst + size_t(z1 == 0 ? nz - 1 : z1 - 1) * plane_bytes,
                                     dst + size_t(z1) * plane_bytes,
                                     dst + size_t(z1 == nz - 1 ? 0 : z1 + 1) * plane_bytes};
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    if (ABB && ((cx(i) > 0 && hi) || (cx(i) < 0 && lo))) {
                        // reflected at a Dirichlet plane: stays here as the opposite population
                        *reinterpret_cast<Real*>(zp[1] + size_t(opp(i)) * run_bytes + (xs + ys)) = out[i];
                    } else {
                        const uint32_t off = (cx(i) > 0 ? xp : (cx(i) < 0 ? xm : xs)) +
                                             (cy(i) > 0 ? yp : (cy(i) < 0 ? ym : ys));
                        *reinterpret_cast<Real*>(zp[cz(i) + 1] + size_t(i) * run_bytes + off) = out[i];
                    }
                }
            }
        }
        // one plane on
        up2 = up1;
        up1 = post[5];
        rest1 = post[0];
        const int u = u2, f = f1, w = w1;
        u2 = u1;
        u1 = u0;
        u0 = u;
        f1 = f0;
        f0 = f;
        w1 = w0;
        w0 = w;
        z = zn;
    }
}

// Threads of a block: 1024 columns in FP32 (four waves per SIMD, 128 VGPRs), 512 in FP64 (two
// waves, 256 VGPRs): one block per CU.
template <class Real>
constexpr int pair_threads() {
    return sizeof(Real) == 4 ? 1024 : 512;
}

// The tiling with the least estimated time, and whether it beats two single steps.
//
// Rounds of blocks over the CUs, times the planes of a sweep with its two extra ones, times
// the time of an iteration: 1.2 us + 0.075 us per 128-byte line that one run (population) of
// the block's loads and stores touches. A tile narrower than the lattice touches a line more
// on each side of a row's loads, and one more for the 10 shifted runs of 19 stored. A tensor
// field adds 6 values per node to the loads of the first step and to those of the second, a
// material table about 0.3. Measured against it over widths of 16 to 384, 1 to 28 rows and 240
// to 2500 tiles: within 16 %, and the tiling it picks is the fastest measured one or within 4 %
// of it (64^3 to 384^3 and four ragged lattices). Single steps: 6.0 TB/s and 2 us of launch.
//
// The two-step kernel is taken when it is estimated 10 % faster: at 64^3 FP32 it is not (8.6
// against 10.8 us), at 96^3 it is (24 against 18; measured 21.6 and 19.0). In FP64 on tiles of
// two or three whole rows, without a tensor field, a source per node adds 10 % and walls 13 % to an
// iteration, which such a tile does not hide: 112^3 between walls 0.93 of the speed of single steps,
// 0.84 with a source; 120^3 with both 0.96, 88^3 0.97. Tiles of more rows (33 x 175 x 173 between walls
// 45 us, single steps 72; 84 x 109 x 109 50 and 61; 80^3 with both 0.99), FP32 (1.02 and more with
// both) and tiles with halo columns (1.04 and more) have room for them.
template <class Real>
static bool pair_plan(const elbm_lattice* h, PairPlan& g) {
    const long long nx = h->cfg.nx, ny = h->cfg.ny, nz = h->cfg.nz, cus = h->cus;
    constexpr int NT = pair_threads<Real>(), SB = int(sizeof(Real)), line = 128 / SB;
    if (nx * ny * Q * SB >= (1LL << 31)) return false;
    const double t_runs = h->t_field_mode == 1 ? 6.0 : 0.0, p_runs = h->t_field_mode == 2 ? 0.3 : 0.0;
    const double s_runs = h->r_mode == 2 ? 1.0 : 0.0;
    double best = 0.0;
    auto consider = [&](long long w, int hx) {
        const long long rows = NT / (w + 2 * hx) - 2;
        if (rows < 1) return;
        const long long tx = (nx + w - 1) / w;
        long long ty = (ny + rows - 1) / rows;
        const long long by = (ny + ty - 1) / ty;
        ty = (ny + by - 1) / by;
        const double wl = double((w + line - 1) / line);
        const double lines = double(by + 2) * (wl + 2 * hx) * (1.0 + (t_runs + p_runs) / Q) + by * wl * (t_runs + p_runs) / Q +
                             by * (wl + (hx ? 10.0 / 19.0 : 0.0));
        for (int rounds = 1; rounds <= 8; ++rounds) {
            long long tz = cus * rounds / (tx * ty);
            if (tz < 1) continue;
            tz = tz < nz ? tz : nz;
            const long long len = (nz + tz - 1) / tz;
            tz = (nz + len - 1) / len;
            const double r = double((tx * ty * tz + cus - 1) / cus);
            const double us = r * double(len + 2) * (1.2 + 0.075 * lines);
            if (best == 0.0 || us < best) {
                best = us;
                g.bx = int(w);
                g.by = int(by);
                g.len = int(len);
                g.tx = int(tx);
                g.ty = int(ty);
                g.tz = int(tz);
            }
        }
    };
    consider(nx, 0);
    for (long long w = line; w < nx && w + 2 <= NT / 3; w += line) consider(w, 1);
    if (best == 0.0) return false;
    if (SB == 8 && g.tx == 1 && g.by <= 3 && t_runs == 0.0)
        best *= 1.0 + 0.1 * s_runs + (h->cfg.bc_x == ELBM_DIRICHLET ? 0.13 : 0.0);
    const double single = 2.0 * (double(h->n) * SB * (2 * Q + t_runs + p_runs) / 6.0e6 + 2.0);
    return best < 0.9 * single;
}

// Whether runs of the lattice take two steps per launch, and how.
template <class Real>
static bool plan_pair(const elbm_lattice* h, PairPlan* plan) {
    // the flags that name a single-step kernel keep it
    const int named = ELBM_FLAG_SCALAR_KERNEL | (0xF << ELBM_VECTOR_WIDTH_SHIFT);
    return Q == 19 && h->u_mode == 0 && h->cfg.root_rho < 0 && !(h->cfg.flags & named) && pair_plan<Real>(h, *plan);
}

template <class Real>
static hipError_t step_pair(const elbm_lattice* h, const void* src, void* dst, const StepPair& p, const PairPlan& plan) {
    if constexpr (Q == 19) {
        constexpr int NT = pair_threads<Real>();
        PairArgs<Real> g{};
        static_cast<PairPlan&>(g) = plan;
        StepArgs<Real> a = make_args<Real>(h, p.mult[0]);
        a.src = src;
        a.dst = dst;
        a.lam_rec = static_cast<Real*>(p.lam[0]);
        a.br_rec = p.br[0];
        g.src_mult = Real(p.mult[1]);
        g.lam_rec = static_cast<Real*>(p.lam[1]);
        g.br_rec = p.br[1];
        const unsigned tiles = unsigned(g.tx) * unsigned(g.ty) * unsigned(g.tz);
        const dim3 grid((tiles + 7) / 8 * 8), block(NT);
        if (a.tfield && a.abb) hipLaunchKernelGGL((k_step_pair<Real, true, true, NT>), grid, block, 0, h->stream, a, g);
        else if (a.tfield) hipLaunchKernelGGL((k_step_pair<Real, true, false, NT>), grid, block, 0, h->stream, a, g);
        else if (a.abb) hipLaunchKernelGGL((k_step_pair<Real, false, true, NT>), grid, block, 0, h->stream, a, g);
        else hipLaunchKernelGGL((k_step_pair<Real, false, false, NT>), grid, block, 0, h->stream, a, g);
    }
    return hipGetLastError();
}

}  // namespace elbm
