// Host program around the library's launch rules: reads one lattice per line of standard input and
// prints the launch shape that the rules choose for it, without a GPU (256 compute units).
//   rows <f64|f32|b16> <flags> <u_mode> <root> <nx> <ny> <nz>  ->  rows pitch threads grid.x grid.y grid.z covered
//   vec <f64|f32|b16> <flags> <u_mode> <t_mode> <nx> <ny> <nz>  ->  V W waves of the row-vector kernel
//   pair <f64|f32> <flags> <walls> <t_mode + 4 r_mode> <nx> <ny> <nz>  ->  taken bx by len tx ty tz
// "covered" is 1 if every node of a plane has exactly one thread, by the arithmetic of node_of.
#include <cstdio>
#include <cstring>
#include <vector>

#include "pair_kernel.h"

using namespace elbm;

static bool covered(const RowGrid& g, int nx, int ny) {
    std::vector<int> seen(size_t(nx) * ny, 0);
    const float inv_pitch = 1.0f / float(g.pitch);
    for (unsigned by = 0; by < g.grid.y; ++by)
        for (unsigned bx = 0; bx < g.grid.x; ++bx)
            for (unsigned th = 0; th < g.block.x; ++th) {
                const int t = int(bx * g.block.x + th);
                const int q = g.rows == 1 ? 0 : int((float(t) + 0.5f) * inv_pitch);
                const int x = t - q * g.pitch, y = int(by) * g.rows + q;
                if (x < nx && q < g.rows && y < ny) {
                    if (x < 0) return false;
                    ++seen[size_t(y) * nx + x];
                }
            }
    for (int s : seen)
        if (s != 1) return false;
    return true;
}

template <class ST>
static VecChoice choice(const elbm_lattice* h) {
    return h->u_mode == 0 ? choose_vec<ST, 0>(h) : h->u_mode == 1 ? choose_vec<ST, 1>(h) : choose_vec<ST, 2>(h);
}

int main() {
    char what[16], form[16];
    int flags, u_mode, mode, nx, ny, nz;
    while (scanf("%15s %15s %d %d %d %d %d %d", what, form, &flags, &u_mode, &mode, &nx, &ny, &nz) == 8) {
        const bool rows = !strcmp(what, "rows"), f64 = !strcmp(form, "f64"), f32 = !strcmp(form, "f32");
        elbm_lattice h{};
        h.cfg.nx = nx;
        h.cfg.ny = ny;
        h.cfg.nz = nz;
        h.cfg.flags = flags;
        h.cfg.root_rho = rows && mode ? 0.0 : -1.0;
        h.n = int64_t(nx) * ny * nz;
        const bool pair = !strcmp(what, "pair");
        h.u_mode = pair ? 0 : u_mode;
        h.cfg.bc_x = pair && u_mode ? ELBM_DIRICHLET : ELBM_PERIODIC;
        h.t_field_mode = rows ? 0 : mode & 3;
        h.r_mode = pair ? mode >> 2 : 0;
        h.cus = 256;
        if (pair) {
            PairPlan p;
            const bool taken = f64 ? plan_pair<double>(&h, &p) : plan_pair<float>(&h, &p);
            printf("%d %d %d %d %d %d %d\n", int(taken), p.bx, p.by, p.len, p.tx, p.ty, p.tz);
        } else if (rows) {
            const RowGrid g = grid_for(&h, f64 ? row_rule<double>(&h) : f32 ? row_rule<float>(&h) : row_rule<_Float16>(&h));
            printf("%d %d %u %u %u %u %d\n", g.rows, g.pitch, g.block.x, g.grid.x, g.grid.y, g.grid.z,
                   int(covered(g, nx, ny)));
        } else {
            const VecChoice c = f64 ? choice<double>(&h) : f32 ? choice<float>(&h) : choice<_Float16>(&h);
            printf("%d %d %d\n", c.V, c.W, c.waves);
        }
    }
    return 0;
}
