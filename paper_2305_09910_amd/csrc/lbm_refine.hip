// lbm_refine.hip -- the packet exchange of a 2:1 grid refinement between a
// coarse lattice and fine lattices below and/or above it (the paper's 2:1
// block refinement, Section 3, joined by coarse-to-fine and fine-to-coarse
// kernels, Section 5.2; the volumetric, mass-conservative scheme of Rohde,
// Kandhai, Derksen & van den Akker 2006).
//
// The interface is a plane normal to y; x and z are periodic on every level
// and a fine lattice has twice the coarse nx and nz.  Within a lattice the
// interface face is a no-slip face (the step kernels see BC_NOSLIP), so the
// packets that cross it come back into the emitting cell.  Every population
// these kernels touch has its source across the interface: its link is cut,
// and in the AA pattern a cut link's population sits in the cell's own slot
// after any number of steps.  So the kernels read and write own slots of the
// interface rows only, whatever the step parity.
//
// Populations are stored as deviations f_i - w_i; w_i = w_opposite(i), so the
// exchange works on deviations directly (a copy is exact, and an average of
// deviations is the deviation of the average).  dy is +1 for a fine lattice
// above the coarse one, -1 below.  For each crossing direction i toward the
// coarse level (c_iy = -dy) and j = opp(i), per coarse step:
//   - the packet coarse interface cell X sent toward the fine level along j
//     is f*_j(X), which the coarse step left in X's own slot i; it stays
//     there until the coarse interface row is filled at the end;
//   - after each of the two fine steps: the fine interface cells x_f with
//     x_f + c_i in X (four of them) sent f*_i(x_f), now in their own slot j;
//     1/8 of their sum is added to acc_i(X), and slot j of the same cells
//     takes X's packet f*_j(X) (the source point x_f - c_j = x_f + c_i of
//     its link lies in X);
//   - after the second fine step, slot i of X takes acc_i(X).
// So one thread per coarse interface cell does all of it with no other
// thread touching its cells' slots, and the exchange is two launches per
// coarse step: k_refine_exchange after the first fine step (first: acc = sum)
// and after the second (last: X's slot i = acc + sum).
// acc is [q][nz_c][nx_c] FP32; only the directions i with c_iy = -dy are used.
//
// Bytes per launch (FP32 storage): per coarse interface cell and crossing
// direction (5 of D3Q19, 9 of D3Q27) 4 fine slots read and written (32 B),
// the coarse slot read (4 B), and acc written (first, 4 B) or read with the
// coarse slot written (last, 8 B).
#include "lattice.h"

namespace lbm {

// the m-th direction with c_y = +1
template <int Q>
__host__ __device__ constexpr int crossing_up(int m)
{
    for (int i = 1; i < Q; ++i)
        if (cdir(i, 1) == 1 && m-- == 0) return i;
    return 0;
}

// One wavefront per workgroup: an interface is a few thousand cells, so small
// workgroups spread it over the most CUs.
constexpr int kRefineThreads = 64;

__device__ inline int wrap_int(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// What the exchange needs of a lattice: its store and the interface row's
// place in it (the whole argument block of a lattice is four times as long,
// and a kernel this short notices the loads).
struct RefineRow {
    void *pdf;
    uint32_t row0, sy;  // stored row of z = 0 in the interface plane, rows per stored plane
    int nx, nz, sx;
};

// one interface: the coarse and the fine row, the sums [q][nz_c][nx_c] FP32, and
// whether the fine lattice is above the coarse one (dy = 1)
struct RefinePair {
    RefineRow coarse, fine;
    float *acc;
    int above;
};

template <int Q>
__device__ inline uint64_t row_index(const RefineRow &r, int i, int z, int x)
{
    return ((uint64_t)(r.row0 + (uint32_t)z * r.sy) * Q + (uint32_t)i) * (uint32_t)r.sx + (uint32_t)x;
}

// The exchange after a fine step (see above): one thread per coarse interface
// cell (X, Z) and interface.  The levels form a stack, so at each depth at most
// two interfaces exchange at the same time, one on either side of the coarsest
// level; they go in one launch (blockIdx.z).
//
// Bound by latency: a launch moves little (2 MB at 256 x 128 coarse interface
// cells), so the time is that of one thread's chain.  All slots are read
// before the first is written: the lattices may be the same memory as far as
// the compiler knows, and with each direction's stores before the next one's
// loads a thread made one round trip to memory per crossing direction.
// Measured at two interfaces of 256 x 128 coarse cells, D3Q19 FP32: 6.1 us for
// both, against 7.8 us each before.
template <int Q, int SC, int SF>
__global__ void __launch_bounds__(kRefineThreads)
    k_refine_exchange(RefinePair p0, RefinePair p1, int last)
{
    using C = Store<SC>;
    using F = Store<SF>;
    const RefinePair p = blockIdx.z ? p1 : p0;
    const RefineRow c = p.coarse, f = p.fine;
    const bool below = !p.above;
    float *acc = p.acc;
    typename C::T *Ac = (typename C::T *)c.pdf;
    typename F::T *Af = (typename F::T *)f.pdf;
    const int X = blockIdx.x * kRefineThreads + threadIdx.x, Z = blockIdx.y;
    if (X >= c.nx) return;
    constexpr int NC = Q == 19 ? 5 : 9;  // crossing directions
    const size_t plane = (size_t)c.nx * c.nz, k = (size_t)Z * c.nx + X;
    // The m-th pair of opposite directions that cross: i leads from the fine
    // to the coarse level (c_iy = -dy), j back.  `up` has c_y = +1, so i = up
    // for the lattice below.
    uint64_t ci[NC], fi[NC][4];
    float v[NC], part[NC][4], before[NC];
    for_dirs<0, NC>([&](auto M) {
        constexpr int m = decltype(M)::value, up = crossing_up<Q>(m);
        const int i = below ? up : opp(up), j = below ? opp(up) : up;
        const int cx = below ? cdir(up, 0) : -cdir(up, 0), cz = below ? cdir(up, 2) : -cdir(up, 2);
        ci[m] = row_index<Q>(c, i, Z, X);
        v[m] = C::ld(Ac + ci[m]);
        before[m] = last ? acc[(size_t)i * plane + k] : 0.f;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int zf = wrap_int(2 * Z + (b >> 1) - cz, f.nz), xf = wrap_int(2 * X + (b & 1) - cx, f.nx);
            fi[m][b] = row_index<Q>(f, j, zf, xf);
            part[m][b] = F::ld(Af + fi[m][b]);
        }
    });
    for_dirs<0, NC>([&](auto M) {
        constexpr int m = decltype(M)::value, up = crossing_up<Q>(m);
        const int i = below ? up : opp(up);
        const auto packet = F::cvt(v[m]);
        float s = 0.f;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            s += part[m][b];
            Af[fi[m][b]] = packet;
        }
        const float w = 0.125f * s;
        if (last)
            Ac[ci[m]] = C::cvt(before[m] + w);
        else
            acc[(size_t)i * plane + k] = w;
    });
}

static RefineRow refine_row(const LatticeArgs &a, int y)
{
    return {a.pdf, (uint32_t)y, (uint32_t)a.sy, a.nx, a.nz, a.sx};
}

hipError_t launch_refine_exchange(const RefineLink *links, int count, int q, int last, hipStream_t s)
{
    RefinePair p[2];
    for (int k = 0; k < count; ++k) {
        const RefineLink &l = links[k];
        p[k] = {refine_row(*l.coarse, l.above ? l.coarse->ny - 1 : 0), refine_row(*l.fine, l.above ? 0 : l.fine->ny - 1),
                l.acc, l.above};
    }
    // one launch where both links have the same storage formats (two links are of
    // one depth, whose levels have the same nx and nz)
    const bool both = count == 2 && links[0].sc == links[1].sc && links[0].sf == links[1].sf;
    for (int k = 0; k < (both ? 1 : count); ++k) {
        const dim3 grid((unsigned)((p[k].coarse.nx + kRefineThreads - 1) / kRefineThreads), (unsigned)p[k].coarse.nz,
                        both ? 2 : 1);
        const hipError_t e = dispatch(q, links[k].sf, [&](auto Q, auto SF) {
            auto go = [&](auto SC) {
                k_refine_exchange<Q.value, SC.value, SF.value>
                    <<<grid, kRefineThreads, 0, s>>>(p[k], p[both ? 1 : k], last);
                return hipGetLastError();
            };
            if (links[k].sc == ST_F32) return go(std::integral_constant<int, ST_F32>{});
            if (links[k].sc == ST_F16) return go(std::integral_constant<int, ST_F16>{});
            return go(std::integral_constant<int, ST_BF16>{});
        });
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lbm
