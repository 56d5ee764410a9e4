// lbm_kernels.hip -- set-up and state kernels of every scheme (initial states,
// canonical populations, moments, totals), the launch shapes, and the choice
// between the two compilations of the AA step (step_aa.h).
#include "lattice.h"

namespace lbm {

template <bool HINT>
hipError_t step_aa(const LatticeArgs &a, const HrrArgs &h, int q, int st, int cl, int coll, int odd, hipStream_t s);
extern template hipError_t step_aa<true>(const LatticeArgs &, const HrrArgs &, int, int, int, int, int, hipStream_t);
extern template hipError_t step_aa<false>(const LatticeArgs &, const HrrArgs &, int, int, int, int, int, hipStream_t);

hipError_t launch_step(const LatticeArgs &a, const HrrArgs &h, int q, int st, int cl, int coll, int odd, hipStream_t s)
{
    return (odd & SC_CACHED) && step_without_hints(a, q, st, cl, coll)
               ? step_aa<false>(a, h, q, st, cl, coll, odd, s)
               : step_aa<true>(a, h, q, st, cl, coll, odd, s);
}


// ---------------------------------------------------------------------------
// set-up and state kernels
// ---------------------------------------------------------------------------
template <int Q>
__global__ void __launch_bounds__(LBM_LB_THREADS) k_build_mask(LatticeArgs a, const uint8_t *flags, uint32_t *mask)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z = blockIdx.z;
    if (x >= a.nx || y >= a.ny) return;
    const Geom g = make_geom(a, x, y, z);
    uint32_t m = flags[cidx(a, g)] ? SELF_SOLID : 0u;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const int dx = cdir(i, 0), dy = cdir(i, 1), dz = cdir(i, 2);
        if (!face_cut(g, dx, dy, dz) && flags[nbr(a, g, dx, dy, dz)]) m |= 1u << i;
    }
    mask[cidx(a, g)] = m;
}

// the run words after the mask (one thread per row and run of 64 cells)
__global__ void __launch_bounds__(256) k_build_mask_runs(LatticeArgs a, uint32_t *mask)
{
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t nr = mask_runs(a.nx);
    if (t >= (uint64_t)a.nrows * nr) return;
    const uint64_t row = t / nr;
    const int x0 = (int)(t - row * nr) * 64, x1 = min(x0 + 64, a.nx);
    uint32_t any = 0;
    for (int x = x0; x < x1; ++x) any |= mask[row * (uint32_t)a.nx + (uint32_t)x];
    mask[cells(a) + t] = any != 0u;
}

template <int Q, int ST>
__global__ void __launch_bounds__(LBM_LB_THREADS) k_init_eq(LatticeArgs a, SparseArgs sp, const double *rho, const double *u)
{
    using S = Store<ST>;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z = blockIdx.z;
    if (x >= a.nx || y >= a.ny) return;
    const Geom g = make_geom(a, x, y, z);
    const bool solid = a.mask && (a.mask[cidx(a, g)] & SELF_SOLID);
    if (sp.on && sp.fmap[cidx(a, g)] < 0) return;  // sparse addressing stores fluid cells only
    const double r = rho[cidx(a, g)], ux = u[cidx(a, g)], uy = u[cells(a) + cidx(a, g)], uz = u[2 * cells(a) + cidx(a, g)];
    const double usq = ux * ux + uy * uy + uz * uz;
    typename S::T *A = (typename S::T *)a.pdf;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const double cu = cdir(i, 0) * ux + cdir(i, 1) * uy + cdir(i, 2) * uz;
        const double dev = wgt<Q>(i) * ((r - 1.0) + r * (3.0 * cu + 4.5 * cu * cu - 1.5 * usq));
        A[index_t0<Q>(a, sp, g, i)] = S::cvt(solid ? 0.f : (float)dev);
    }
}

template <int Q, int ST>
__global__ void __launch_bounds__(LBM_LB_THREADS) k_set_pdfs(LatticeArgs a, SparseArgs sp, const double *f)
{
    using S = Store<ST>;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z = blockIdx.z;
    if (x >= a.nx || y >= a.ny) return;
    const Geom g = make_geom(a, x, y, z);
    if (sp.on && sp.fmap[cidx(a, g)] < 0) return;  // sparse addressing stores fluid cells only
    typename S::T *A = (typename S::T *)a.pdf;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        A[index_t0<Q>(a, sp, g, i)] = S::cvt((float)(f[(uint64_t)i * cells(a) + cidx(a, g)] - wgt<Q>(i)));
    }
}

// The state readers that a run calls one after the other read the lattice in
// alternating directions: totals and closure features from the first plane to
// the last, canonical populations and moments from the last to the first.  The
// second of two readers then starts on what the first left in the 256 MB
// last-level cache (320 MB state at 256x128x128: totals, moments, features and
// populations together 440 -> 407 us, with the shorter totals); in one
// direction each would find the cache holding the other end.  No streaming hint
// on these reads for the same reason (moments 60 -> 69 us, populations 165 -> 179
// us with it), unless the outputs alone overrun the cache (LLC_BYTES).
// STREAM: populations written with the streaming hint.
template <int Q, int ST, bool STREAM>
__global__ void __launch_bounds__(LBM_LB_THREADS) k_get_pdfs(LatticeArgs a, SparseArgs sp, int odd, double *f)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z = a.nz - 1 - (int)blockIdx.z;
    if (x >= a.nx || y >= a.ny) return;
    const Geom g = make_geom(a, x, y, z);
    const uint32_t m = a.mask ? a.mask[cidx(a, g)] : 0u;
    float d[Q];
    if (m & SELF_SOLID) {
#pragma unroll
        for (int i = 0; i < Q; ++i) d[i] = 0.f;
    } else {
        load_state<Q, ST>(a, sp, g, m, odd, d);
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) st_pop<STREAM>(f + (uint64_t)i * cells(a) + cidx(a, g), wgt<Q>(i) + (double)d[i]);
}

template <int Q, int ST>
__global__ void __launch_bounds__(256) k_gather(LatticeArgs a, SparseArgs sp, int odd, const int64_t *cells, int64_t ncell,
                                                double *out)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= ncell) return;
    const int64_t c = cells[r];
    if (c < 0 || c >= (int64_t)lbm::cells(a)) {
#pragma unroll
        for (int i = 0; i < Q; ++i) out[r * Q + i] = __builtin_nan("");
        return;
    }
    const int x = (int)(c % a.nx), y = (int)((c / a.nx) % a.ny), z = (int)(c / ((int64_t)a.nx * a.ny));
    const Geom g = make_geom(a, x, y, z);
    const uint32_t m = a.mask ? a.mask[cidx(a, g)] : 0u;
    float d[Q];
    if (m & SELF_SOLID) {
#pragma unroll
        for (int i = 0; i < Q; ++i) d[i] = 0.f;
    } else {
        load_state<Q, ST>(a, sp, g, m, odd, d);
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) out[r * Q + i] = wgt<Q>(i) + (double)d[i];
}

template <int Q, int ST, bool STREAM>
__global__ void __launch_bounds__(LBM_LB_THREADS) k_moments(LatticeArgs a, SparseArgs sp, int odd, float *rho, float *u)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z = a.nz - 1 - (int)blockIdx.z;
    if (x >= a.nx || y >= a.ny) return;
    const Geom g = make_geom(a, x, y, z);
    const uint32_t m = a.mask ? a.mask[cidx(a, g)] : 0u;
    auto put = [&](float r, float ux, float uy, float uz) {
        const uint64_t n = cells(a), c = cidx(a, g);
        st_pop<STREAM>(rho + c, r);
        st_pop<STREAM>(u + c, ux);
        st_pop<STREAM>(u + n + c, uy);
        st_pop<STREAM>(u + 2 * n + c, uz);
    };
    if (m & SELF_SOLID) {
        put(1.f, 0.f, 0.f, 0.f);
        return;
    }
    float d[Q];
    load_state<Q, ST, STREAM>(a, sp, g, m, odd, d);
    float drho;
    const Macro M = moments<Q>(a, d, drho);
    put(M.rho, M.ux, M.uy, M.uz);
}

// Deterministic FP64 totals: each block owns a fixed slice of cells and
// reduces it in a fixed order (lanes, then wavefronts); a second kernel sums
// the block partials in a fixed order.
constexpr int TOT_BLOCKS = 1024;

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sums over the workgroup's threads of acc, component by component: lanes, then
// wavefronts in order.  red: one row of components per wavefront.
template <int WAVES>
__device__ inline void block_sums(const double (&acc)[5], double (*red)[5], double *out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const double v = wave_sum(acc[k]);
        if (lane == 0) red[wave][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) v += red[w][threadIdx.x];
        out[threadIdx.x] = v;
    }
}

// Bound by memory (q populations read per cell).  WIDE: the cell index needs
// 64 bits; below 2^32 cells it is split with 32-bit divisions, since the three
// 64-bit ones per cell cost more than the loads could hide.  512 threads, so
// that the 1024 blocks are the 32 wavefronts a CU holds: 256x128x128 FP32 52 us
// (6.1 TB/s) on a clean cache; 88 behind 256 MB of dirty lines, where 256 threads
// and 64-bit divisions took 96.
constexpr int TOT_THREADS = 512;

template <int Q, int ST, bool WIDE>
__global__ void __launch_bounds__(TOT_THREADS) k_totals(LatticeArgs a, SparseArgs sp, int odd, double *partial)
{
    using I = std::conditional_t<WIDE, uint64_t, uint32_t>;
    double acc[5] = {0, 0, 0, 0, 0};
    const uint64_t n = cells(a);
    const uint64_t per_block = (n + TOT_BLOCKS - 1) / TOT_BLOCKS;
    const uint64_t lo = (uint64_t)blockIdx.x * per_block;
    const uint64_t hi = lo + per_block < n ? lo + per_block : n;
    for (uint64_t c = lo + threadIdx.x; c < hi; c += TOT_THREADS) {
        const I row = (I)c / (I)(uint32_t)a.nx;
        const int x = (int)((I)c - row * (I)(uint32_t)a.nx);
        const int z = (int)((uint32_t)row / (uint32_t)a.ny);
        const int y = (int)((uint32_t)row - (uint32_t)z * (uint32_t)a.ny);
        const Geom g = make_geom(a, x, y, z);
        const uint32_t m = a.mask ? a.mask[cidx(a, g)] : 0u;
        if (m & SELF_SOLID) continue;
        float d[Q];
        load_state<Q, ST>(a, sp, g, m, odd, d);
        float s = 0.f, jx = 0.f, jy = 0.f, jz = 0.f;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            s += d[i];
            jx += cdir(i, 0) * d[i];
            jy += cdir(i, 1) * d[i];
            jz += cdir(i, 2) * d[i];
        }
        acc[0] += (double)s;
        acc[1] += (double)jx;
        acc[2] += (double)jy;
        acc[3] += (double)jz;
        acc[4] += isfinite(s) ? 0.0 : 1.0;
    }
    __shared__ double red[TOT_THREADS / 64][5];
    block_sums<TOT_THREADS / 64>(acc, red, partial + blockIdx.x * 5);
}

// One workgroup; thread t sums the partials of blocks t, t + 256, ... (a single
// thread per component over all of them is a chain of 1024 loads: 25 us, now 6).
__global__ void __launch_bounds__(256) k_totals_final(const double *partial, double *out)
{
    double acc[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < TOT_BLOCKS / 256; ++b)
#pragma unroll
        for (int k = 0; k < 5; ++k) acc[k] += partial[(b * 256 + threadIdx.x) * 5 + k];
    __shared__ double red[4][5];
    block_sums<4>(acc, red, out);
}

// Copy: one 16-byte vector per thread, loaded and stored with the
// nontemporal hint (each line is touched once).  Of the shapes measured on
// MI355X (1 or 4 vectors per thread, with and without the hint) this one
// moves the most bytes per second.
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(256) k_copy(const f32x4 *__restrict__ src, f32x4 *__restrict__ dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
Launch lattice_launch(const LatticeArgs &a, int st, int cl, int coll, bool cached)
{
    // A workgroup is BX cells along x (a row segment) times BY rows.  Three
    // things pull at it: the +-1 shifted accesses of a step share a line at
    // each seam between the workgroups of a row, which different XCDs then
    // fetch twice; lanes past the end of the row idle; and kernels with many
    // registers (solids, MRT) keep fewer wavefronts resident when workgroups
    // are large, above all with five to seven wavefronts, which four SIMDs of
    // four each cannot share out.  All figures: us per step.
    auto shape = [&](int bx, int by) {
        Launch L;
        L.block = dim3(bx, by, 1);
        L.grid = dim3((a.nx + bx - 1) / bx, (a.ny + by - 1) / by, a.nz);
        return L;
    };
    const bool light = coll == COLL_TRT && cl != CL_MLP && !a.mask;
    // Rows of whole 512-cell segments: one workgroup each for the light
    // kernels (TRT 193, 195 with 256), 256 cells for the others (512x128x128:
    // MRT 202 / 213, HRR 255 / 264, D3Q27 with solids 360 / 371, learned
    // closure 260 / 266).
    if (a.nx % LBM_WIDE == 0) return shape(light || a.et ? LBM_WIDE : 256, 1);
    // Rows that 64 or 128 do not divide.  Not with the learned closure, bound
    // by its vector instructions, where idle lanes and the table per workgroup
    // cost more than seams (130: 59 in segments of 64, 66 in whole rows).
    // Measured at 26 row lengths from 70 to 1000, with 0.7 M and 6 M cells (16-bit
    // 2.5 M as well), for 25 forms; quoted is the time over that of segments of 64 x 4, or 32 x 8 for
    // multiples of 32 (geometric mean, largest).
    if (a.nx > 64 && a.nx % 128 != 0 && cl != CL_MLP) {
        const bool f32 = st == ST_F32;
        auto up = [&](int w) { return (a.nx + w - 1) / w * w; };
        const int row64 = up(64), half = ((a.nx + 1) / 2 + 31) / 32 * 32;
        // 16-bit lattices that are no larger than the L2s prefer other shapes
        const bool small = cells(a) < (1u << 20);
        // the widest segment that idles no more lanes than 64 x 4 does: what
        // kernels with many registers bear (beyond 256 cells, with solids FP32
        // 0.98, 1.05; 16-bit 0.95, 1.05, where whole or half rows are 0.98, 1.32)
        auto widest = [&] {
            if (f32 && up(256) == row64) return shape(256, 1);
            return up(128) == row64 ? shape(128, 2) : shape(64, 4);
        };
        if (a.et && a.mask && (f32 || (row64 == 128 && !cached))) {
            // whole rows where the lattice stays in the cache (0.97, 1.00; not
            // multiples of 32: 160 1.04), nothing to gain elsewhere
            if (cached && row64 == 128) return shape(128, 2);
            if (cached && row64 <= 256 && a.nx % 32 != 0) return shape(row64, 1);
        } else if (row64 == 128) {
            return shape(128, 2);  // 0.91, 1.00
        } else if (a.mask) {
            // whole rows (FP32 0.92, 1.00 beyond the cache; in it 0.98, without
            // multiples of 32, where 160 is 1.05; 16-bit Esoteric Twist in the
            // cache 0.91, 1.02); 300: FP32 beyond the cache 0.98, 16-bit Esoteric
            // Twist in it 0.97 (AA 1.02), its half rows beyond 320 cells 0.88; 444:
            // FP32 beyond the cache 0.95
            if (row64 <= 256 && (f32 || (a.et && cached))) {
                if (!f32 || !cached || a.nx % 32 != 0) return shape(row64, 1);
            } else {
                if (row64 == 320 && (f32 ? !cached : cached && a.et)) return shape(128, 2);
                if (!f32 && cached && a.et && row64 > 320 && a.nx < LBM_WIDE) return shape(half, 1);
                if (f32 && !cached && coll == COLL_TRT && row64 == 448 && 2 * half - a.nx <= a.nx / 10) return shape(half, 1);
                return widest();
            }
        } else if (row64 <= 256) {
            return shape(row64, 1);  // one workgroup per row: 0.87, 1.05
        } else if (a.et && !f32 && (!cached || (coll == COLL_MRT && !small))) {
            return widest();  // 0.95, 1.01; whole rows 1.03, 1.16
        } else if (a.nx > LBM_WIDE) {
            // longer than a workgroup: 256 cells (16-bit 0.87, 1.05), FP32 320
            // where that idles fewer lanes (0.90, 0.98); MRT and HRR 128 x 2 (0.94,
            // 1.06), FP32 where 256 fit as well (672 HRR 304 us, 340 with 128 x 2)
            if (light && f32 && up(320) < up(256)) return shape(320, 1);
            return light || a.et || (f32 && up(256) - a.nx <= a.nx / 7) ? shape(256, 1) : shape(128, 2);
        } else if (a.et || (light && (!f32 || row64 == 320))) {
            return shape(row64, 1);  // 0.89, 1.06
        } else if (!f32) {
            // 300: 0.94 to 0.99, small 1.04; the others 0.93, 1.02
            if (row64 == 320 && !small) return coll == COLL_HRR ? shape(320, 1) : shape(128, 2);
            return widest();
        } else if (row64 == 320) {
            return coll == COLL_HRR && cached ? shape(320, 1) : shape(128, 2);  // 0.98, 1.00
        } else {
            // half rows (0.91, 0.99); MRT and HRR beyond the cache where few
            // lanes idle (400, with 48 of 448: 1.02, 424: 0.90)
            return light || cached || 2 * half - a.nx <= a.nx / 10 ? shape(half, 1) : widest();
        }
    }
    // LBM_BLOCK threads, BX the largest power of two up to LBM_BLOCK that
    // divides nx, else 64 with a masked tail
    int bx = LBM_BLOCK;
    while (bx > 32 && a.nx % bx != 0) bx >>= 1;
    if (a.nx % bx != 0) bx = 64;
    if (bx > a.nx) bx = a.nx <= 32 ? 32 : 64;
    return shape(bx, LBM_BLOCK / bx);
}

hipError_t launch_build_mask(const LatticeArgs &a, int q, const uint8_t *flags, uint32_t *mask, hipStream_t s)
{
    const Launch L = lattice_launch(a, ST_F32);
    if (q == 19)
        k_build_mask<19><<<L.grid, L.block, 0, s>>>(a, flags, mask);
    else
        k_build_mask<27><<<L.grid, L.block, 0, s>>>(a, flags, mask);
    const uint64_t nruns = (uint64_t)a.nrows * mask_runs(a.nx);
    k_build_mask_runs<<<(unsigned)((nruns + 255) / 256), 256, 0, s>>>(a, mask);
    return hipGetLastError();
}

// Last-level cache.  Outputs that are larger are written with the streaming hint:
// nobody finds them in the cache, and what they leave there dirty is written back
// during the next kernel (and, with moments, their populations are then read with
// it too).  Moments of 512x256x256 FP32 with the box filter behind them: 580 + 125
// us, now 505 + 109; totals after the populations of 256x128x128 (637 MB) were
// written: 88 us, now 52.
constexpr uint64_t LLC_BYTES = 256ull << 20;

hipError_t launch_init_eq(const LatticeArgs &a, const SparseArgs &sp, int q, int st, const double *rho,
                          const double *u, hipStream_t s)
{
    const Launch L = lattice_launch(a, st);
    return dispatch(q, st, [&](auto Q, auto ST) {
        k_init_eq<Q.value, ST.value><<<L.grid, L.block, 0, s>>>(a, sp, rho, u);
        return hipGetLastError();
    });
}

hipError_t launch_set_pdfs(const LatticeArgs &a, const SparseArgs &sp, int q, int st, const double *f, hipStream_t s)
{
    const Launch L = lattice_launch(a, st);
    return dispatch(q, st, [&](auto Q, auto ST) {
        k_set_pdfs<Q.value, ST.value><<<L.grid, L.block, 0, s>>>(a, sp, f);
        return hipGetLastError();
    });
}

hipError_t launch_get_pdfs(const LatticeArgs &a, const SparseArgs &sp, int q, int st, int odd, double *f,
                           hipStream_t s)
{
    const Launch L = lattice_launch(a, st);
    return dispatch(q, st, [&](auto Q, auto ST) {
        if (cells(a) * Q.value * 8 >= LLC_BYTES)
            k_get_pdfs<Q.value, ST.value, true><<<L.grid, L.block, 0, s>>>(a, sp, odd, f);
        else
            k_get_pdfs<Q.value, ST.value, false><<<L.grid, L.block, 0, s>>>(a, sp, odd, f);
        return hipGetLastError();
    });
}

hipError_t launch_gather(const LatticeArgs &a, const SparseArgs &sp, int q, int st, int odd, const int64_t *cells,
                         int64_t ncell, double *out, hipStream_t s)
{
    if (ncell <= 0) return hipSuccess;
    const dim3 grid((unsigned)((ncell + 255) / 256)), block(256);
    return dispatch(q, st, [&](auto Q, auto ST) {
        k_gather<Q.value, ST.value><<<grid, block, 0, s>>>(a, sp, odd, cells, ncell, out);
        return hipGetLastError();
    });
}

hipError_t launch_moments(const LatticeArgs &a, const SparseArgs &sp, int q, int st, int odd, float *rho, float *u,
                          hipStream_t s)
{
    const Launch L = lattice_launch(a, st);
    return dispatch(q, st, [&](auto Q, auto ST) {
        if (cells(a) * 16 >= LLC_BYTES)
            k_moments<Q.value, ST.value, true><<<L.grid, L.block, 0, s>>>(a, sp, odd, rho, u);
        else
            k_moments<Q.value, ST.value, false><<<L.grid, L.block, 0, s>>>(a, sp, odd, rho, u);
        return hipGetLastError();
    });
}

int totals_blocks() { return TOT_BLOCKS; }

hipError_t launch_totals(const LatticeArgs &a, const SparseArgs &sp, int q, int st, int odd, double *partial,
                         double *final_out, hipStream_t s)
{
    hipError_t e = dispatch(q, st, [&](auto Q, auto ST) {
        if (cells(a) >> 32)
            k_totals<Q.value, ST.value, true><<<TOT_BLOCKS, TOT_THREADS, 0, s>>>(a, sp, odd, partial);
        else
            k_totals<Q.value, ST.value, false><<<TOT_BLOCKS, TOT_THREADS, 0, s>>>(a, sp, odd, partial);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    k_totals_final<<<1, 256, 0, s>>>(partial, final_out);
    return hipGetLastError();
}

__global__ void __launch_bounds__(64) k_build_mlp_table(const float *P, uint32_t *T)
{
    build_table_lane(P, threadIdx.x, T);
}

hipError_t launch_build_mlp_table(const float *params, uint32_t *table, hipStream_t s)
{
    k_build_mlp_table<<<1, 64, 0, s>>>(params, table);
    return hipGetLastError();
}

hipError_t launch_copy(const void *src, void *dst, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16;
    const size_t blocks = (n + 255) / 256;
    if (n == 0) return hipSuccess;
    if (blocks > 0x7fffffffu) return hipErrorInvalidValue;
    k_copy<<<(unsigned)blocks, 256, 0, s>>>((const f32x4 *)src, (f32x4 *)dst, n);
    return hipGetLastError();
}

}  // namespace lbm
