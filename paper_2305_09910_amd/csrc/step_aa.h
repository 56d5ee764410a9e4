// step_aa.h -- fused in-place stream-collide kernel of the AA pattern for gfx950.
//
// Compiled twice: lbm_step.hip with the streaming hints, lbm_step_cached.hip
// without them (SC_CACHED).
//
// One population set lives in HBM as deviations d_i = f_i - w_i, in rows of
// q direction segments [z][y][q][x]: structure of arrays within each row,
// so every wavefront access to one direction is contiguous, with the q
// segments of a row kept together in one block.  Streaming (the paper's Eq. (2)) and collision
// (Eq. (1), read as TRT with Guo forcing) are fused into one kernel per time
// step with the AA access pattern, an in-place scheme of the same family as
// the Esoteric Twist the paper's LAGOON runs use (Section 5.2):
//
//   even step: cell x reads d_i from its own slot i, collides, and writes
//              the post-collision value of direction i into its own slot
//              opposite(i);
//   odd step:  cell x reads d_i from slot opposite(i) of cell x - c_i,
//              collides, and writes direction i into slot i of cell x + c_i.
//
// After an odd step the array holds the canonical post-stream state in the
// natural slots; after an even step the post-collision values sit in
// swapped slots of the emitting cell.  In both steps the set of slots a cell
// reads equals the set it writes, so the update is race free in place.
//
// Walls: a link cut by a wall face or a solid neighbour is closed at write
// time inside the emitting cell: the (possibly modified) value goes into
// the cell's own slot opposite(i), which is exactly where that cell reads
// its returning population next step.  Velocity and pressure faces modify
// the value there with the emitting cell's own velocity.
//
// The kernel is bound by HBM bandwidth (every population is read once and
// written once per step); no matrix cores are used here.  All arithmetic is
// FP32 on deviations, which keeps small forcing increments above the FP32
// rounding of w_i.
#pragma once

#include "lattice.h"

namespace lbm {

// ---------------------------------------------------------------------------
// the fused stream-collide kernel
// ---------------------------------------------------------------------------
// flags: bit 0 the step parity (1: odd step); bit 1 (SC_SOLID_ODD): on the
// odd step solid lanes write zero deviations into their own slots (see
// below); bit 2
// (SC_MASK_RUNS): mask words only in runs that touch a solid
//
// ROW: every wavefront of the launch lies in one row of cells, so the row and
// all that follows from it (the neighbour rows' addresses, the y and z face
// tests) is the same for its lanes and is kept in scalar registers.  Used with
// the learned closure, whose kernel is bound by its vector instructions; the
// bandwidth-bound kernels lose more by the changed register budget than the
// address arithmetic costs them.
// PAIRWISE: SC_PAIRWISE is set (TRT, FP32 storage).
template <int Q, int ST, int CL, bool MASK, int COLL, bool ROW, bool PAIRWISE, bool HINT>
__global__ void __launch_bounds__(LBM_LB_THREADS, LBM_MIN_WAVES)
    k_stream_collide(LatticeArgs a, int flags, [[maybe_unused]] HrrArgs h)
{
    using S = Store<ST>;
    const int odd = flags & 1;
    constexpr bool kUnified =
        LBM_UNIFIED == 1 || (LBM_UNIFIED == 2 && (MASK || ST == ST_F32) && CL != CL_MLP);
    const dim3 block = step_block(!HINT && (flags & SC_SLABS));
    const int x = block.x * blockDim.x + threadIdx.x;
    int y = block.y * blockDim.y + threadIdx.y;
    if constexpr (ROW) y = __builtin_amdgcn_readfirstlane(y);
    const int z = block.z;
    bool active = x < a.nx && y < a.ny;
    // The learned closure runs on the matrix cores across the whole
    // wavefront, so with it every lane stays to the end; otherwise lanes
    // outside the domain or on solid cells leave at once.
    if constexpr (CL != CL_MLP) {
        if (!active) return;
    }
    [[maybe_unused]] const uint32_t *tab = nullptr;
    [[maybe_unused]] MlpTable table;
    if constexpr (CL == CL_MLP) table.fetch(a);
    // Solid cells on the even step: their lanes load and store their own
    // slots unchanged, in the same instructions as the fluid lanes of the
    // wavefront.  No other cell touches a solid cell's slots, so this is race
    // free, and every cache line the wavefront writes is then written whole;
    // lanes that skip would leave holes in the lines along sphere surfaces,
    // and partially written lines cost ~20% of the even step's time on the
    // 384^3 obstacle flow.  On the odd step no fluid cell reads or writes a
    // solid cell's slots either (links into a solid are cut, and cut links
    // use the fluid cell's own slots), so with SC_SOLID_ODD a solid lane
    // writes zero deviations into its own slots on the odd step, filling the
    // holes that solid cells leave in the lines its row's neighbours write
    // (no cell ever reads a solid cell's slots, and the state readers report
    // solid cells as at rest).  That costs the solid cells' store bytes: it
    // pays on sparse solids (384^3 obstacle flow, 10% solid: odd step -4%
    // against no fill) and not on dense ones (70%-solid porous medium), so
    // the host sets the flag by the solid fraction.
    constexpr bool kKeepSolid = MASK && kUnified && CL != CL_MLP;
    bool keep = false;
    const Geom g = make_geom(a, active ? x : 0, y < a.ny ? y : 0, z);
    uint32_t m = 0;
    if constexpr (MASK) {
        // with SC_MASK_RUNS the cell's mask word only where its run of 64
        // cells touches a solid
        if (active && (!(flags & SC_MASK_RUNS) || a.mask[cells(a) + (uint64_t)g.frow * mask_runs(a.nx) + ((uint32_t)x >> 6)]))
            m = a.mask[cidx(a, g)];
        if (m & SELF_SOLID) {
            if constexpr (kKeepSolid) {
                if (odd) {
                    if (flags & SC_SOLID_ODD) {
                        // no cell reads a solid cell's slots (state readers
                        // report solids as at rest), so zero deviations do
                        typename S::T *A = (typename S::T *)a.pdf;
#pragma unroll
                        for (int i = 0; i < Q; ++i) S::st(A + pidx<Q>(a, i, g.row, g.x), 0.0f);
                    }
                    return;
                }
                keep = true;
            } else {
                if constexpr (CL != CL_MLP) return;
                active = false;
            }
        }
    }
    // no link of this cell crosses a non-periodic face: the common case,
    // without face logic (solid neighbours are handled inside the plain path)
    const bool plain = !(g.cxl || g.cxh || g.cyl || g.cyh || g.czl || g.czh);
    float d[Q];
    if (CL == CL_MLP && !active) {
#pragma unroll
        for (int i = 0; i < Q; ++i) d[i] = 0.f;
    } else if (kUnified) {
        load_all<Q, ST, MASK, HINT>(a, g, m, odd, d);
    } else if (plain) {
        load_plain<Q, ST, MASK, HINT>(a, g, m, odd, d);
    } else {
        load_canonical<Q, ST>(a, g, m, odd, d);
    }
    if constexpr (CL == CL_MLP) {
        // the per-lane operand table of the network, staged once per workgroup
        __shared__ __align__(16) uint32_t tab_lds[TAB_WORDS * 64];
        table.put(tab_lds);
        __syncthreads();
        tab = tab_lds;
    }

    Macro M;
    if constexpr (COLL == COLL_TRT) {
        M = trt_cell<Q, ST, CL, PAIRWISE>(a, tab, d, active, keep);
    } else {
        float drho, wp, wm;
        M = moments<Q>(a, d, drho);
        closure_rates<Q, CL>(a, tab, d, drho, M, active, wp, wm);
        if constexpr (COLL == COLL_MRT) {
            mrt_collide<Q>(a, d, drho, M, wp, keep);
        } else {
            // finite-difference gradient of the previous step's velocities; this
            // step's velocities go to the other field (solid cells keep zeros)
            float G[3][3] = {};
            if (!keep) {
                fd_gradient<Q>(a, h, g, m, G);
                h.unext[cidx(a, g)] = M.ux;
                h.unext[cells(a) + cidx(a, g)] = M.uy;
                h.unext[2 * cells(a) + cidx(a, g)] = M.uz;
            }
            hrr_collide<Q>(a, h.sigma, G, d, drho, M, keep);
        }
    }
    if constexpr (CL == CL_MLP) {
        if (!active) return;
    }

    typename S::T *A = (typename S::T *)a.pdf;
    if (kUnified) {
        store_all<Q, ST, MASK, COLL != COLL_TRT, HINT>(a, g, m, odd, d, M, keep);
    } else if (plain) {
        store_plain<Q, ST, MASK, HINT>(a, g, m, odd, d);
    } else if (!odd) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            float v = d[i];
            if (a.any_vp) {
                const int dx = cdir(i, 0), dy = cdir(i, 1), dz = cdir(i, 2);
                if (face_cut(g, dx, dy, dz)) v = wall_value<Q>(a, deciding_face(a, g, dx, dy, dz), i, v, M);
            }
            S::st(A + pidx<Q>(a, opp(i), g.row, g.x), v);
        }
    } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int dx = cdir(i, 0), dy = cdir(i, 1), dz = cdir(i, 2);
            const bool fcut = face_cut(g, dx, dy, dz);
            const bool cut = fcut || ((m >> i) & 1u);
            float v = d[i];
            if (a.any_vp && fcut) v = wall_value<Q>(a, deciding_face(a, g, dx, dy, dz), i, v, M);
            const uint64_t own = pidx<Q>(a, opp(i), g.row, g.x);
            const uint64_t dst = pidx_nbr<Q>(a, g, i, dx, dy, dz);
            S::st(A + (cut ? own : dst), v);
        }
    }
}

// Even step of 16-bit storage without a solid mask, two neighbouring cells
// per thread.  A wavefront access of one 16-bit value per lane covers a
// single 128-byte line, and such accesses reach only ~93% of the bandwidth of
// 4-byte ones; here each lane loads and stores one aligned 32-bit word per
// direction (cells x0 and x0 + 1, x0 even), so a wavefront moves two lines
// per instruction as the FP32 kernel does (even step 2-6% faster, the whole
// step 2-4% on the FP16/BF16 channels).  The per-cell arithmetic is the
// step kernel's: moments, closure rates, collision, wall values of cut links.
// Needs nx a multiple of 128 (whole wavefronts of pairs; rows start on lines).
#ifndef LBM_PAIR16
#define LBM_PAIR16 1
#endif

template <int Q, int ST, int CL, int COLL, bool HINT>
__global__ void __launch_bounds__(256, LBM_MIN_WAVES) k_even_pair16(LatticeArgs a)
{
    using S = Store<ST>;
    const int x0 = 2 * (int)(blockIdx.x * blockDim.x + threadIdx.x);
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z = blockIdx.z;
    if (x0 >= a.nx || y >= a.ny) return;
    const Geom g[2] = {make_geom(a, x0, y, z), make_geom(a, x0 + 1, y, z)};
    // the row's direction segments start on 128-byte lines and x0 is even:
    // every word below is 4-byte aligned
    uint32_t *R = (uint32_t *)((typename S::T *)a.pdf + pidx<Q>(a, 0, g[0].row, x0));
    const uint32_t pitch = (uint32_t)a.sx / 2u;
    float d[2][Q];
    for_dirs<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        const uint32_t w = ld_pop<HINT>(R + (uint64_t)i * pitch);
        d[0][i] = S::from_bits(w);
        d[1][i] = S::from_bits(w >> 16);
    });
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        Macro M;
        if constexpr (COLL == COLL_TRT) {
            M = trt_cell<Q, ST, CL>(a, nullptr, d[c], true, false);
        } else {
            float drho, wp, wm;
            M = moments<Q>(a, d[c], drho);
            closure_rates<Q, CL>(a, nullptr, d[c], drho, M, true, wp, wm);
            mrt_collide<Q>(a, d[c], drho, M, wp);
        }
        if (a.any_vp) {
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                const int dx = cdir(i, 0), dy = cdir(i, 1), dz = cdir(i, 2);
                if (face_cut(g[c], dx, dy, dz))
                    d[c][i] = wall_value<Q>(a, deciding_face(a, g[c], dx, dy, dz), i, d[c][i], M);
            }
        }
    }
    // direction i goes into slot opposite(i) of the same cell
    for_dirs<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        const uint32_t w = S::to_bits(d[0][i]) | (S::to_bits(d[1][i]) << 16);
        st_pop<HINT>(R + (uint64_t)opp(i) * pitch, w);
    });
}

// LDS to be set aside (and not used) by each workgroup so that at most `waves`
// wavefronts run on a CU: the least that keeps one workgroup more from fitting
// the 160 KB.
inline unsigned lds_for_waves(const Launch &L, unsigned waves)
{
    const unsigned per = (L.block.x * L.block.y + 63) / 64, groups = waves / per;
    return 160 * 1024 / (groups + 1) + 1280;
}

template <int Q, int ST, int CL, bool MASK, int COLL, bool HINT>
static void launch_sc(const LatticeArgs &a, const HrrArgs &h, int odd, const Launch &L, hipStream_t s)
{
    if (!HINT && step_in_slabs(a, Q, ST, L.grid)) odd |= SC_SLABS;
    if constexpr (CL == CL_MLP) {
        if (L.block.x % 64 == 0) {
            k_stream_collide<Q, ST, CL, MASK, COLL, true, false, HINT><<<L.grid, L.block, 0, s>>>(a, odd, h);
            return;
        }
    }
    if constexpr (ST == ST_F32 && CL != CL_MLP && COLL == COLL_TRT) {
        if (odd & SC_PAIRWISE) {
            k_stream_collide<Q, ST, CL, MASK, COLL, false, true, HINT><<<L.grid, L.block, 0, s>>>(a, odd, h);
            return;
        }
    }
    // The registers of the two-vector collision allow 24 wavefronts per CU; beyond
    // the cache the steps run better with fewer, as the pairwise form had them.  us
    // per step without / with the limit: 512-cell rows 512x256x256 867 / 859, D3Q27
    // 1318 / 1311, 1024x128x128 421 / 416, D3Q27 637 / 624; with solids (D3Q19,
    // 20 instead of 24) 90x299x298 293 / 280, 246x181x180 256 / 246, 512x125x125 239 / 240.
    unsigned lds = 0;
    if constexpr (ST == ST_F32 && CL != CL_MLP && COLL == COLL_TRT && HINT) {
        if (MASK && Q == 19 && CL == CL_NONE) lds = lds_for_waves(L, 20);
        if (!MASK && L.block.x == LBM_WIDE) lds = lds_for_waves(L, 16);
    }
    k_stream_collide<Q, ST, CL, MASK, COLL, false, false, HINT><<<L.grid, L.block, lds, s>>>(a, odd, h);
}

template <int Q, int ST, int COLL, bool HINT>
static void step_coll(const LatticeArgs &a, const HrrArgs &h, int cl, bool mk, int odd, const Launch &L,
                      hipStream_t s)
{
    if (cl == CL_NONE) {
        if (mk)
            launch_sc<Q, ST, CL_NONE, true, COLL, HINT>(a, h, odd, L, s);
        else
            launch_sc<Q, ST, CL_NONE, false, COLL, HINT>(a, h, odd, L, s);
    } else {
        if (mk)
            launch_sc<Q, ST, CL_SMAG, true, COLL, HINT>(a, h, odd, L, s);
        else
            launch_sc<Q, ST, CL_SMAG, false, COLL, HINT>(a, h, odd, L, s);
    }
}

// Launch of the paired even step: nx / 2 threads per row, rows of whole
// wavefronts (nx a multiple of 128).
template <int Q, int ST, bool HINT>
static bool even_pair16(const LatticeArgs &a, int cl, int coll, hipStream_t s)
{
    if constexpr (ST == ST_F32 || !LBM_PAIR16) {
        return false;
    } else {
        // TRT only: with MRT the two collisions per thread cost more than
        // the wider accesses gain (measured +5% even-step time on 512x256x256)
        if (a.mask || a.et || cl == CL_MLP || coll != COLL_TRT || a.nx % 128 != 0) return false;
        int bx = 256;
        while ((a.nx / 2) % bx != 0) bx >>= 1;  // nx / 2 is a multiple of 64
        const int by = 256 / bx;
        const dim3 grid(a.nx / 2 / bx, (a.ny + by - 1) / by, a.nz), block(bx, by, 1);
        if (cl == CL_NONE)
            k_even_pair16<Q, ST, CL_NONE, COLL_TRT, HINT><<<grid, block, 0, s>>>(a);
        else
            k_even_pair16<Q, ST, CL_SMAG, COLL_TRT, HINT><<<grid, block, 0, s>>>(a);
        return true;
    }
}

template <int Q, int ST, bool HINT>
static hipError_t step_q_st(const LatticeArgs &a, const HrrArgs &h, int cl, int coll, int odd, hipStream_t s)
{
    if (!(odd & 1) && even_pair16<Q, ST, HINT>(a, cl, coll, s)) return hipGetLastError();
    const Launch L = lattice_launch(a, ST, cl, coll, odd & SC_CACHED);
    const bool mk = a.mask != nullptr;
    if (cl == CL_MLP) {  // the learned closure runs with the TRT collision
        if (coll != COLL_TRT) return hipErrorInvalidValue;
        if (mk)
            launch_sc<Q, ST, CL_MLP, true, COLL_TRT, HINT>(a, h, odd, L, s);
        else
            launch_sc<Q, ST, CL_MLP, false, COLL_TRT, HINT>(a, h, odd, L, s);
    } else if (coll == COLL_HRR) {  // D3Q19, no closure
        if constexpr (Q == 19) {
            if (cl != CL_NONE) return hipErrorInvalidValue;
            if (mk)
                launch_sc<Q, ST, CL_NONE, true, COLL_HRR, HINT>(a, h, odd, L, s);
            else
                launch_sc<Q, ST, CL_NONE, false, COLL_HRR, HINT>(a, h, odd, L, s);
        } else {
            return hipErrorInvalidValue;
        }
    } else if (coll == COLL_MRT) {
        step_coll<Q, ST, COLL_MRT, HINT>(a, h, cl, mk, odd, L, s);
    } else {
        step_coll<Q, ST, COLL_TRT, HINT>(a, h, cl, mk, odd, L, s);
    }
    return hipGetLastError();
}

// HINT off: the lattices that step together fit the last-level cache (SC_CACHED).
template <bool HINT>
hipError_t step_aa(const LatticeArgs &a, const HrrArgs &h, int q, int st, int cl, int coll, int odd, hipStream_t s)
{
    return dispatch(q, st, [&](auto Q, auto ST) { return step_q_st<Q.value, ST.value, HINT>(a, h, cl, coll, odd, s); });
}

}  // namespace lbm
