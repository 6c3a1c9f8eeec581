// HIP kernels (gfx950) of one PIC step and its bookkeeping.
//
// Step pipeline on one stream:
//   k_push        gather, RICS drag / events, kick, move, fixed-point current
//                 deposit (LDS window per tile), per-cell histogram of the new
//                 positions, pair injection by append
//   k_append      photon conversion into pairs and refill of the surface
//                 layers, both by append
//   k_field       Ampere E -= 4 pi (j - j_twist), averages
//   k_plan        live counts, tile plan of the next push, step counter
//   k_sort_*      every sort_interval steps: counting sort by position (cell and
//                 eighth of a cell) per segment, dropping absorbed particles
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"
#include "rics_dev.h"

namespace pic1d {

// ---------------------------------------------------------------------------
// small wave / block reductions (wavefront of 64 lanes)
// ---------------------------------------------------------------------------
__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// The sum over a wavefront, in its last lane, by register moves between lanes (the shuffles
// above go through the LDS unit).
__device__ __forceinline__ uint32_t wave_sum_last(uint32_t v) {
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);     // row_shr 1, 2, 4, 8:
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);     //   sums over rows of 16
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);     //   in their last lanes
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);    // row_bcast 15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);    // row_bcast 31 into rows 2 and 3
    return (uint32_t)x;
}

// Data that the running kernel never writes (segment tables, line constants),
// read at a wave-uniform index: through the constant address space the compiler
// issues scalar loads into SGPRs instead of holding the values in VGPRs.
template <typename T>
__device__ __forceinline__ auto kconst(const T* p) {
#if defined(__HIP_DEVICE_COMPILE__)
    return (const __attribute__((address_space(4))) T*)(p);
#else
    return p;
#endif
}

// Whether an earlier error stops the kernel, the same answer for the whole block: a kernel
// that may set the error word itself, and whose wavefronts wait for each other, must not
// lose some of them to it.
__device__ __forceinline__ bool block_stopped(const DevScalars* sc) {
    __shared__ int s_err;
    if (threadIdx.x == 0) s_err = sc->err;
    __syncthreads();
    return s_err != 0;
}

// Segment of a global tile index by binary search over the tile prefix.
template <typename P>
__device__ __forceinline__ int find_segment(P prefix, int nseg, int t) {
    int lo = 0, hi = nseg;           // prefix[lo] <= t < prefix[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

// XCD-aware tile walk: the 8 XCDs each take a contiguous range of tiles (blocks
// are dispatched round-robin over XCDs, so block b runs on XCD b % 8).
// Same walk at wavefront granularity: wavefront w of block b takes tile slots of
// its XCD's range.
struct WaveWalk {
    int t, end, stride;
    __device__ WaveWalk(int total, int xcd = 1) {
        const int wpb = blockDim.x >> 6;
        const int nb = gridDim.x >> 3;
        // wave-uniform: keeps every per-tile quantity in scalar registers
        const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if (!xcd || nb == 0 || (gridDim.x & 7) != 0) {
            t = blockIdx.x * wpb + wid; end = total; stride = gridDim.x * wpb;
            return;
        }
        const int x = blockIdx.x & 7, lw = (blockIdx.x >> 3) * wpb + wid;
        const int chunk = (total + 7) >> 3;
        t = x * chunk + lw;
        end = min(total, (x + 1) * chunk);
        stride = nb * wpb;
    }
};

struct TileWalk {
    int t, end, stride;
    __device__ TileWalk(int total) {
        const int nb = gridDim.x >> 3;
        const int x = blockIdx.x & 7, lb = blockIdx.x >> 3;
        if (nb == 0 || (gridDim.x & 7) != 0) { t = blockIdx.x; end = total; stride = gridDim.x; return; }
        const int chunk = (total + 7) >> 3;
        t = x * chunk + lb;
        end = min(total, (x + 1) * chunk);
        stride = nb;
    }
};

// {b, mu, x} of a cell's lower node and their change over the cell.
struct GeoCell {
    float b, mu, x, db, dmu, dx;
    __device__ __forceinline__ void load(const float4& lo, const float4& hi) {
        b = lo.x; mu = lo.y; x = lo.z;
        db = hi.x - lo.x; dmu = hi.y - lo.y; dx = hi.z - lo.z;
    }
};

// Geometry of a particle at offset f in its cell: linear between the two nodes.
__device__ __forceinline__ Geo geo_lerp(const LineDev& L, const GeoCell& c, float f) {
    Geo g;
    g.b = fmaf(f, c.db, c.b);
    g.mu = fmaf(f, c.dmu, c.mu);
    const float xr = fmaf(f, c.dx, c.x);
    g.ix2 = frcp(xr * xr);
    g.by = g.b * L.inv_theta;
    return g;
}

__device__ __forceinline__ Geo geo_lerp(const LineDev& L, const float4& lo, const float4& hi, float f) {
    GeoCell c;
    c.load(lo, hi);
    return geo_lerp(L, c, f);
}

// What the RICS evaluations of one particle share: its geometry and (table
// backend) its table rows.
struct PartGeo {
    Geo g;
    TabRows rows;
    TabMemo memo;
};

// The line's table, and how far its Ndot lies behind its F.
__device__ __forceinline__ const char* tab_base(const PushArgs& a, const LineDev& L) {
    return reinterpret_cast<const char*>(a.table + 2 * (int64_t)L.table_off);
}
__device__ __forceinline__ uint32_t tab_n_off(const PushArgs& a) { return 8u * (uint32_t)(a.ns * a.nlg); }

// F_hat at u with what dF/du needs (evaluated only where the midpoint asks for it).
template <int BACKEND>
__device__ __forceinline__ auto rics_eval(const PushArgs& a, const LineDev& L, float u, PartGeo& pg) {
    if constexpr (BACKEND == RICS_TABLE) {
        const char* tb = tab_base(a, L);
        return table_eval(L, tb, tab_n_off(a), a.nlg, pg.rows, u, pg.memo);
    } else {
        return exact_eval(L, u, pg.g);
    }
}
__device__ __forceinline__ float eval_dF(const LineDev& L, const TableEval& e) { return e.dF(L); }
__device__ __forceinline__ float eval_dF(const LineDev&, const ExactEval& e) { return e.dF(); }

template <int BACKEND>
__device__ __forceinline__ float rics_N(const PushArgs& a, const LineDev& L, float u, PartGeo& pg) {
    if constexpr (BACKEND == RICS_TABLE) {
        const char* tb = tab_base(a, L);
        return table_N(L, tb, tab_n_off(a), a.nlg, pg.rows, u, pg.memo);
    } else {
        return exact_N(L, u, pg.g);
    }
}

// Geometry and table rows of a particle at x = c0 + o0 in float64 (the general
// form; the pusher forms the rows per cell where it can).
template <int BACKEND>
__device__ __forceinline__ PartGeo part_geo(const PushArgs& a, const LineDev& L, const float4& n0, const float4& n1,
                                            int c0, float o0) {
    PartGeo pg;
    pg.g = geo_lerp(L, n0, n1, o0);
    if constexpr (BACKEND == RICS_TABLE) pg.rows = table_rows(L, a.ns, 8 * a.nlg, (double)c0 + (double)o0);
    return pg;
}

// Newton-Raphson on u1 - u0 - (h/4)(F(u0) + F(u1)) = 0 from the explicit start
// (kept out of line: it is rarely needed at these step sizes).
template <int BACKEND>
__device__ __forceinline__ float newton_midpoint(const PushArgs& a, const LineDev& L, float u0, float F0, float u1,
                                              PartGeo& g) {
    const float hq = 0.25f * L.h;
#pragma unroll 1
    for (int it = 0; it < 4; ++it) {
        const auto e1 = rics_eval<BACKEND>(a, L, u1, g);
        const float G = u1 - u0 - hq * (F0 + e1.F);
        const float del = G / (1.0f - hq * eval_dF(L, e1));
        u1 -= del;
        if (fabsf(del) <= 0x1.0p-24f * fabsf(u1)) break;
    }
    return u1;
}

// One drag update over h/2 (Sec. 3): implicit midpoint where |F(p0)| tau_min <= |p0|,
// solved by Newton from the explicit start p0 + (h/2) F(p0) -- needed only when
// the predicted correction (h/4)|F'|(h/2)|F0| exceeds half an ulp of the result,
// F' taken at p0 -- and exponential relaxation towards p_tilde = mu / (1 - mu^2)^(1/2)
// otherwise.
template <int BACKEND>
__device__ __forceinline__ float drag_half(const PushArgs& a, const LineDev& L, float u0, PartGeo& g,
                                           float ptilde, bool alive, int& n_limited, int& n_newton) {
    const auto e0 = rics_eval<BACKEND>(a, L, u0, g);
    const float F0 = e0.F;
    const bool implicit = fabsf(F0) * L.tau_hat <= fabsf(u0);
    float u1 = implicit ? fmaf(0.5f * L.h, F0, u0) : fmaf(-(u0 - ptilde), L.damp, u0);
    n_limited += (alive && !implicit) ? 1 : 0;
    // F = 0 beyond the Planck cutoff (cold particles): the explicit start is the root
    if (implicit && F0 != 0.0f &&
        0.25f * L.h * fabsf(eval_dF(L, e0)) * 0.5f * L.h * fabsf(F0) > 0x1.0p-25f * fabsf(u1)) {
        n_newton += alive ? 1 : 0;
        u1 = newton_midpoint<BACKEND>(a, L, u0, F0, u1, g);
    }
    return u1;
}

// Per-tile constants of the pusher (species of the tile, step, count buffers).
struct TileCtx {
    uint64_t step;
    int32_t* hist_out;          // counts of the new positions
    float inv_mass;             // m_e / m
    bool negative;              // negative charge
    bool gravity;               // the tile touches an atmosphere layer
    int item;                   // work item (the queue of the network's pusher)
};

struct Counts {
    int events = 0, pairs = 0, escaped = 0, absorbed = 0, clipped = 0, limited = 0, newton = 0, pushed = 0,
        draws = 0, mlp = 0, pushed_ion = 0, mlp_need = 0;
};

// Stochastic regime (b >= b_thr, Sec. 3): after the kick, a scattering event with
// probability min(Ndot h, 1) from the Philox draw keyed by (step, id); the event
// emits eps = gamma (1 - (1+2b)^-1/2) and leaves gamma / (1+2b)^1/2 (Appendix A), or,
// with an angular emission pattern, the photon leaves the excited lepton's rest frame
// at the cosine drawn from the block's other words.
// Append regions fill by the wavefront's slot where each wavefront walks fixed tiles; from
// the queue, which hands items out by timing, by the item, so that whether a region overflows
// follows from the state alone: consecutive items go to regions of their own, and (the
// second term) so do the same items of lines a multiple of 256 items long.
template <bool QUEUE>
__device__ __forceinline__ float stochastic_step(const PushArgs& a, const LineDev& L, const TileCtx& T, int line,
                                              int64_t k, int c0, float o0, float u, const Geo& g, float ndot,
                                              Counts& cnt) {
    const float lam = ndot * L.h;
    if (lam > 1.0f) ++cnt.clipped;
    if (!(lam > 0.0f)) return u;
    ++cnt.draws;
    const uint64_t pid = a.id[k];
    // (the round keys formed here: kept for the launch, they spill)
    uint32_t k0 = a.key0, k1 = a.key1;
    asm volatile("" : "+s"(k0), "+s"(k1));
    const uint4 w = philox4x32_10_wide(make_uint4((uint32_t)T.step, (uint32_t)pid, (uint32_t)(pid >> 32), STREAM_RICS),
                                       k0, k1);
    if (!(uniform24(w.x) < fminf(lam, 1.0f))) return u;
    ++cnt.events;
    const float gam = fsqrt(fmaf(u, u, 1.0f));
    const float dir = (u >= 0.0f) ? 1.0f : -1.0f;
    const float u_pre = u;
    float eps, mu_r = 0.0f;
    if (a.emission == 0) {
        eps = photon_energy(gam, g.b);
        const float gnew = gam * frsq(fmaf(2.0f, g.b, 1.0f));
        u = dir * fsqrt(fmaxf((gnew - 1.0f) * (gnew + 1.0f), 0.0f));
    } else {
        mu_r = emission_cosine(w, a.emission);
        eps = angled_event(gam, g.b, mu_r, dir, u);
    }
    if (a.pairs && eps >= 2.0f) {
        // record for the conversion kernel; lanes of a wavefront reserve their slots together
        const unsigned long long m = __ballot(1);
        const int lane = threadIdx.x & 63;
        const int leader = __ffsll((long long)m) - 1;
        const int r = QUEUE ? (T.item ^ (T.item >> 8)) & (PHOTON_REPL - 1)
                            : (int)((blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) & (PHOTON_REPL - 1));
        int slot0 = 0;
        if (lane == leader) slot0 = atomicAdd(&a.n_photons[r], __popcll(m));
        const int slot = __shfl(slot0, leader, 64) + __popcll(m & ((1ull << lane) - 1ull));
        if (slot < a.photon_region) {
            PhotonRec& p = a.photons[(size_t)r * a.photon_region + slot];
            p.pid = pid;
            p.line = line;
            p.cell = c0;
            p.off = o0;
            p.u_pre = u_pre;
            p.b = g.b;
            p.mu = mu_r;
        } else {
            set_error(&a.sc->err, -3);
        }
    } else {
        ++cnt.escaped;
    }
    return u;
}

// ---------------------------------------------------------------------------
// Surrogate-network RICS (RICS_MLP).  The network runs on the matrix cores for
// the 64 particles of a wavefront at once (four groups of 16 samples), so every
// lane must reach each evaluation: the callers below are wave-uniform.
// ---------------------------------------------------------------------------
struct MlpRics {
    float F, N;
};

// F_hat and Ndot_hat at momentum u of a particle with geometry g at arc-length
// fraction sl (x / n): the network gives G = |F_hat| / |gamma mu - u| and Ndot at
// (log10 gamma, s/L of the particle or of its mirror point, log10 b, kT);
// F_hat = (gamma mu - u) G, and both vanish beyond the Planck cutoff.
__device__ __forceinline__ MlpRics mlp_rics(const PushArgs& a, const bf16x8* W, const float* Wb, float u,
                                            const Geo& g, float sl, int& n_eval) {
    const int lane = threadIdx.x & 63, g4 = lane >> 4, r = lane & 15;
    ++n_eval;
    const float ua = fabsf(u);
    const float gam = fsqrt(fmaf(ua, ua, 1.0f));
    constexpr float LOG10_2 = 0.301029995663981f;
    float xn[4];
    xn[0] = __builtin_amdgcn_logf(gam) * (LOG10_2 * 0.25f) - 1.0f;
    xn[1] = fmaf(u >= 0.0f ? sl : 1.0f - sl, 2.0f, -1.0f);
    xn[2] = fmaf(__builtin_amdgcn_logf(g.b) * LOG10_2 + 2.0f, 0.4f, -1.0f);
    xn[3] = a.mlp_kTn;
    float o0 = 0.0f, o1 = 0.0f;
#pragma unroll 1
    for (int G = 0; G < 4; ++G) {
        float xg[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) xg[k] = __shfl(xn[k], 16 * G + r, 64);
        const bf16x8 bin = mlp_input_operand(xg, g4);
        const f32x4 out = mlp_group_forward(W, Wb, bin);
        const float v0 = __shfl(out[0], r, 64), v1 = __shfl(out[1], r, 64);
        if (g4 == G) {
            o0 = v0;
            o1 = v1;
        }
    }
    constexpr float LOG2_10 = 3.32192809488736f;
    const float y = g.by * frcp(fmaf(-u, g.mu, gam));
    const bool inside = y <= Y_CUT;
    MlpRics res;
    res.F = inside ? fmaf(gam, g.mu, -u) * exp2f(fmaf(a.mlp_std[0], o0, a.mlp_mean[0]) * LOG2_10) : 0.0f;
    res.N = inside ? exp2f(fmaf(a.mlp_std[1], o1, a.mlp_mean[1]) * LOG2_10) : 0.0f;
    return res;
}

// Drag half step with the surrogate force F0 = F(u0) (Sec. 3): damping branch where
// |F0| tau_min > |u0|; otherwise the implicit midpoint u1 = u0 + (h/4)(F0 + F(u1)),
// from the explicit start and refined by fixed-point iteration (contraction
// (h/4)|F'| << 1 on this branch) where (h/2)|F0| exceeds 2^-12 |u0|, until the
// next correction, predicted from the secant slope, is below half an ulp.  The
// network gives no derivative without another evaluation, so the gate is on F0
// alone: a skipped correction is (h/4)|F'| (h/2)|F0| / (1 - (h/4)|F'|), at most
// 2^-12 (|F'| h/4) / (1 - |F'| h/4) |u0| -- below half an ulp of u0 while
// |F'| h/4 < 2^-13, and within the 1e-5 momentum budget while |F'| h/4 < 0.04.
// Lanes with active == false return u0 but still take part in the network
// evaluations.
__device__ __forceinline__ float mlp_drag_half(const PushArgs& a, const bf16x8* W, const float* Wb, const LineDev& L,
                                               float u0, float F0, const Geo& g, float sl, float ptilde, bool active,
                                               bool alive, Counts& cnt) {
    const bool implicit = fabsf(F0) * L.tau_hat <= fabsf(u0);
    float u1 = implicit ? fmaf(0.5f * L.h, F0, u0) : fmaf(-(u0 - ptilde), L.damp, u0);
    cnt.limited += (active && alive && !implicit) ? 1 : 0;
    bool refine = active && implicit && F0 != 0.0f && 0.5f * L.h * fabsf(F0) > 0x1.0p-12f * fabsf(u0);
    cnt.newton += (refine && alive) ? 1 : 0;
#pragma unroll 1
    for (int it = 0; it < 4; ++it) {
        if (__ballot(refine) == 0ull) break;
        cnt.mlp_need += (refine && alive) ? 1 : 0;
        const float F1 = mlp_rics(a, W, Wb, u1, g, sl, cnt.mlp).F;
        const float un = fmaf(0.25f * L.h, F0 + F1, u0);
        // the next correction would be (h/4) F' (un - u1); F' from the secant through
        // the evaluations at u0 and u1.  Stop once it is below half an ulp of un.
        const float du = u1 - u0;
        const float slope = du != 0.0f ? (F1 - F0) / du : 0.0f;
        const bool more = 0.25f * L.h * fabsf(slope) * fabsf(un - u1) > 0x1.0p-25f * fabsf(un);
        u1 = refine ? un : u1;
        refine = refine && more;
    }
    return active ? u1 : u0;
}

// Field and geometry of the cell a lane is working in.  A lane's particles are
// consecutive in cell order, so the cache is reloaded only when the cell changes.
// The kick q E / (m C) is kept as its value at the cell centre and its change per
// cell towards the neighbouring centres, whose E is clamped at the walls (the
// gather is constant beyond the outermost cell centres).  The table backend
// keeps the per-cell part of the particle's table rows (k_cell_records): for offset o the
// row position is rows0.pos.wj + o s_scale (u >= 0) and rows0.neg.wj - o s_scale
// (mirrored), valid for the whole cell where the cell lies between two rows, clear
// of the clamped ends.
struct CellCache {
    int cell;
    float K0, KsL, KsU;
    GeoCell geo;
    TabRows rows0;          // (rows0.pos.off < 0: the general form)
    TabMemo memo;           // the lane's last table record (reset per tile)
};

template <int BACKEND>
__device__ __forceinline__ void cache_load(CellCache& cc, const PushArgs& a, const LineDev& L, float qmC, int c0) {
    cc.cell = c0;
    // (32-bit byte offsets from the line's arrays: one address register per load)
    struct __attribute__((packed, aligned(4))) Three { float m, c, p; };
    const uint32_t e = 4u * (uint32_t)c0;
    const Three E = *reinterpret_cast<const Three*>(reinterpret_cast<const char*>(a.E32 + L.field_base - 1) + e);
    cc.K0 = qmC * E.c;
    cc.KsL = qmC * (E.c - E.m);
    cc.KsU = qmC * (E.p - E.c);
    if constexpr (BACKEND == RICS_TABLE) {
        const char* rec = reinterpret_cast<const char*>(a.cell_rec + 2 * (size_t)L.cell_base);
        const float4 g = *reinterpret_cast<const float4*>(rec + 8u * e);
        const float4 r = *reinterpret_cast<const float4*>(rec + (8u * e + 16u));
        cc.geo.b = g.x;
        cc.geo.mu = g.y;
        cc.geo.db = g.z;
        cc.geo.dmu = g.w;
        cc.geo.x = cc.geo.dx = 0.0f;       // (in the table's values already)
        cc.rows0.pos.off = __float_as_int(r.x);
        cc.rows0.pos.wj = r.y;
        cc.rows0.neg.off = __float_as_int(r.z);
        cc.rows0.neg.wj = r.w;
    } else if constexpr (BACKEND != RICS_OFF) {
        const char* nd = reinterpret_cast<const char*>(a.nodes + L.node_base);
        const float4 lo = *reinterpret_cast<const float4*>(nd + 4u * e);
        const float4 hi = *reinterpret_cast<const float4*>(nd + (4u * e + 16u));
        cc.geo.load(lo, hi);
    }
}

// What the table backend's particle kernel reads of a cell, in one place, once per
// state: {b, mu} at its lower face and their change over it; the table rows {row offset,
// weight} at the lower face for u >= 0 and mirrored, an offset of -1 where a particle
// has to form its rows itself.
__global__ __launch_bounds__(256) void k_cell_records(float4* rec, const float4* nodes, const int32_t* cell_line,
                                                      const LineDev* lines, int n_total, int ns, int nlg) {
    for (int g = blockIdx.x * 256 + threadIdx.x; g < n_total; g += gridDim.x * 256) {
        const LineDev& L = lines[cell_line[g]];
        const int c = g - L.cell_base;
        GeoCell geo;
        geo.load(nodes[L.node_base + c], nodes[L.node_base + c + 1]);
        rec[2 * (size_t)g] = make_float4(geo.b, geo.mu, geo.db, geo.dmu);
        const double sc = L.s_scale;
        const double fp = fma((double)c, sc, -0.5);
        const double fn = fma((double)(L.n_cells - c), sc, -0.5);
        const double jp = floor(fp), jn = floor(fn);
        const double top = (double)(ns - 2);
        constexpr double M = 0x1.0p-20;      // margin for the float32 row weight
        const bool simple = jp >= 0.0 && jp <= top && fp + sc <= jp + 1.0 - M &&
                            jn >= 0.0 && jn <= top && fn - sc >= jn + M;
        const int nlg8 = 8 * nlg;
        rec[2 * (size_t)g + 1] = make_float4(__int_as_float(simple ? (int)jp * nlg8 : -1), (float)(fp - jp),
                                             __int_as_float(simple ? (int)jn * nlg8 : -1), (float)(fn - jn));
    }
}

// Everything one particle does in one step: gather, RICS, kick, move, and the
// deposit of its path in fixed point.  Written without data-dependent branches on
// the common path.  Dead slots (absorbed particles and the padding of a partial
// tile) enter at o0 = 1/2, u = 0, are held at u = 0, and so stay in their cell and
// deposit nothing.  c0 is the cached cell.
// Returns the new cell (DEAD_CELL when absorbed or dead) in c1, d = c1 - c0 in
// {-1, 0, 1}, and the path's overlaps with cells c0-1, c0, c0+1 in units of 2^-28
// cell (unsigned by the charge; jm and jp vanish unless the path leaves the cell).
template <int BACKEND>
__device__ __forceinline__ void advance_particle(const PushArgs& a, const LineDev& L, const TileCtx& T,
                                                 CellCache& cc, bool alive, int line, int sp, int64_t k,
                                                 int c0, float o0, float& u, Counts& cnt, int& c1, float& o1,
                                                 int& jm, int& j0, int& jp, int& d, bool& gone, const bf16x8* W,
                                                 const float* Wb) {
    const int n = L.n_cells;
    constexpr bool RICS = BACKEND != RICS_OFF;

    // field gather: E at x^n, linear between cell centres (as the kick per step)
    const float ws = o0 - 0.5f;
    float kick = fmaf(ws, ws >= 0.0f ? cc.KsU : cc.KsL, cc.K0);
    if (T.gravity) {
        const double x = (double)c0 + (double)o0;
        const double dw = fmin(x, (double)n - x);
        const float gk = ((x < (double)L.half_n) ? -1.0f : 1.0f) * L.grav * T.inv_mass;
        kick += (dw <= L.atm_depth) ? gk : 0.0f;
    }

    if constexpr (BACKEND == RICS_MLP) {
        if (sp != 3) {            // wave-uniform: a tile holds one species
            const Geo g = geo_lerp(L, cc.geo, o0);
            const float sl = (float)(((double)c0 + (double)o0) / (double)n);
            const bool cont = g.b < L.b_thr;
            const float pt = g.mu * frsq(fmaxf(fmaf(-g.mu, g.mu, 1.0f), 1e-30f));
            // the force at u^n is needed only in the continuous regime: a wavefront with
            // no live lane there skips the first evaluation (the step needs F at u^n and
            // at the kicked u in that regime, Ndot at the kicked u in the stochastic one)
            const bool any_cont = __ballot(cont && alive) != 0ull;
            cnt.mlp_need += alive ? (cont ? 2 : 1) : 0;
            if (any_cont) {
                const MlpRics ra = mlp_rics(a, W, Wb, u, g, sl, cnt.mlp);
                u = mlp_drag_half(a, W, Wb, L, u, ra.F, g, sl, pt, cont, alive, cnt);
            }
            u += kick;
            const MlpRics rb = mlp_rics(a, W, Wb, u, g, sl, cnt.mlp);
            if (any_cont) u = mlp_drag_half(a, W, Wb, L, u, rb.F, g, sl, pt, cont, alive, cnt);
            if (!cont && alive) u = stochastic_step<true>(a, L, T, line, k, c0, o0, u, g, rb.N, cnt);
        } else {
            u += kick;
        }
    } else if (RICS && sp != 3) {
        PartGeo pg;
        pg.g = geo_lerp(L, cc.geo, o0);
        if constexpr (BACKEND == RICS_TABLE) {
            pg.memo = cc.memo;
            if (cc.rows0.pos.off >= 0) {
                pg.rows.pos.off = cc.rows0.pos.off;
                pg.rows.pos.wj = fmaf(o0, L.s_scale_f, cc.rows0.pos.wj);
                pg.rows.neg.off = cc.rows0.neg.off;
                pg.rows.neg.wj = fmaf(-o0, L.s_scale_f, cc.rows0.neg.wj);
            } else {
                pg.rows = table_rows(L, a.ns, 8 * a.nlg, (double)c0 + (double)o0);
            }
        }
        if (pg.g.b < L.b_thr) {
            // continuous regime: Strang splitting drag h/2, Lorentz kick, drag h/2, both
            // at x^n; the damping branch relaxes towards p_tilde = mu / (1 - mu^2)^(1/2)
            const float pt = pg.g.mu * frsq(fmaxf(fmaf(-pg.g.mu, pg.g.mu, 1.0f), 1e-30f));
            u = drag_half<BACKEND>(a, L, u, pg, pt, alive, cnt.limited, cnt.newton);
            u += kick;
            u = drag_half<BACKEND>(a, L, u, pg, pt, alive, cnt.limited, cnt.newton);
        } else {
            u += kick;
            if (alive) u = stochastic_step<false>(a, L, T, line, k, c0, o0, u, pg.g, rics_N<BACKEND>(a, L, u, pg), cnt);
        }
        if constexpr (BACKEND == RICS_TABLE) cc.memo = pg.memo;
    } else {
        u += kick;
    }
    u = alive ? u : 0.0f;      // (a non-finite u is reported once per tile by the caller)

    // move x^{n+1} = x^n + C u / gamma with the offset carried into the cell index
    // (|C u / gamma| < 1/2, so the carry is -1, 0 or 1 and o1 - carry is exact; o1 + 1
    // may round up to 1)
    const float o1r = fmaf(L.C * u, frsq(fmaf(u, u, 1.0f)), o0);
    const float carry = floorf(o1r);
    o1 = o1r - carry;
    const bool fix = o1 >= 1.0f;
    o1 = fix ? 0.0f : o1;
    d = (int)carry + (fix ? 1 : 0);
    c1 = c0 + d;
    // fixed-point deposit of the path from the stored old and new offsets quantised
    // to 2^-28 cell: X1 is the new position relative to the old cell's left face.
    // Differences of quantised stored positions telescope, so the deposit equals the
    // change of the quantised charge density exactly.  The parts beyond a wall land
    // in cells -1 or n, which the flush drops.
    constexpr int ONE = 1 << POS_BITS;
    const int f0 = (int)(o0 * POS_SCALE);
    const int X1 = d * ONE + (int)(o1 * POS_SCALE);
    jm = min(X1, 0);
    j0 = min(max(X1, 0), ONE) - f0;
    jp = max(X1 - ONE, 0);
    const bool out = (unsigned)c1 >= (unsigned)n;
    cnt.absorbed += (alive && out) ? 1 : 0;
    gone = out || !alive;
    c1 = gone ? DEAD_CELL : c1;
}

__device__ __forceinline__ void counts_flush(unsigned long long* counters, int line, Counts& c) {
    const int v[12] = {c.events, c.pairs, c.escaped, c.absorbed, c.clipped, c.limited, c.newton, c.pushed, c.draws,
                       c.mlp, c.pushed_ion, c.mlp_need};
    const int slot[12] = {0, 1, 2, 3, 4, 5, 6, 8, 9, 10, 12, 13};
    const size_t rep = ((size_t)line * CNT_REPL + (blockIdx.x & (CNT_REPL - 1))) * NCOUNT;
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const int s = wave_sum_i(v[i]);
        if ((threadIdx.x & 63) == 0 && s != 0) atomicAdd(&counters[rep + slot[i]], (unsigned long long)s);
    }
    c = Counts();
}

// Waves per SIMD the particle kernel is compiled for, per backend.  A wavefront's
// LDS is its staged tile (768 bytes per particle per lane: 6 KB at 8) plus its
// deposit window (12 bytes per cell): at 8 particles per lane and 128 cells five
// 256-thread blocks fit a CU (five waves per SIMD, what the table backend's
// registers allow), at 32 cells six (the closed-form and field-only backends, in
// 80 registers with at most a few spilled).  The tile (4, 8 or 16 particles per
// lane) and the window (cells) are template parameters picked by the autotuner;
// tiles whose cells span more than the window deposit through global atomics.
constexpr int push_waves(int backend) {
    return backend == RICS_MLP ? 2 : backend == RICS_TABLE ? 5 : 6;
}

// Sorting network on PPT keys (ascending): the 19-comparator network for 8, five
// comparators for 4, Batcher's bitonic network for 16.
template <int PPT>
__device__ __forceinline__ void sort_keys(uint32_t* k) {
    auto cx = [&](int i, int j) {
        const uint32_t x = k[i], y = k[j];
        k[i] = min(x, y);
        k[j] = max(x, y);
    };
    if constexpr (PPT == 2) {
        cx(0, 1);
    } else if constexpr (PPT == 4) {
        cx(0, 1); cx(2, 3); cx(0, 2); cx(1, 3); cx(1, 2);
    } else if constexpr (PPT == 8) {
        constexpr int NET[19][2] = {{0, 2}, {1, 3}, {4, 6}, {5, 7}, {0, 4}, {1, 5}, {2, 6}, {3, 7}, {0, 1}, {2, 3},
                                    {4, 5}, {6, 7}, {2, 4}, {3, 5}, {1, 4}, {3, 6}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
        for (int e = 0; e < 19; ++e) cx(NET[e][0], NET[e][1]);
    } else {
#pragma unroll
        for (int size = 2; size <= PPT; size <<= 1)
#pragma unroll
            for (int stride = size >> 1; stride > 0; stride >>= 1)
#pragma unroll
                for (int i = 0; i < PPT; ++i) {
                    const int j = i ^ stride;
                    if (j > i) {
                        if ((i & size) == 0) cx(i, j);
                        else cx(j, i);
                    }
                }
    }
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The particle kernel.  Work is split into tiles of 64 PPT consecutive particles
// of one (line, species) segment, one tile per wavefront at a time, PPT
// consecutive particles per lane (128-bit loads and stores).  Each lane
// accumulates its deposit and new-cell counts over runs of particles in the same
// cell (three cells wide: the run's cell and its neighbours); each wavefront
// merges its lanes in a private LDS window and flushes the window to the global
// fixed-point current with one atomic per touched cell.  No block-level
// synchronisation.
// Bound, with the table, by vector issue (70-80% of the cycles) and by the latency of
// the loads at a change of cell and of the table gathers, five wavefronts per SIMD
// covering the rest.  So a change of cell is three wide loads of ready values
// (k_cell_records, the field's neighbours in one), a table lookup one gather, the
// Philox keys are formed where they are used, and a run's sums go to the window as they
// are.  2.7e7 heated particles on 65,536 cells: 244 -> 225 us; 4e7 at the density limit
// 433 -> 389; the cascade lines 644 -> 581; 40 uneven lines 736 -> 696 (against eight
// loads and the rows in float64 at every change of cell, and two gathers).
template <int BACKEND, int PPT, int WW, int KIND, int SUB>
__global__ __launch_bounds__(BACKEND == RICS_MLP ? PUSH_TPB_MLP : PUSH_TPB)
__attribute__((amdgpu_waves_per_eu(push_waves(BACKEND)))) void k_push(PushArgs a) {
    static_assert(PPT == 2 || PPT == 4 || PPT == 8 || PPT == 16, "2, 4, 8 or 16 particles per lane");
    // A wavefront's item: TILE particles, one of the SUB parts of a planned tile.
    constexpr int TILE = 64 * PPT;
    // With the surrogate network a particle costs between one evaluation and six,
    // depending on where it is: the wavefronts take their items from a queue, and half
    // a planned tile at a time, as a few of these fill a launch (4.9e6 particles on 16,384
    // cells: 2.40 ms where each XCD walked its own range of whole tiles, the wavefronts
    // of the cheap ranges idle 45% of the launch; 1.56 to 1.65 ms so, by card, with two
    // wavefronts per SIMD; three spill, 1.87 ms beside 1.65).  States of fewer items than
    // wavefronts leave some without one (10 steps of 4,000 cells of 60 pairs 9.3 ms, 13.1
    // before the queue; of 1,000 cells 5.2 and 6.1; 500 cells of 30 pairs 3.3 and 4.7).
    // Bound by vector issue: 1,500 instructions and 308 MFMAs per 16 evaluations.
    constexpr bool QUEUE = BACKEND == RICS_MLP;
    using VecI = std::conditional_t<PPT == 2, int2, int4>;
    using VecF = std::conditional_t<PPT == 2, float2, float4>;
    constexpr int VN = PPT == 2 ? 2 : 4;          // particles per vector load
    constexpr int TPB = BACKEND == RICS_MLP ? PUSH_TPB_MLP : PUSH_TPB;
    __shared__ unsigned long long sJ[TPB / 64][WW];
    __shared__ int sH[TPB / 64][WW];
    __shared__ int sPc[TPB / 64][PPT][64];      // the wave's tile: cell, offset, momentum
    __shared__ float sPo[TPB / 64][PPT][64];
    __shared__ float sPu[TPB / 64][PPT][64];
    // surrogate weights, staged once per block (the network runs on them for every particle)
    __shared__ bf16x8 sW[BACKEND == RICS_MLP ? FT_TOTAL * 64 : 1];
    if constexpr (BACKEND == RICS_MLP) {
        // before the error check: every wave of the block reaches the barrier
        for (int e = threadIdx.x; e < FT_TOTAL * 64; e += TPB) sW[e] = a.mlp_ft[e];
        __syncthreads();
    }
    if (a.sc->err != 0) return;
    const uint64_t step = a.sc->step;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.sc->step_field = step;
    int32_t* hist_out = (step & 1) ? a.hist[0] : a.hist[1];
    const int total = SUB * a.tile_prefix[a.nseg];
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Counts cnt;
    int cur_line = -1;
    int seg = 0, seg_t0 = 0, seg_t1 = 0;       // segment of the previous tile and its tile range
    // The next tile's particles are fetched (vector loads into registers) before the
    // current tile's results are stored and its deposit window flushed, so that the
    // loads are in flight while the stores and atomics drain.
    WaveWalk ww(total, a.xcd_walk);
    auto pop = [&] {
        int t = 0;
        if (lane == 0) t = atomicAdd(a.queue, 1);
        return __builtin_amdgcn_readfirstlane(t);
    };
    if constexpr (QUEUE) {
        ww.t = pop();
        ww.end = total;
    }
    int f_seg = 0, f_ib = 0, f_nv = 0;
    bool f_full = false;
    int64_t f_base = 0;
    VecI fc[PPT / VN];
    VecF fo[PPT / VN], fu[PPT / VN];
    // (every call assigns all fetched values, so that none stays live across the loop)
    auto fetch = [&](int item) {
        const bool have = item < ww.end;
        const int t = SUB == 1 ? item : item / SUB;
        if (have && (t < seg_t0 || t >= seg_t1)) {
            seg = find_segment(kconst(a.tile_prefix), a.nseg, t);
            seg_t0 = kconst(a.tile_prefix)[seg];
            seg_t1 = kconst(a.tile_prefix)[seg + 1];
        }
        f_seg = seg;
        f_base = kconst(a.seg_base)[seg];
        // this lane's PPT consecutive particles (vector loads; slots up to the
        // capacity, a multiple of 256, always exist)
        const int t0 = SUB == 1 ? (t - seg_t0) * TILE : (item - SUB * seg_t0) * TILE;
        const int ncur = kconst(a.n_cur)[seg];
        f_full = have && ncur - t0 >= TILE;        // wave-uniform
        f_ib = t0 + lane * PPT;
        f_nv = have ? max(0, min(PPT, ncur - f_ib)) : 0;
        const VecI* cp = reinterpret_cast<const VecI*>(a.cell + f_base + f_ib);
        const VecF* op = reinterpret_cast<const VecF*>(a.off + f_base + f_ib);
        const VecF* up = reinterpret_cast<const VecF*>(a.u + f_base + f_ib);
#pragma unroll
        for (int h = 0; h < PPT / VN; ++h) {
            if constexpr (PPT == 2) {
                fc[h] = make_int2(DEAD_CELL, DEAD_CELL);
                fo[h] = make_float2(0.5f, 0.5f);
                fu[h] = make_float2(0.f, 0.f);
            } else {
                fc[h] = make_int4(DEAD_CELL, DEAD_CELL, DEAD_CELL, DEAD_CELL);
                fo[h] = make_float4(0.5f, 0.5f, 0.5f, 0.5f);
                fu[h] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            if (f_nv > 0) { fc[h] = cp[h]; fo[h] = op[h]; fu[h] = up[h]; }
        }
    };
    fetch(ww.t);
    int next = 0;
    for (; ww.t < ww.end; ww.t = QUEUE ? next : ww.t + ww.stride) {
        if constexpr (QUEUE) next = pop();
        const int tseg = f_seg, ib = f_ib, nv = f_nv;
        const int64_t base = f_base;
        const int line = tseg >> 2, sp = tseg & 3;
        if (line != cur_line) {
            if (cur_line >= 0) counts_flush(a.counters, cur_line, cnt);
            cur_line = line;
        }
        const LineDev L = kconst(a.lines)[line];
        // the surrogate's states with lines on both sources push them in two launches
        // (table lines at the table kernel's occupancy): a tile of the other kind is
        // left to the other launch
        if constexpr (KIND != 0) {
            if ((L.use_table != 0) != (KIND == 1)) {
                fetch(QUEUE ? next : ww.t + ww.stride);
                continue;
            }
        }
        // the fetched particles, staged in the wave's LDS slots [q][lane] so the
        // particle loop indexes them freely without bank conflicts.  Dead slots are
        // stored as (DEAD_CELL, 1/2, 0); the padding of a partial tile is made so.
        // The lane's cell range: DEAD_CELL is the largest cell as unsigned and the
        // smallest as signed, so neither bound sees it.
        unsigned lo_u = 0xffffffffu;
        int hi_s = INT32_MIN;
        int cst[PPT];
        auto stage = [&](auto full) {
#pragma unroll
            for (int h = 0; h < PPT / VN; ++h) {
                int cv[VN];
                float ov[VN], uv[VN];
                cv[0] = fc[h].x; cv[1] = fc[h].y;
                ov[0] = fo[h].x; ov[1] = fo[h].y;
                uv[0] = fu[h].x; uv[1] = fu[h].y;
                if constexpr (PPT != 2) {
                    cv[2] = fc[h].z; cv[3] = fc[h].w;
                    ov[2] = fo[h].z; ov[3] = fo[h].w;
                    uv[2] = fu[h].z; uv[3] = fu[h].w;
                }
#pragma unroll
                for (int i = 0; i < VN; ++i) {
                    const int q = VN * h + i;
                    const bool valid = decltype(full)::value || q < nv;
                    const int c = valid ? cv[i] : DEAD_CELL;
                    cst[q] = c;
                    lo_u = min(lo_u, (unsigned)c);
                    hi_s = max(hi_s, c);
                    sPc[wid][q][lane] = c;
                    sPo[wid][q][lane] = valid ? ov[i] : 0.5f;
                    sPu[wid][q][lane] = valid ? uv[i] : 0.0f;
                }
            }
        };
        if (f_full) stage(std::true_type{});
        else stage(std::false_type{});
        const bool lane_any = hi_s >= 0;
        const int first = lane_any ? (int)lo_u : 0;
        // the first cell's cache, loaded early so that its latency hides under the
        // tile set-up below
        const float qmC = ((sp == 0 || sp == 2) ? -1.0f : (sp == 1 ? 1.0f : a.qm_ion)) * L.invC;
        CellCache cc;
        cache_load<BACKEND>(cc, a, L, qmC, first);
        // The order in which the lane visits its slots: by cell (dead slots last), so
        // that the run accumulator and the cell cache see each cell once however the
        // particles of a cell are ordered in memory.  A sorting network on keys
        // (cell - first) * 2^VB + slot; the slot order is packed in VB-bit fields.
        // Slots already in that order (as unsigned, DEAD_CELL is the largest) keep
        // it; the network runs when any lane of the wavefront needs it.
        constexpr int VB = PPT == 2 ? 1 : PPT == 4 ? 2 : PPT == 8 ? 3 : 4;
        using Visit = std::conditional_t<PPT == 16, uint64_t, uint32_t>;
        constexpr Visit IN_ORDER = [] {
            Visit v = 0;
            for (int q = 0; q < PPT; ++q) v |= (Visit)q << (VB * q);
            return v;
        }();
        Visit visit = IN_ORDER;
        bool ordered = true;
#pragma unroll
        for (int q = 1; q < PPT; ++q) ordered = ordered && (uint32_t)cst[q] >= (uint32_t)cst[q - 1];
        if (__ballot(!ordered) != 0ull) {
            visit = 0;
            uint32_t k[PPT];
#pragma unroll
            for (int q = 0; q < PPT; ++q)
                k[q] = (cst[q] == DEAD_CELL ? (0xffffffffu << VB) : (uint32_t)(cst[q] - first) << VB) | (uint32_t)q;
            sort_keys<PPT>(k);
#pragma unroll
            for (int q = 0; q < PPT; ++q) visit |= (Visit)(k[q] & ((1u << VB) - 1u)) << (VB * q);
        }
        // window [lo, hi] of cells this wavefront's deposit can touch: in a tile in
        // position order, the first lane's lowest and the last lane's highest cell;
        // checked, and reduced over the wavefront where that guess fails
        const int lane_lo = lane_any ? (int)lo_u - 1 : INT32_MAX;
        const int lane_hi = lane_any ? hi_s + 1 : INT32_MIN;
        int lo = __builtin_amdgcn_readfirstlane(lane_lo);
        int hi = __builtin_amdgcn_readlane(lane_hi, 63);
        if (__ballot(lane_lo < lo || lane_hi > hi) != 0ull) {
            lo = wave_min_i(lane_lo);
            hi = wave_max_i(lane_hi);
        }
        const bool any = lo <= hi;
        lo = any ? lo : 0;
        hi = any ? hi : -1;
        const bool use_lds = any && (hi - lo + 1) <= WW;
        const int span = use_lds ? (hi - lo + 1) : 0;
        for (int cc = lane; cc < span; cc += 64) {
            sJ[wid][cc] = 0ull;
            sH[wid][cc] = 0;
        }
        wave_sync();

        TileCtx T;
        T.step = step;
        T.item = ww.t;
        T.hist_out = hist_out;
        T.negative = (sp == 0 || sp == 2);
        T.inv_mass = (sp == 3) ? a.inv_mass_ion : 1.0f;
        T.gravity = a.gravity && any && ((double)lo <= L.atm_depth + 1.0 ||
                                         (double)(L.n_cells - 1 - hi) <= L.atm_depth + 1.0);
        unsigned long long* Jg = a.J + L.cell_base;
        int* Hg = hist_out + 4 * (size_t)L.cell_base + sp;
        // per-lane run accumulator over consecutive particles of one cell: deposits
        // (2^-28 cell) into cells key-1, key, key+1 and the new-cell counts of the same
        // three cells packed in 10-bit fields of hc
        int key = cc.cell;
        int jv0 = 0, jv1 = 0, jv2 = 0, hc = 0;
        // flush the lowest `ncells` cells of the run's three (all of them, or only
        // key-1 when the next run starts in key+1 and the other two carry over).  The
        // window holds the sums unsigned and unshifted and has room for the cells beyond
        // the walls, so that no bounds are tested and nothing is converted here; an outer
        // cell of a whole run that got nothing is skipped (not so 709 us on 40 uneven lines
        // and 394 on the line at the density limit instead of 696 and 389)
        auto flush_run = [&](int ncells) {
            const int jv[3] = {jv0, jv1, jv2};
            if (use_lds) {
                if (lane_any) {
                    unsigned long long* wj = &sJ[wid][key - 1 - lo];
                    int* wh = &sH[wid][key - 1 - lo];
#pragma unroll
                    for (int r = 0; r < 3; ++r) {
                        if (r >= ncells) continue;
                        const int hv = (hc >> (10 * r)) & 1023;
                        if (ncells == 3 && r != 1 && (jv[r] | hv) == 0) continue;
                        atomicAdd(wj + r, (unsigned long long)(long long)jv[r]);
                        atomicAdd(wh + r, hv);
                    }
                }
                return;
            }
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                const int cell = key - 1 + r;
                const int hv = (hc >> (10 * r)) & 1023;
                if (r < ncells && cell >= 0 && cell < L.n_cells) {
                    const long long j = (long long)(T.negative ? -jv[r] : jv[r]) << POS_TO_FIX;
                    if (j != 0) atomicAdd(&Jg[cell], (unsigned long long)j);
                    if (hv != 0) atomicAdd(&Hg[4 * (size_t)cell], hv);
                }
            }
        };
        float nonfinite = 0.0f;       // NaN once a momentum is not finite
        int n_alive = 0;
#pragma unroll 1
        for (int q = 0; q < PPT; ++q) {
            const int slot = (int)(visit >> (VB * q)) & ((1 << VB) - 1);
            const int c0 = sPc[wid][slot][lane];
            const bool alive = c0 != DEAD_CELL;
            if (alive && c0 != cc.cell) {
                if (c0 == key + 1) {
                    // slide the run one cell up: key and key+1 carry over
                    flush_run(1);
                    jv0 = jv1;
                    jv1 = jv2;
                    jv2 = 0;
                    hc >>= 10;
                } else {
                    flush_run(3);
                    jv0 = jv1 = jv2 = hc = 0;
                }
                cache_load<BACKEND>(cc, a, L, qmC, c0);
                key = c0;
            }
            float uq = sPu[wid][slot][lane];
            const float oq = sPo[wid][slot][lane];
            int c1, d, jm, j0, jp;
            float o1;
            bool gone;
            advance_particle<BACKEND>(a, L, T, cc, alive, line, sp, base + ib + slot, cc.cell, oq, uq, cnt, c1, o1,
                                      jm, j0, jp, d, gone, sW, a.mlp_bias);
            nonfinite = fmaf(uq, 0.0f, nonfinite);
            n_alive += __popcll(__ballot(alive));
            jv0 += jm;
            jv1 += j0;
            jv2 += jp;
            hc += alive ? (1 << (10 * (d + 1))) : 0;
            sPc[wid][slot][lane] = c1;
            sPo[wid][slot][lane] = gone ? 0.5f : o1;
            sPu[wid][slot][lane] = gone ? 0.0f : uq;
        }
        flush_run(3);
        cnt.pushed += lane == 0 ? n_alive : 0;
        cnt.pushed_ion += lane == 0 && sp == 3 ? n_alive : 0;
        if (nonfinite != nonfinite) set_error(&a.sc->err, -5);
        // write back (vector stores for full groups; never touch slots >= ncur, where
        // appended particles may be landing)
        if (PPT == 2 && nv == PPT) {
            *reinterpret_cast<int2*>(a.cell + base + ib) = make_int2(sPc[wid][0][lane], sPc[wid][1][lane]);
            *reinterpret_cast<float2*>(a.off + base + ib) = make_float2(sPo[wid][0][lane], sPo[wid][1][lane]);
            *reinterpret_cast<float2*>(a.u + base + ib) = make_float2(sPu[wid][0][lane], sPu[wid][1][lane]);
        } else if (nv == PPT) {
            int4* cp = reinterpret_cast<int4*>(a.cell + base + ib);
            float4* op = reinterpret_cast<float4*>(a.off + base + ib);
            float4* up = reinterpret_cast<float4*>(a.u + base + ib);
#pragma unroll
            for (int h = 0; h < PPT / 4; ++h) {
                cp[h] = make_int4(sPc[wid][4 * h][lane], sPc[wid][4 * h + 1][lane], sPc[wid][4 * h + 2][lane],
                                  sPc[wid][4 * h + 3][lane]);
                op[h] = make_float4(sPo[wid][4 * h][lane], sPo[wid][4 * h + 1][lane], sPo[wid][4 * h + 2][lane],
                                    sPo[wid][4 * h + 3][lane]);
                up[h] = make_float4(sPu[wid][4 * h][lane], sPu[wid][4 * h + 1][lane], sPu[wid][4 * h + 2][lane],
                                    sPu[wid][4 * h + 3][lane]);
            }
        } else {
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                if (q < nv) {
                    a.cell[base + ib + q] = sPc[wid][q][lane];
                    a.off[base + ib + q] = sPo[wid][q][lane];
                    a.u[base + ib + q] = sPu[wid][q][lane];
                }
            }
        }
        fetch(QUEUE ? next : ww.t + ww.stride);
        // flush the window
        wave_sync();
        for (int cc2 = lane; cc2 < span; cc2 += 64) {
            const int cell = lo + cc2;
            const long long sj = (long long)sJ[wid][cc2] << POS_TO_FIX;
            const int sh = sH[wid][cc2];
            if ((unsigned)cell < (unsigned)L.n_cells) {
                if (sj != 0) atomicAdd(&Jg[cell], (unsigned long long)(T.negative ? -sj : sj));
                if (sh != 0) atomicAdd(&Hg[4 * (size_t)cell], sh);
            }
        }
        wave_sync();
    }
    if (cur_line >= 0) counts_flush(a.counters, cur_line, cnt);
}

// the shapes the autotuner chooses from: 4, 8 or 16 particles per lane, and two
// deposit windows per backend
template __global__ void k_push<RICS_OFF, 4, 32, 0, 1>(PushArgs);
template __global__ void k_push<RICS_OFF, 8, 32, 0, 1>(PushArgs);
template __global__ void k_push<RICS_OFF, 16, 32, 0, 1>(PushArgs);
template __global__ void k_push<RICS_OFF, 8, 64, 0, 1>(PushArgs);
template __global__ void k_push<RICS_EXACT, 4, 32, 0, 1>(PushArgs);
template __global__ void k_push<RICS_EXACT, 8, 32, 0, 1>(PushArgs);
template __global__ void k_push<RICS_EXACT, 16, 32, 0, 1>(PushArgs);
template __global__ void k_push<RICS_EXACT, 8, 64, 0, 1>(PushArgs);
template __global__ void k_push<RICS_TABLE, 4, 128, 0, 1>(PushArgs);
template __global__ void k_push<RICS_TABLE, 8, 128, 0, 1>(PushArgs);
template __global__ void k_push<RICS_TABLE, 16, 128, 0, 1>(PushArgs);
template __global__ void k_push<RICS_TABLE, 8, 64, 0, 1>(PushArgs);
template __global__ void k_push<RICS_MLP, 4, 32, 0, 2>(PushArgs);
// parts of the default tile, for states whose tiles are too few to fill the chip
template __global__ void k_push<RICS_OFF, 4, 32, 0, 2>(PushArgs);
template __global__ void k_push<RICS_OFF, 2, 32, 0, 4>(PushArgs);
template __global__ void k_push<RICS_EXACT, 4, 32, 0, 2>(PushArgs);
template __global__ void k_push<RICS_EXACT, 2, 32, 0, 4>(PushArgs);
template __global__ void k_push<RICS_TABLE, 4, 128, 0, 2>(PushArgs);
template __global__ void k_push<RICS_TABLE, 2, 128, 0, 4>(PushArgs);
// the surrogate's states with lines on both sources: the table lines alone, the
// network lines alone
template __global__ void k_push<RICS_TABLE, 8, 128, 1, 1>(PushArgs);
template __global__ void k_push<RICS_MLP, 4, 32, 2, 2>(PushArgs);

// ---------------------------------------------------------------------------
// Photon conversion (Sec. 3): every recorded photon with E >= 2 m_e c^2 turns into
// an e-/e+ pair at gamma = eps/2 each where it converts -- at the emission point,
// or where the straight photon leaves the curved line by arcsin(2 m_e c^2/E) --
// if that point lies on the line and the cell's count at the start of the step
// is below n_max.  Float64 throughout: the member momenta are ill-conditioned in
// eps when eps/2 is close to 1.
// ---------------------------------------------------------------------------
// The records of all regions form one index space (regions in order); a block takes
// a chunk of consecutive records at a time, up to CONV_K per thread: as few as give
// every block one, for a chunk is a chain of dependent loads, scans and atomics and
// the blocks' chunks run side by side.  The slots of a chunk's pairs are reserved with
// one atomic per (block, line) on each allocation counter: those counters are single
// addresses that every block hits, and device-wide atomics on one address serialise.
// On a single line no record's line is looked for, and a chunk whose pairs all fit their
// segments needs no third scan.  Bound by the latency of that chain: k_append 9.3 us a
// step at a few thousand records on 512 cells, 13 us on a line with some 2e4 and 20 us on
// lines with some 1e5 (20, 26 and 34 us with CONV_K records a thread always, three scans
// a line and the two reservations one after the other).
constexpr int CONV_K = 4;
static_assert(PHOTON_REPL % 64 == 0 && PHOTON_REPL <= 256, "region fills: PHOTON_REPL / 64 per lane of one wave");

struct ConvRec {
    int line, cell;
    float off, up;
    uint64_t pid;
    bool valid, convert;
};

// The lab photon energy of an angled event in float64 (the arithmetic of
// angled_event); dir turns into the photon's direction along s, the lepton's sign
// times that of c + beta_e.
__device__ __forceinline__ double angled_photon(double gam, double q, double c, double& dir) {
    const double ge = gam / q;
    const double g2m1 = (ge - 1.0) * (ge + 1.0);
    const bool boost = g2m1 > 0.0;
    const double be = boost ? sqrt(g2m1) / ge : 0.0;
    const double omb = boost ? 1.0 / (ge * ge * (1.0 + be)) : 1.0;
    const double eg = (q - 1.0 / q) / (1.0 + sqrt(c * c + (1.0 - c) * (1.0 + c) / (q * q)));
    const double dopp = c >= 0.0 ? fma(be, c, 1.0) : fma(be, 1.0 + c, omb);
    if (c + be < 0.0) dir = -dir;
    return ge * eg * dopp;
}

__device__ __forceinline__ ConvRec convert_record(const ConvertArgs& a, const int32_t* hist_in, const PhotonRec& p,
                                                  bool valid) {
    ConvRec c;
    c.valid = valid;
    c.convert = false;
    c.line = valid ? p.line : INT32_MAX;
    c.cell = p.cell;
    c.off = p.off;
    c.up = 0.0f;
    c.pid = p.pid;
    if (!valid) return c;
    const LineDev& L = a.lines[p.line];
    const int n = L.n_cells;
    const double ud = (double)p.u_pre;
    const double qd = sqrt(1.0 + 2.0 * (double)p.b);
    double dir = ud >= 0.0 ? 1.0 : -1.0;
    const double eps = p.mu == 0.0f ? sqrt(1.0 + ud * ud) * (2.0 * (double)p.b) / (qd * (1.0 + qd))
                                    : angled_photon(sqrt(1.0 + ud * ud), qd, (double)p.mu, dir);
    bool ok = true;
    if (a.conversion != 0) {
        const double* rc = a.rc_nodes + L.node_base + p.cell;
        const double rcx = fma((double)p.off, rc[1] - rc[0], rc[0]);
        const double sp = (double)p.cell + (double)p.off + dir * rcx * L.inv_ds * asin(fmin(2.0 / eps, 1.0));
        ok = (sp >= 0.0) && (sp < (double)n);
        c.cell = ok ? (int)floor(sp) : 0;
        c.off = ok ? (float)(sp - (double)c.cell) : 0.0f;
        if (c.off >= 1.0f) { c.off = 0.0f; c.cell += 1; ok = ok && c.cell < n; }
    }
    if (ok) {
        const int* hc = hist_in + 4 * (size_t)(L.cell_base + c.cell);
        c.convert = (float)(hc[0] + hc[1] + hc[2] + hc[3]) < L.nmax;
        const double gp = 0.5 * eps;
        c.up = (float)(dir * sqrt(fmax((gp - 1.0) * (gp + 1.0), 0.0)));
    }
    return c;
}

// block-wide sum and exclusive prefix (in thread order) of one int per thread
__device__ __forceinline__ int block_scan(int v, int& total, int* s_part) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) s_part[w] = inc;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int pk = s_part[k];
        before += (k < w) ? pk : 0;
        total += pk;
    }
    __syncthreads();
    return before + inc - v;
}

__device__ __forceinline__ void convert_photons(const ConvertArgs& a, int blk, int nblk) {
    __shared__ int s_pref[PHOTON_REPL + 1];    // exclusive prefix of the region fills
    __shared__ int s_part[4];
    __shared__ int s_base[2];
    const uint64_t step = a.sc->step;
    const int32_t* hist_in = (step & 1) ? a.hist[1] : a.hist[0];
    int32_t* hist_out = (step & 1) ? a.hist[0] : a.hist[1];
    const int lane = threadIdx.x & 63;
    constexpr int RPL = PHOTON_REPL / 64;      // regions per lane
    if (threadIdx.x < 64) {
        // after an error there is nothing to convert, for the whole block (see block_stopped)
        const bool stopped = a.sc->err != 0;
        int f[RPL], sum = 0;
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            f[k] = stopped ? 0 : min(a.n_photons[lane * RPL + k], a.photon_region);
            sum += f[k];
        }
        int inc = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(inc, o, 64);
            if (lane >= o) inc += t;
        }
        int run = inc - sum;
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            s_pref[lane * RPL + k] = run;
            run += f[k];
        }
        if (lane == 63) s_pref[PHOTON_REPL] = inc;
    }
    __syncthreads();
    const int total = s_pref[PHOTON_REPL];
    const int per = max(1, min(CONV_K, (total - 1) / (nblk * 256) + 1));     // records per thread
    const int chunk = 256 * per;
    const bool one_line = a.n_lines == 1;
    for (int c0 = blk * chunk; c0 < total; c0 += nblk * chunk) {
        ConvRec rec[CONV_K];
#pragma unroll
        for (int k = 0; k < CONV_K; ++k) {
            const int g = c0 + k * 256 + (int)threadIdx.x;
            const bool valid = k < per && g < total;
            PhotonRec p{};
            if (valid) {
                int lo = 0, hi = PHOTON_REPL;          // s_pref[lo] <= g < s_pref[hi]
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_pref[mid] <= g) lo = mid; else hi = mid;
                }
                p = a.photons[(size_t)lo * a.photon_region + (g - s_pref[lo])];
            }
            rec[k] = convert_record(a, hist_in, p, valid);
        }
        // one reservation per line present in the chunk, lowest line first
        while (true) {
            int gl = 0;
            if (!one_line) {
                int m = INT32_MAX;
#pragma unroll
                for (int k = 0; k < CONV_K; ++k) m = min(m, rec[k].line);
                m = wave_min_i(m);
                if (lane == 0) s_part[threadIdx.x >> 6] = m;
                __syncthreads();
                gl = min(min(s_part[0], s_part[1]), min(s_part[2], s_part[3]));
                __syncthreads();
                if (gl == INT32_MAX) break;
            }
            int mine = 0, seen = 0;
#pragma unroll
            for (int k = 0; k < CONV_K; ++k) {
                mine += (rec[k].line == gl && rec[k].convert) ? 1 : 0;
                seen += (rec[k].line == gl) ? 1 : 0;
            }
            int nconv = 0;
            const int before = block_scan(mine, nconv, s_part);
            int nseen = min(chunk, total - c0);
            if (!one_line) block_scan(seen, nseen, s_part);
            // (the two round trips side by side, from two wavefronts)
            if (threadIdx.x == 0) s_base[0] = nconv > 0 ? atomicAdd(&a.alloc[4 * gl + 0], nconv) : 0;
            if (threadIdx.x == 64) s_base[1] = nconv > 0 ? atomicAdd(&a.alloc[4 * gl + 1], nconv) : 0;
            __syncthreads();
            const int base_e = s_base[0] + before, base_p = s_base[1] + before;
            const bool fits = slots_in(s_base[0], nconv, a.seg_cap[4 * gl + 0]) &&
                              slots_in(s_base[1], nconv, a.seg_cap[4 * gl + 1]);
            __syncthreads();
            int made = 0, j = 0;
#pragma unroll
            for (int k = 0; k < CONV_K; ++k) {
                if (rec[k].line != gl) continue;
                if (rec[k].convert) {
                    const int se = base_e + j, spp = base_p + j;
                    ++j;
                    const bool e_ok = slot_in(se, a.seg_cap[4 * gl + 0]), p_ok = slot_in(spp, a.seg_cap[4 * gl + 1]);
                    if (!e_ok || !p_ok) set_error(&a.sc->err, -3);
                    const uint4 wc = philox4x32_10(make_uint4((uint32_t)step, (uint32_t)rec[k].pid,
                                                              (uint32_t)(rec[k].pid >> 32), STREAM_CHILD),
                                                   a.key0, a.key1);
                    if (e_ok) {
                        const int64_t q = a.seg_base[4 * gl + 0] + se;
                        a.cell[q] = rec[k].cell; a.off[q] = rec[k].off; a.u[q] = rec[k].up;
                        a.id[q] = id_from_words(wc.x, wc.y);
                    }
                    if (p_ok) {
                        const int64_t q = a.seg_base[4 * gl + 1] + spp;
                        a.cell[q] = rec[k].cell; a.off[q] = rec[k].off; a.u[q] = rec[k].up;
                        a.id[q] = id_from_words(wc.z, wc.w);
                    }
                    if (e_ok && p_ok) {
                        const LineDev& L = a.lines[gl];
                        int* ho = hist_out + 4 * (size_t)(L.cell_base + rec[k].cell);
                        atomicAdd(&ho[0], 1);
                        atomicAdd(&ho[1], 1);
                        atomicAdd(&a.pair_step[L.cell_base + rec[k].cell], 1);
                        ++made;
                    }
                }
                rec[k].line = INT32_MAX;      // done with this record
            }
            int n_made = nconv;
            if (!fits) block_scan(made, n_made, s_part);
            if (threadIdx.x == 0) {
                const size_t rep = ((size_t)gl * CNT_REPL + (blk & (CNT_REPL - 1))) * NCOUNT;
                if (n_made) atomicAdd(&a.counters[rep + 1], (unsigned long long)n_made);
                if (nseen - n_made) atomicAdd(&a.counters[rep + 2], (unsigned long long)(nseen - n_made));
            }
            if (one_line) break;
        }
    }
}

// ---------------------------------------------------------------------------
// Atmosphere (Appendix B.1): every layer cell is refilled to its hydrostatic
// target with co-located (e-, ion) pairs; one wavefront per layer cell.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void refill_atmosphere(const AtmArgs& a, int blk, int nblk) {
    if (a.sc->err != 0) return;
    const uint64_t step = a.sc->step;
    int32_t* hist_out = a.hist[(step & 1) ^ 1];
    const int lane = threadIdx.x & 63;
    const int wglob = (blk * blockDim.x + threadIdx.x) >> 6;
    const int nw = (nblk * blockDim.x) >> 6;
    for (int e = wglob; e < a.n_layer; e += nw) {
        const int g = a.layer_cell[e];         // global cell
        const int line = a.layer_line[e];
        const int target = a.layer_target[e];
        int* h = hist_out + 4 * (size_t)g;
        const int have = min(h[2], h[3]);
        const int D = max(target - have, 0);
        if (D == 0) continue;
        const LineDev& L = a.lines[line];
        const int segE = 4 * line + 2, segI = 4 * line + 3;
        int baseE = 0, baseI = 0;
        if (lane == 0) {
            baseE = atomicAdd(&a.alloc[segE], D);
            baseI = atomicAdd(&a.alloc[segI], D);
        }
        baseE = __shfl(baseE, 0, 64);
        baseI = __shfl(baseI, 0, 64);
        if (!slots_in(baseE, D, a.seg_cap[segE]) || !slots_in(baseI, D, a.seg_cap[segI])) {
            if (lane == 0) set_error(&a.sc->err, -3);
            continue;
        }
        const int c = g - L.cell_base;
        for (int kk = lane; kk < D; kk += 64) {
            const uint4 wa = philox4x32_10(make_uint4((uint32_t)step, (uint32_t)g, (uint32_t)kk, STREAM_ATM_A), a.key0, a.key1);
            const uint4 wb = philox4x32_10(make_uint4((uint32_t)step, (uint32_t)g, (uint32_t)kk, STREAM_ATM_B), a.key0, a.key1);
            const uint4 wc = philox4x32_10(make_uint4((uint32_t)step, (uint32_t)g, (uint32_t)kk, STREAM_ATM_ID), a.key0, a.key1);
            const float off = uniform24(wa.x);
            const float ue = a.sig_e * sqrtf(-2.0f * logf(uniform24_open0(wa.y))) * cospif(2.0f * uniform24(wa.z));
            const float ui = a.sig_i * sqrtf(-2.0f * logf(uniform24_open0(wb.x))) * cospif(2.0f * uniform24(wb.y));
            const int64_t ke = a.seg_base[segE] + baseE + kk;
            const int64_t ki = a.seg_base[segI] + baseI + kk;
            a.cell[ke] = c; a.off[ke] = off; a.u[ke] = ue; a.id[ke] = id_from_words(wc.x, wc.y);
            a.cell[ki] = c; a.off[ki] = off; a.u[ki] = ui; a.id[ki] = id_from_words(wc.z, wc.w);
        }
        if (lane == 0) {
            h[2] += D;
            h[3] += D;
            atomicAdd(&a.counters[((size_t)line * CNT_REPL + (blk & (CNT_REPL - 1))) * NCOUNT + 7],
                      (unsigned long long)D);
        }
    }
}

// The step's appends in one launch: blocks [0, conv_blocks) convert the recorded
// photons into pairs (species 0 and 1), the rest refill the atmosphere (species 2
// and 3).  The two touch different segments and different species counts, so they
// run side by side.
__global__ __launch_bounds__(256) void k_append(ConvertArgs ca, AtmArgs aa, int conv_blocks) {
    if ((int)blockIdx.x < conv_blocks) convert_photons(ca, blockIdx.x, conv_blocks);
    else refill_atmosphere(aa, blockIdx.x - conv_blocks, gridDim.x - conv_blocks);
}

// Block-wide (256 threads) exclusive scan of one int; writes the block total.
__device__ __forceinline__ int block_excl_scan(int v, int& total) {
    __shared__ int sWave[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) sWave[w] = inc;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = sWave[i];
        before += i < w ? t : 0;
        total += t;
    }
    __syncthreads();
    return before + inc - v;
}

// ---------------------------------------------------------------------------
// Per-step bookkeeping shared by k_field and k_plan: live counts <- allocation
// counters (after a sort, its counts; clamped to capacity), tile plan of the next push.
// Nothing (false) after an error.
// ---------------------------------------------------------------------------
__device__ bool bookkeeping(const BookArgs& b) {
    const int nseg = b.nseg;
    const int per = (nseg + 255) / 256;
    const int s0 = threadIdx.x * per, s1 = min(s0 + per, nseg);
    auto count = [&](int s) { return min(b.new_count ? b.new_count[s] : b.alloc[s], b.seg_cap[s]); };
    // did the annihilation find the particles in the cells over the limit that are counted
    // there?  (asked by the second wavefront while the first reads the error word; the
    // scan's barriers make both known to the block, see block_stopped)
    __shared__ int s_err;
    __shared__ uint32_t s_differ;
    if (threadIdx.x == 0) s_err = b.sc->err;
    if (threadIdx.x >= 64 && threadIdx.x < 128) {
        const int lane = threadIdx.x & 63;
        const uint32_t differ = wave_sum_last(b.ann_tags && lane < ANN_TAGS ? b.ann_tags[32 * lane] : 0u);
        if (lane == 63) s_differ = differ;
    }
    int sum = 0, n_last = 0;
    for (int s = s0; s < s1; ++s) {
        n_last = count(s);
        sum += tiles_of(n_last, b.tile);
    }
    int total;
    int run = block_excl_scan(sum, total);
    if (s_err != 0) return false;
    if (s_differ != 0u) {
        if (threadIdx.x == 0) set_error(&b.sc->err, -4);
        return false;
    }
    if (b.n_photons && threadIdx.x < PHOTON_REPL) b.n_photons[threadIdx.x] = 0;
    if (threadIdx.x == 0) b.queue[0] = 0;
    for (int s = s0; s < s1; ++s) {
        // (one segment per thread up to 256 segments: its count is still in a register)
        const int n = per == 1 ? n_last : count(s);
        b.n_cur[s] = n;
        b.alloc[s] = n;
        b.tile_prefix[s] = run;
        run += tiles_of(n, b.tile);
    }
    if (threadIdx.x == 255) {
        b.tile_prefix[nseg] = total;
        b.sc->tiles = total;
        if (b.new_count) b.sc->live = b.live;
    }
    return true;
}

// Bookkeeping kernel of every step (and after init, sort, set_particles): one block.
__global__ __launch_bounds__(256) void k_plan(BookArgs b, int advance_step) {
    bookkeeping(b);
    if (advance_step && threadIdx.x == 0 && b.sc->err == 0) b.sc->step += 1;
}

// ---------------------------------------------------------------------------
// Pair annihilation at the density limit (Sec. 3: pairs annihilate where the
// total density approaches n_max, which keeps the skin depth resolved; the paper
// gives no mechanics, so these are readings).  A cell whose end-of-step count N
// of all particles exceeds n_max loses k = min(N-, N+, ceil((N - n_max)/2))
// e-/e+ pairs (species 0 and 1): the k of each species with the smallest
// (key, id), key the 64-bit Philox draw (step, id, STREAM_ANNIH), so the choice
// does not depend on where the particles sit in memory.  Each pair annihilates
// as if its positron first moved to its electron: the cell's face current gains
// sum q(x-) - sum q(x+) in the deposit's fixed point (the same quantised
// positions the push deposits from), and the neutral pair leaves no charge.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t annih_key(uint64_t step, uint64_t id, uint32_t k0, uint32_t k1) {
    const uint4 w = philox4x32_10_wide(make_uint4((uint32_t)step, (uint32_t)id, (uint32_t)(id >> 32), STREAM_ANNIH),
                                       k0, k1);
    return ((uint64_t)w.y << 32) | (uint64_t)w.x;
}

// The gather records only the candidates whose key's high word is at most the
// cell's threshold, which admits lambda = k + 8 k^1/2 + 20 of the m keys of the
// smaller species on average (the keys are uniform): fewer than k of them pass with
// a probability below 1e-12 a cell, and k_field then searches the segment for the whole
// cell.  Keys are uniform because ids differ: a program that sets the same id many times
// could have every cell searched, hours of work on a long line.  So after ANN_SEARCHES
// searches a state records every candidate from its next step on, and a cell that would
// have been the next one to search keeps its pairs for that step.
__device__ __forceinline__ uint32_t annih_threshold(int k, int m) {
    const float lam = (float)k + 8.0f * sqrtf((float)k) + 20.0f;
    return lam < (float)m ? (uint32_t)(lam / (float)m * 4294967040.0f) : 0xffffffffu;
}

// Adds a wavefront's tags (see cell_tag) to their sum.
__device__ __forceinline__ void add_tags(uint32_t* tags, uint32_t v) {
    if (__ballot(v != 0u) == 0ull) return;
    const uint32_t sum = wave_sum_last(v);
    if ((threadIdx.x & 63) == 63 && sum != 0u)
        atomicAdd(&tags[32 * ((blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) % ANN_TAGS)], sum);
}

// Every cell's k from its end-of-step counts, and for the cells over the limit a
// run of candidate records (room for all their e- then their e+), one allocation
// per block.
__global__ __launch_bounds__(256) void k_annih_plan(AnnihArgs a) {
    __shared__ int s_err;                 // (read once for the block, see block_stopped)
    if (threadIdx.x == 0) s_err = a.sc->err;
    const uint64_t step = a.sc->step;
    const int32_t* hist_out = a.hist[(step & 1) ^ 1];
    const bool all = a.sc->ann_all != 0;
    __shared__ int s_base;
    for (int g0 = blockIdx.x * 256; g0 < a.n_total; g0 += gridDim.x * 256) {
        const int g = g0 + (int)threadIdx.x;
        int k = 0, need = 0, h0 = 0, h1 = 0;
        if (g < a.n_total) {
            const int* h = hist_out + 4 * (size_t)g;
            h0 = h[0];
            h1 = h[1];
            const int N = h0 + h1 + h[2] + h[3];
            const double nmax = (double)a.lines[a.cell_line[g]].nmax;
            if ((double)N > nmax) k = (int)fmin(fmin((double)h0, (double)h1), ceil(((double)N - nmax) * 0.5));
            need = k > 0 ? h0 + h1 : 0;
        }
        add_tags(a.ann_tags, k > 0 ? 0u - (uint32_t)h0 * cell_tag(g, 0) - (uint32_t)h1 * cell_tag(g, 1) : 0u);
        int total = 0;
        const int excl = block_excl_scan(need, total);
        if (s_err != 0) return;
        if (total > 0 && threadIdx.x == 0) {
            s_base = atomicAdd(&a.ann_ctl[0], total);
            atomicOr(&a.ann_ctl[1], 1);
        }
        __syncthreads();
        if (k > 0) {
            const int64_t off = (int64_t)s_base + excl;
            if (off + need > a.cand_cap || off + need > (int64_t)INT32_MAX) {
                set_error(&a.sc->err, -3);
                k = 0;
            } else {
                a.ann_off[g] = (int)off;
                a.ann_fill[2 * (size_t)g] = 0;
                a.ann_fill[2 * (size_t)g + 1] = 0;
            }
        }
        if (g < a.n_total) {
            a.ann_k[g] = k;
            a.ann_thr[g] = k > 0 ? (all ? 0xffffffffu : annih_threshold(k, min(h0, h1))) : 0u;
        }
        __syncthreads();
    }
}

__device__ __forceinline__ long long wave_sum_ll(long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t w = __shfl_xor(v, o, 64);
        v = w < v ? w : v;
    }
    return v;
}

// Candidates per lane held in registers by the register selection (at most
// 64 * ANNIH_KPL candidates of a species); larger cells take the radix select
// over the records in memory.
constexpr int ANNIH_KPL = 8;
constexpr int ANNIH_EXTRACT_K = 8;

// The `k` smallest (key, id) of one species' m candidates, with the keys in
// registers: for k <= ANNIH_EXTRACT_K extracted one at a time by wave-wide
// minima, else an 8-bit radix select on a per-wavefront LDS histogram `hist`
// (256 ints) followed by the keys below the k-th.  Ids are read only where keys
// tie exactly.  Bit j of the result: the lane's j-th candidate (record
// lane + 64 j) is taken.
__device__ uint32_t annih_select_regs(const AnnihArgs& a, int64_t rec0, int64_t base, int m, int k, int* hist) {
    const int lane = threadIdx.x & 63;
    uint64_t key[ANNIH_KPL];
#pragma unroll
    for (int j = 0; j < ANNIH_KPL; ++j) {
        const int r = lane + 64 * j;
        key[j] = r < m ? a.cand_key[rec0 + r] : ~0ull;
    }
    auto valid = [&](int j) { return lane + 64 * j < m; };
    uint32_t taken = 0;
    // take `n` more of the untaken candidates whose key is kmin, smallest id first
    auto take_ties = [&](uint64_t kmin, int n) {
        for (int t = 0; t < n; ++t) {
            uint64_t idmin = ~0ull;
            int jmin = -1;
#pragma unroll
            for (int j = 0; j < ANNIH_KPL; ++j) {
                if (!((taken >> j) & 1u) && valid(j) && key[j] == kmin) {
                    const uint64_t id = a.id[base + a.cand_slot[rec0 + lane + 64 * j]];
                    if (id < idmin) { idmin = id; jmin = j; }
                }
            }
            const uint64_t wid = wave_min_u64(idmin);
            if (jmin >= 0 && idmin == wid) taken |= 1u << jmin;
        }
    };
    if (k <= ANNIH_EXTRACT_K) {
        for (int round = 0; round < k; ++round) {
            uint64_t mine = ~0ull;
#pragma unroll
            for (int j = 0; j < ANNIH_KPL; ++j)
                if (!((taken >> j) & 1u) && valid(j) && key[j] < mine) mine = key[j];
            const uint64_t kmin = wave_min_u64(mine);
            int ties = 0;
#pragma unroll
            for (int j = 0; j < ANNIH_KPL; ++j) ties += (!((taken >> j) & 1u) && valid(j) && key[j] == kmin) ? 1 : 0;
            if (wave_sum_i(ties) == 1) {
#pragma unroll
                for (int j = 0; j < ANNIH_KPL; ++j)
                    if (valid(j) && key[j] == kmin) taken |= 1u << j;
            } else {
                take_ties(kmin, 1);
            }
        }
        return taken;
    }
    // radix select, most significant byte first: kth ends as the k-th smallest key
    uint64_t kth = 0;
    int want = k;
    for (int p = 7; p >= 0; --p) {
        const int sh = 8 * p;
        for (int i = lane; i < 256; i += 64) hist[i] = 0;
        wave_sync();
#pragma unroll
        for (int j = 0; j < ANNIH_KPL; ++j) {
            const bool match = valid(j) && (p == 7 || (key[j] >> (sh + 8)) == (kth >> (sh + 8)));
            if (match) atomicAdd(&hist[(int)((key[j] >> sh) & 255ull)], 1);
        }
        wave_sync();
        const int c0 = hist[4 * lane], c1 = hist[4 * lane + 1], c2 = hist[4 * lane + 2], c3 = hist[4 * lane + 3];
        const int t = c0 + c1 + c2 + c3;
        int inc = t;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(inc, o, 64);
            if (lane >= o) inc += v;
        }
        const int excl = inc - t;
        const unsigned long long hb = __ballot(excl < want && want <= inc);
        const int L = __ffsll((long long)hb) - 1;
        int d = 0, below = excl;
        if (lane == L) {
            const int w = want - excl;
            if (w <= c0) { d = 0; }
            else if (w <= c0 + c1) { d = 1; below += c0; }
            else if (w <= c0 + c1 + c2) { d = 2; below += c0 + c1; }
            else { d = 3; below += c0 + c1 + c2; }
        }
        d = __shfl(d, L, 64);
        below = __shfl(below, L, 64);
        kth |= (uint64_t)(4 * L + d) << sh;
        want -= below;
        wave_sync();
    }
    int eq = 0;
#pragma unroll
    for (int j = 0; j < ANNIH_KPL; ++j) {
        if (valid(j) && key[j] < kth) taken |= 1u << j;
        eq += (valid(j) && key[j] == kth) ? 1 : 0;
    }
    if (wave_sum_i(eq) == want) {
#pragma unroll
        for (int j = 0; j < ANNIH_KPL; ++j)
            if (valid(j) && key[j] == kth) taken |= 1u << j;
    } else {
        take_ties(kth, want);
    }
    return taken;
}

// Removes the particle in a slot; returns its quantised offset (2^-28 cell).
__device__ __forceinline__ long long annih_remove(const AnnihArgs& a, int64_t kidx) {
    const long long q = (long long)(int)(a.off[kidx] * POS_SCALE);
    a.cell[kidx] = DEAD_CELL;
    a.off[kidx] = 0.5f;
    a.u[kidx] = 0.0f;
    return q;
}

// Records every e- (s = 0) or e+ (s = 1) of local cell c of a segment, where the
// gather's threshold let fewer than k through; returns how many.
__device__ __forceinline__ int annih_record_all(const AnnihArgs& a, uint64_t step, int seg, int c, int64_t rec0, int room) {
    const int lane = threadIdx.x & 63;
    const int n = min(a.alloc[seg], a.seg_cap[seg]);
    const int64_t base = a.seg_base[seg];
    int found = 0;
    for (int64_t i0 = 0; i0 < n; i0 += 64) {
        const int64_t i = i0 + lane;
        const bool mine = i < n && a.cell[base + i] == c;
        const unsigned long long m = __ballot(mine);
        const int r = found + __popcll(m & ((1ull << lane) - 1ull));
        if (mine && r < room) {
            a.cand_key[rec0 + r] = annih_key(step, a.id[base + i], a.key0, a.key1);
            a.cand_slot[rec0 + r] = (int)i;
        }
        found += __popcll(m);
    }
    __threadfence();                     // the records are read back by other lanes of the wavefront
    return found;
}

__device__ __forceinline__ uint32_t lane_word(uint32_t v, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}

// Whether this lane's key (lane < m) is among the k smallest (key, id) of m <= 64
// records: its rank by one comparison of the high words with every other key's,
// broadcast from its lane through a scalar register -- no reduction over the
// wavefront, and one load per lane in all.  If exactly k lanes rank below k these are
// the k smallest; otherwise equal high words lie around the k-th, and the whole keys
// and the ids decide.
__device__ __forceinline__ bool annih_rank64(const AnnihArgs& a, uint64_t key, int slot, int64_t base, int m, int k) {
    const int lane = threadIdx.x & 63;
    const uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32);
    int rank = 0;
    for (int i = 0; i < m; ++i) rank += lane_word(hi, i) < hi ? 1 : 0;
    bool take = lane < m && rank < k;
    if (__popcll(__ballot(take)) != k) {
        const uint64_t id = lane < m ? a.id[base + slot] : ~0ull;
        const uint32_t il = (uint32_t)id, ih = (uint32_t)(id >> 32);
        rank = 0;
        for (int i = 0; i < m; ++i) {
            const uint64_t ki = (uint64_t)lane_word(hi, i) << 32 | lane_word(lo, i);
            const uint64_t di = (uint64_t)lane_word(ih, i) << 32 | lane_word(il, i);
            rank += (ki < key || (ki == key && di < id)) ? 1 : 0;
        }
        take = lane < m && rank < k;
    }
    return take;
}

// What k_field knows of a cell over the limit.
struct AnnihCell {
    int g, k, line;
    int h0, h1;          // its e- and e+
    int r0, r1;          // ... of which the gather recorded
    int off;             // first record
};

// One wavefront removes a cell's k annihilating pairs (every lane calls it with the
// same cell): the k of each species with the smallest (key, id).  Up to 64 records of
// a species -- the thresholds leave about k + 8 k^1/2 + 20 of them -- one per lane
// and ranked; up to 512 in registers (annih_select_regs); beyond, a
// most-significant-bit-first radix select over the records in memory.  Returns (to
// every lane) the annihilation current in the deposit's units (2^-28 cell); the
// caller adds it to J[g] and takes the pairs removed (k, or none where the searches are
// used up) off the cell's e-/e+ counts.  Latency-bound: two
// dependent round trips per cell, and the removed particles' scattered lines.  With
// every candidate recorded and k wave-wide minima per species k_field took 57 us on
// a 512-cell line, 51 us on 9,973 cells and 92 us on 65,536 (600 per cell); 21, 24
// and 71 us now.
__device__ long long annihilate_cell(const AnnihArgs& a, const AnnihCell& c, uint64_t step, int* hist, int& removed) {
    const int lane = threadIdx.x & 63;
    const int k = c.k;
    removed = k;
    int m[2] = {c.r0, c.r1};
    if (m[0] > c.h0 || m[1] > c.h1) {
        if (lane == 0) set_error(&a.sc->err, -4);
        return 0;
    }
    if (m[0] < k || m[1] < k) {
        int n = 0;
        if (lane == 0) n = atomicAdd(&a.ann_ctl[3], 1);
        if (__builtin_amdgcn_readfirstlane(n) >= ANN_SEARCHES) {
            if (lane == 0) a.sc->ann_all = 1;
            removed = 0;
            return 0;
        }
        const int cl = c.g - a.lines[c.line].cell_base;
        for (int s = 0; s < 2; ++s) {
            if (m[s] >= k) continue;
            const int h = s ? c.h1 : c.h0;
            m[s] = annih_record_all(a, step, 4 * c.line + s, cl, (int64_t)c.off + (s ? c.h0 : 0), h);
            if (m[s] != h) {
                if (lane == 0) set_error(&a.sc->err, -4);
                return 0;
            }
        }
    }
    const int64_t rec[2] = {(int64_t)c.off, (int64_t)c.off + c.h0};
    const int64_t base[2] = {a.seg_base[4 * c.line], a.seg_base[4 * c.line + 1]};
    long long dq = 0;
    if (m[0] <= 64 && m[1] <= 64) {
        uint64_t key[2];
        int slot[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            key[s] = lane < m[s] ? a.cand_key[rec[s] + lane] : ~0ull;
            slot[s] = lane < m[s] ? a.cand_slot[rec[s] + lane] : 0;
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (annih_rank64(a, key[s], slot[s], base[s], m[s], k)) {
                const long long q = annih_remove(a, base[s] + slot[s]);
                dq += s == 0 ? q : -q;
            }
        }
        return wave_sum_ll(dq);
    }
    for (int s = 0; s < 2; ++s) {
        const int ms = m[s];
        const int64_t rec0 = rec[s];
        if (ms <= 64 * ANNIH_KPL) {
            const uint32_t taken = annih_select_regs(a, rec0, base[s], ms, k, hist);
#pragma unroll
            for (int j = 0; j < ANNIH_KPL; ++j) {
                if ((taken >> j) & 1u) {
                    const long long q = annih_remove(a, base[s] + a.cand_slot[rec0 + lane + 64 * j]);
                    dq += s == 0 ? q : -q;
                }
            }
            continue;
        }
        uint64_t kth = 0;
        int want = k;                 // rank sought among the keys that match kth so far
        for (int b = 63; b >= 0; --b) {
            const uint64_t above = b == 63 ? 0ull : (~0ull << (b + 1));
            int n0 = 0;
            for (int r = lane; r < ms; r += 64) {
                const uint64_t key = a.cand_key[rec0 + r];
                n0 += ((key & above) == kth && ((key >> b) & 1ull) == 0ull) ? 1 : 0;
            }
            n0 = wave_sum_i(n0);
            if (want > n0) {
                want -= n0;
                kth |= 1ull << b;
            }
        }
        // kth is the k-th smallest key; `want` of the keys equal to it are taken
        for (int r = lane; r < ms; r += 64) {
            const uint64_t key = a.cand_key[rec0 + r];
            const int slot = a.cand_slot[rec0 + r];
            bool take = key < kth;
            if (key == kth) {
                const uint64_t id = a.id[base[s] + slot];
                int below = 0;
                for (int r2 = 0; r2 < ms; ++r2)
                    below += (a.cand_key[rec0 + r2] == kth && a.id[base[s] + a.cand_slot[rec0 + r2]] < id) ? 1 : 0;
                take = below < want;
            }
            if (take) {
                const long long q = annih_remove(a, base[s] + slot);
                dq += s == 0 ? q : -q;
            }
        }
    }
    return wave_sum_ll(dq);
}

// Ampere's law with the static twist current (Sec. 3): E -= 4 pi (j - j_twist),
// plus time averages and the reset of the step's accumulators.  A block of its own does
// the step's bookkeeping (live counts, the next push's tile plan) and advances the
// step counter; the cells read the running step from the copy the push left.
__global__ __launch_bounds__(256) void k_field(FieldArgs f, BookArgs b) {
    // One block plans the next push and advances the step counter, beside the cells' blocks
    // rather than before one of them (none of them reads what it writes, but for the
    // allocation counters, which annih_record_all clamps to the same value that they are
    // given here): the last one, or, where the chip holds the grid only in rounds, the first,
    // so that its chain of round trips does not come after theirs (380,000 cells in a quiet
    // step 17.4 us, 19.7 as the last; 512 cells 0.25 us a step the other way).
    const int nb = gridDim.x - 1;
    const int block = nb >= FIELD_ROUND ? (int)blockIdx.x - 1 : (int)blockIdx.x == nb ? -1 : (int)blockIdx.x;
    // (it asks for itself, all its wavefronts together)
    if (block >= 0 && f.sc->err != 0) return;
    const uint64_t step = f.sc->step_field;
    const int n = f.n_total;
    const int hin = (int)(step & 1);
    int* hist_in = f.hist[hin];
    int* hist_out = f.hist[hin ^ 1];
    const bool averaging = f.avg_start >= 0 && step >= (uint64_t)f.avg_start;
    if (block < 0) {
        if (!bookkeeping(b)) return;
        if (threadIdx.x == 0) {
            if (b.sc->err == 0) b.sc->step += 1;
            if (f.annihilation) {
                // the plan of the next step allocates from zero (no other block reads these)
                f.an.ann_ctl[0] = 0;
                f.an.ann_ctl[1] = 0;
            }
            if (averaging) f.avg_count[0] += 1;
        }
        return;
    }
    // Each wavefront takes cpw consecutive cells per iteration: all 64 lanes, or, in a
    // step where some cell is over the limit, as few as spread the cells over the
    // grid's wavefronts, at most 4: a wavefront runs its selections one after another
    // (with 64 cells a wavefront most of the grid's blocks find no cells).
    __shared__ int sHist[4][256];            // per wavefront: the radix histogram of the selection
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int wpb = blockDim.x >> 6;
    const int nw = nb * wpb;
    const int cpw = (f.annihilation && f.an.ann_ctl[2] != 0) ? max(1, min(4, (n + nw - 1) / nw)) : 64;
    for (int gw = (block * wpb + wid) * cpw; gw < n; gw += nw * cpw) {
        const int g = gw + lane;
        const bool own = lane < cpw && g < n;
        long long dJ = 0;        // this lane's cell: annihilation current and pairs removed
        int k_own = 0;
        if (f.annihilation) {
            // this wavefront's cells over the limit, one at a time, before their Ampere;
            // what their selections need is read for all of them at once
            const int k = own ? f.an.ann_k[g] : 0;
            unsigned long long m = __ballot(k > 0);
            if (m != 0ull) {
                const bool over = k > 0;
                const int line = over ? f.cell_line[g] : 0;
                const int h0 = over ? hist_out[4 * (size_t)g] : 0;
                const int h1 = over ? hist_out[4 * (size_t)g + 1] : 0;
                const int r0 = over ? f.an.ann_fill[2 * (size_t)g] : 0;
                const int r1 = over ? f.an.ann_fill[2 * (size_t)g + 1] : 0;
                const int off = over ? f.an.ann_off[g] : 0;
                while (m != 0ull) {
                    const int lead = __ffsll((long long)m) - 1;
                    m &= m - 1ull;
                    auto of = [&](int v) { return __builtin_amdgcn_readlane(v, lead); };
                    const AnnihCell c{gw + lead, of(k), of(line), of(h0), of(h1), of(r0), of(r1), of(off)};
                    int removed;
                    const long long d = annihilate_cell(f.an, c, step, sHist[wid], removed);
                    if (lane == lead) {
                        dJ = d;
                        k_own = removed;
                    }
                }
                if (k_own > 0) {
                    hist_out[4 * (size_t)g] -= k_own;
                    hist_out[4 * (size_t)g + 1] -= k_own;
                    atomicAdd(&f.an.counters[((size_t)line * CNT_REPL + (blockIdx.x & (CNT_REPL - 1))) * NCOUNT + 11],
                              (unsigned long long)k_own);
                }
            }
        }
        if (!own) continue;
        const int line = f.cell_line[g];
        const LineDev& L = f.lines[line];
        const long long J = (long long)f.J[g] + dJ * (1ll << POS_TO_FIX);
        const double j = (double)J * FIX_INV * L.Q;
        f.J[g] = 0ull;
        f.j_last[g] = j;
        if (!f.frozen) {
            const double En = f.E[g] - 4.0 * 3.14159265358979323846 * (j - L.j_tw);
            f.E[g] = En;
            const int c = g - L.cell_base;
            float* e32 = f.E32 + L.field_base + c;
            e32[0] = (float)En;
            if (c == 0) e32[-1] = (float)En;
            if (c == L.n_cells - 1) e32[1] = (float)En;
        }
        const int ps = f.pair_step[g];
        f.pair_step[g] = 0;
        if (averaging) {
            f.E_sum[g] += f.E[g];
            f.j_sum[g] += j;
            f.pair_sum[g] += ps;
#pragma unroll
            for (int s = 0; s < 4; ++s) f.n_sum[4 * (size_t)g + s] += hist_out[4 * (size_t)g + s];
        }
        f.pair_last[g] = ps;
#pragma unroll
        for (int s = 0; s < 4; ++s) hist_in[4 * (size_t)g + s] = 0;
    }
}

// ---------------------------------------------------------------------------
// Sort by position (counting sort per segment on the key cell * sub +
// floor(offset * sub), sub bins per cell, eight unless the launch tuner picks
// another power of two), dropping absorbed particles.  Ordering by parts of a
// cell, not only by cell, keeps a lane's consecutive particles together in
// space, so that after a step the ones that crossed a face are grouped instead
// of spread through every lane's slots.  Counts live in bins[cell * sub + k] as
// one int4 (the four species):
//   k_sort_zero     clears the bins; a block of its own plans the sort's tiles
//   k_sort_count    counts the live particles per bin
//   k_sort_chunks   per chunk of SCAN_CELLS cells: its counts
//   k_sort_lines    per line: exclusive scan over its chunks, and the new counts
//   k_sort_cursors  per chunk: each bin's first slot
//   k_sort_scan     the three of them in one launch, for lines of few chunks
//   k_sort_scatter  every particle takes the next slot of its bin
//   k_plan          takes over the new counts
//
// Particles move a few cells between sorts, so a tile of SORT_TILE consecutive ones
// touches few bins: the tile is counted in LDS, each bin of it costs one global
// atomic, and the scatter orders the tile by bin in LDS first, so that it writes
// runs of consecutive slots.  A tile whose bins span more than SORT_PASSES windows
// of SORT_W (appended particles in no order) goes straight to the global bins.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int sort_bin(int cell_base, int c, float off, int sub) {
    return (cell_base + c) * sub + min((int)(off * (float)sub), sub - 1);    // off * sub is exact
}

__device__ __forceinline__ int& int4_at(int4& v, int k) {
    return k == 0 ? v.x : k == 1 ? v.y : k == 2 ? v.z : v.w;
}

// The candidates: every live e- and e+ (appends included) of a cell over the limit
// whose key is at most the cell's threshold records its key and slot.  A thread takes
// U particles per pass, four consecutive ones by one load, and issues its loads
// together.
template <int U>
__device__ __forceinline__ void annih_gather(const AnnihArgs& a) {
    const uint64_t step = a.sc->step;
    const int32_t* hist_out = a.hist[(step & 1) ^ 1];
    constexpr int CHUNK = 256 * U;
    // the chunks of all segments are dealt to the blocks in turn
    int64_t first = blockIdx.x;                                  // this block's next chunk, from the segment's start
    uint32_t tags = 0u;
    for (int l = 0; l < a.n_lines; ++l) {
        const int cb = a.lines[l].cell_base;
        for (int s = 0; s < 2; ++s) {
            const int seg = 4 * l + s;
            const int n = min(a.alloc[seg], a.seg_cap[seg]);
            const int64_t base = a.seg_base[seg];
            const int64_t nchunk = (n + (int64_t)CHUNK - 1) / CHUNK;     // (a segment may hold nearly 2^31 slots)
            for (; first < nchunk; first += gridDim.x) {
                // four consecutive particles at a time; a group that starts below n lies within
                // the segment (capacities are multiples of 256)
                const int64_t i0 = first * CHUNK + 4 * (int)threadIdx.x;
                auto at = [&](int u) { return i0 + (u >> 2) * 1024 + (u & 3); };
                int cu[U];
                uint32_t tu[U];
                uint64_t du[U];
#pragma unroll
                for (int u = 0; u < U; u += 4) {
                    const int4 c = at(u) < n ? *reinterpret_cast<const int4*>(a.cell + base + at(u))
                                             : make_int4(DEAD_CELL, DEAD_CELL, DEAD_CELL, DEAD_CELL);
                    cu[u] = c.x;
                    cu[u + 1] = at(u + 1) < n ? c.y : DEAD_CELL;
                    cu[u + 2] = at(u + 2) < n ? c.z : DEAD_CELL;
                    cu[u + 3] = at(u + 3) < n ? c.w : DEAD_CELL;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) tu[u] = cu[u] != DEAD_CELL ? a.ann_thr[cb + cu[u]] : 0u;
#pragma unroll
                for (int u = 0; u < U; u += 4) {
                    ulonglong2 d0 = make_ulonglong2(0ull, 0ull), d1 = d0;
                    if ((tu[u] | tu[u + 1] | tu[u + 2] | tu[u + 3]) != 0u) {
                        d0 = *reinterpret_cast<const ulonglong2*>(a.id + base + at(u));
                        d1 = *reinterpret_cast<const ulonglong2*>(a.id + base + at(u) + 2);
                    }
                    du[u] = d0.x;
                    du[u + 1] = d0.y;
                    du[u + 2] = d1.x;
                    du[u + 3] = d1.y;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (tu[u] == 0u) continue;
                    tags += cell_tag(cb + cu[u], s);
                    const uint64_t key = annih_key(step, du[u], a.key0, a.key1);
                    if ((uint32_t)(key >> 32) > tu[u]) continue;
                    const int g = cb + cu[u];
                    const int r = atomicAdd(&a.ann_fill[2 * (size_t)g + s], 1);
                    const int* h = hist_out + 4 * (size_t)g;
                    if (r >= h[s]) {              // counts and particles disagree: cannot happen
                        set_error(&a.sc->err, -4);
                        continue;
                    }
                    const int64_t rec = (int64_t)a.ann_off[g] + (s ? h[0] : 0) + r;
                    a.cand_key[rec] = key;
                    a.cand_slot[rec] = (int)at(u);
                }
            }
            first -= nchunk;
        }
    }
    add_tags(a.ann_tags, tags);
}

// Exits at once when no cell is over the limit.  Bound by HBM: 4 bytes of cell, and in a
// cell over the limit 8 of id, per particle, and by the latency of the chain cell ->
// threshold -> id -> key -> record, so a thread takes eight particles at a time where
// the grid's blocks all find a chunk that long, and four below.  70 us on a 65,536-cell
// line of 600 per cell, 109 us on eight lines of 32,768, 12 us on one of 9,973 (81, 134
// and 12 us by fours, 72, 112 and 15 us by eights; 88, 137 and 13.5 us by fours with one
// load a particle); the tag sums add 1.4, 1.2 and 0.4 us.  Eight wavefronts per SIMD: with
// one less 77 and 119 us.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_annih_gather(AnnihArgs a) {
    if (a.sc->err != 0) return;
    // a copy of the over-limit flag for k_field, which clears [1] for the next step
    // while its other blocks still need to know
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ann_ctl[2] = a.ann_ctl[1];
    if (a.ann_ctl[1] == 0) return;
    if ((int64_t)a.sc->tiles * a.tile >= (int64_t)gridDim.x * 256 * 8) annih_gather<8>(a);
    else annih_gather<4>(a);
}

// Segment of a tile by the whole wavefront: 64-way search over the tile prefix (the
// last segment whose first tile is at most t).
__device__ __forceinline__ int find_segment_wave(const int32_t* prefix, int nseg, int t) {
    const int lane = threadIdx.x & 63;
    int lo = 0, n = nseg;
    while (n > 1) {
        const int step = (n + 63) >> 6;
        const int i = lane * step;
        const unsigned long long m = __ballot(i < n && prefix[lo + i] <= t);     // lane 0 always
        const int at = (63 - __clzll((long long)m)) * step;
        lo += at;
        n = min(step, n - at);
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

__global__ __launch_bounds__(256) void k_sort_zero(SortArgs s) {
    if (s.sc->err != 0) return;
    const int nb = gridDim.x - 1;
    if ((int)blockIdx.x == nb) {
        // tiles of SORT_TILE slots per segment
        const int per = (s.nseg + 255) / 256;
        const int s0 = threadIdx.x * per, s1 = min(s0 + per, s.nseg);
        int sum = 0;
        for (int k = s0; k < s1; ++k) sum += tiles_of(s.n_cur[k], SORT_TILE);
        int total;
        int run = block_excl_scan(sum, total);
        for (int k = s0; k < s1; ++k) {
            s.sort_prefix[k] = run;
            run += tiles_of(s.n_cur[k], SORT_TILE);
        }
        if (threadIdx.x == 255) s.sort_prefix[s.nseg] = total;
        return;
    }
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < s.n_bins; i += nb * blockDim.x)
        s.bins[i] = make_int4(0, 0, 0, 0);
}

// One tile of the sort.  In the scatter a wavefront takes 64 SORT_U consecutive
// particles, 64 at a time, so that the ranks within a bin, which LDS atomics hand out,
// mostly keep the particles' order: neighbours in memory stay neighbours in space
// below a bin's width, and the next push's lanes find their table records again (with
// four consecutive particles per lane the scatter was 3% faster and the following
// pushes of a quiet line 4% slower: 757 against 726 us on 40 lines).  The count, which
// leaves no order, takes four per lane: its LDS atomics then meet in fewer bins.
struct SortTile {
    int sp, ncur, i0, cap;
    int64_t base;
    const LineDev* L;
    __device__ SortTile(const SortArgs& s, int t) {
        const int seg = find_segment_wave(s.sort_prefix, s.nseg, t);
        sp = seg & 3;
        ncur = s.n_cur[seg];
        cap = s.seg_cap[seg];
        base = s.seg_base[seg];
        i0 = (t - s.sort_prefix[seg]) * SORT_TILE;
        L = &s.lines[seg >> 2];
    }
    // slot of the thread's q-th particle of the scatter
    __device__ int slot(int q) const {
        return i0 + (int)(threadIdx.x >> 6) * (64 * SORT_U) + 64 * q + (int)(threadIdx.x & 63);
    }
};

// The lowest and highest bin of a tile over the block; s_range: 2 ints per wavefront.
__device__ __forceinline__ void tile_range(int& lo, int& hi, int* s_range) {
    lo = wave_min_i(lo);
    hi = wave_max_i(hi);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_range[2 * w] = lo;
        s_range[2 * w + 1] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SORT_TPB / 64; ++k) {
        lo = min(lo, s_range[2 * k]);
        hi = max(hi, s_range[2 * k + 1]);
    }
}

// Counts per bin, a tile in LDS at a time.  Bound by HBM: 8 bytes per particle, 70 us for
// 3.9e7 particles (4.5 TB/s); with a match over each wavefront's keys instead, 256 us.
__global__ __launch_bounds__(SORT_TPB) void k_sort_count(SortArgs s) {
    if (s.sc->err != 0) return;
    __shared__ int sCnt[SORT_W];
    __shared__ int sRange[2 * SORT_TPB / 64];
    int32_t* bins = reinterpret_cast<int32_t*>(s.bins);
    const int total = s.sort_prefix[s.nseg];
    for (int b = threadIdx.x; b < SORT_W; b += SORT_TPB) sCnt[b] = 0;
    for (TileWalk tw(total); tw.t < tw.end; tw.t += tw.stride) {
        const SortTile T(s, tw.t);
        const int cb = T.L->cell_base;
        int bin[SORT_U];
        int lo = INT32_MAX, hi = -1;
#pragma unroll
        for (int h = 0; h < SORT_U / 4; ++h) {
            // four consecutive particles per lane; a group that starts below ncur lies within
            // the segment (capacities are multiples of 256)
            const int g = T.i0 + 4 * (h * SORT_TPB + (int)threadIdx.x);
            int4 c = make_int4(DEAD_CELL, DEAD_CELL, DEAD_CELL, DEAD_CELL);
            float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
            if (g < T.ncur) {
                c = *reinterpret_cast<const int4*>(s.cell + T.base + g);
                o = *reinterpret_cast<const float4*>(s.off + T.base + g);
            }
            const int cv[4] = {c.x, c.y, c.z, c.w};
            const float ov[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool live = g + j < T.ncur && cv[j] != DEAD_CELL;
                bin[4 * h + j] = live ? sort_bin(cb, cv[j], ov[j], s.sub) : -1;
            }
        }
#pragma unroll
        for (int q = 0; q < SORT_U; ++q) {
            lo = min(lo, bin[q] >= 0 ? bin[q] : INT32_MAX);
            hi = max(hi, bin[q]);
        }
        tile_range(lo, hi, sRange);
        const int windows = hi < 0 ? 0 : (hi - lo) / SORT_W + 1;
        const bool direct = windows > SORT_PASSES;
        if (direct) {
#pragma unroll
            for (int q = 0; q < SORT_U; ++q)
                if (bin[q] >= 0) atomicAdd(&bins[4 * (size_t)bin[q] + T.sp], 1);
        }
        for (int k = 0; !direct && k < windows; ++k) {
            const int w0 = lo + k * SORT_W;
#pragma unroll
            for (int q = 0; q < SORT_U; ++q) {
                const int r = bin[q] - w0;
                if (bin[q] >= 0 && r >= 0 && r < SORT_W) atomicAdd(&sCnt[r], 1);
            }
            __syncthreads();
            const int nbin = min(SORT_W, hi - w0 + 1);
            for (int b = threadIdx.x; b < nbin; b += SORT_TPB) {
                const int c = sCnt[b];
                if (c != 0) {
                    atomicAdd(&bins[4 * (size_t)(w0 + b) + T.sp], c);
                    sCnt[b] = 0;
                }
            }
            __syncthreads();
        }
        if (windows == 0 || direct) __syncthreads();       // sRange is read before the next tile writes it
    }
}

// Block-wide exclusive scan of one int4 per thread (256 threads); returns the
// thread's prefix and writes the block total.
__device__ __forceinline__ int4 block_scan_int4(int4 v, int4& total) {
    __shared__ int4 sPart[256];
    const int t = threadIdx.x;
    sPart[t] = v;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const int4 w = t >= o ? sPart[t - o] : make_int4(0, 0, 0, 0);
        __syncthreads();
        if (t >= o) sPart[t] = make_int4(sPart[t].x + w.x, sPart[t].y + w.y, sPart[t].z + w.z, sPart[t].w + w.w);
        __syncthreads();
    }
    const int4 inc = sPart[t];
    total = sPart[255];
    __syncthreads();
    return make_int4(inc.x - v.x, inc.y - v.y, inc.z - v.z, inc.w - v.w);
}

// Counts of one cell (thread) of a chunk (block), summed over its bins.
__device__ __forceinline__ int4 cell_counts(const SortArgs& s, int chunk, int& gcell, bool& in) {
    const int line = s.chunk_line[chunk];
    const LineDev& L = s.lines[line];
    const int c = (chunk - s.line_chunk0[line]) * SCAN_CELLS + (int)threadIdx.x;
    in = c < L.n_cells;
    gcell = L.cell_base + c;
    int4 n = make_int4(0, 0, 0, 0);
    if (in) {
        const int4* bc = s.bins + (size_t)gcell * s.sub;
#pragma unroll 8
        for (int k = 0; k < s.sub; ++k) {
            const int4 b = bc[k];
            n.x += b.x; n.y += b.y; n.z += b.z; n.w += b.w;
        }
    }
    return n;
}

__global__ __launch_bounds__(256) void k_sort_chunks(SortArgs s) {
    if (s.sc->err != 0) return;
    int gcell;
    bool in;
    const int4 n = cell_counts(s, blockIdx.x, gcell, in);
    int4 total;
    (void)block_scan_int4(n, total);
    if (threadIdx.x == 0) s.chunk_sum[blockIdx.x] = total;
}

// One block per line: the chunks' first slots (exclusive scan over the line's
// chunks, per species) and the line's new live counts.
__global__ __launch_bounds__(256) void k_sort_lines(SortArgs s) {
    if (s.sc->err != 0) return;
    const int line = blockIdx.x;
    const int c0 = s.line_chunk0[line], c1 = s.line_chunk0[line + 1];
    int4 run = make_int4(0, 0, 0, 0);
    for (int b = c0; b < c1; b += 256) {
        const int k = b + (int)threadIdx.x;
        const int4 v = k < c1 ? s.chunk_sum[k] : make_int4(0, 0, 0, 0);
        int4 total;
        const int4 ex = block_scan_int4(v, total);
        if (k < c1) s.chunk_sum[k] = make_int4(run.x + ex.x, run.y + ex.y, run.z + ex.z, run.w + ex.w);
        run = make_int4(run.x + total.x, run.y + total.y, run.z + total.z, run.w + total.w);
    }
    if (threadIdx.x < 4) s.new_count[4 * line + threadIdx.x] = int4_at(run, threadIdx.x);
}

// Each bin's first slot, from its cell's (the thread's).
__device__ __forceinline__ void cell_cursors(const SortArgs& s, int gcell, int4 run) {
    int4* bc = s.bins + (size_t)gcell * s.sub;
#pragma unroll 8
    for (int k = 0; k < s.sub; ++k) {
        const int4 b = bc[k];
        bc[k] = run;
        run = make_int4(run.x + b.x, run.y + b.y, run.z + b.z, run.w + b.w);
    }
}

__global__ __launch_bounds__(256) void k_sort_cursors(SortArgs s) {
    if (s.sc->err != 0) return;
    int gcell;
    bool in;
    const int4 n = cell_counts(s, blockIdx.x, gcell, in);
    int4 total;
    const int4 ex = block_scan_int4(n, total);
    if (!in) return;
    const int4 c0 = s.chunk_sum[blockIdx.x];
    cell_cursors(s, gcell, make_int4(c0.x + ex.x, c0.y + ex.y, c0.z + ex.z, c0.w + ex.w));
}

// k_sort_chunks, k_sort_lines and k_sort_cursors of one line in one block: 11 us at
// two chunks instead of three launches of 5 us each; beyond SCAN_MAX_CHUNKS the
// chunks one after another cost more than the launches.
__global__ __launch_bounds__(256) void k_sort_scan(SortArgs s) {
    if (s.sc->err != 0) return;
    const int line = blockIdx.x;
    int4 run = make_int4(0, 0, 0, 0);
    for (int k = s.line_chunk0[line]; k < s.line_chunk0[line + 1]; ++k) {
        int gcell;
        bool in;
        const int4 n = cell_counts(s, k, gcell, in);
        int4 total;
        const int4 ex = block_scan_int4(n, total);
        if (in) cell_cursors(s, gcell, make_int4(run.x + ex.x, run.y + ex.y, run.z + ex.z, run.w + ex.w));
        run = make_int4(run.x + total.x, run.y + total.y, run.z + total.z, run.w + total.w);
    }
    if (threadIdx.x < 4) s.new_count[4 * line + threadIdx.x] = int4_at(run, threadIdx.x);
}

// Block-wide exclusive scan of one int per thread (SORT_TPB threads).
__device__ __forceinline__ int tile_scan(int v, int& total, int* s_part) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) s_part[w] = inc;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < SORT_TPB / 64; ++k) {
        const int pk = s_part[k];
        before += k < w ? pk : 0;
        total += pk;
    }
    return before + inc - v;
}

// Every live particle takes the next slot of its bin.  Per tile: ranks within the
// bins by LDS atomics, one global reservation per bin, then the particles pass
// through LDS in bin order and are written as runs.  Bound by HBM: 40 bytes per
// particle, 365 us for 3.9e7 particles on 65,536 cells and 871 us for 1.03e8 on 40
// lines (4.3 and 4.7 TB/s; a large copy reaches 5.5), where reserving by the wavefront
// and writing each lane's particle where it fell took 653 and 1,372 us.  The tile of
// 4,096 is the largest of which two fit a CU's LDS: the longer a bin's run, the fewer
// lines a store touches.
__global__ __launch_bounds__(SORT_TPB) __attribute__((amdgpu_waves_per_eu(4))) void k_sort_scatter(SortArgs s) {
    if (block_stopped(s.sc)) return;
    // the windows of the ranking, and after it the tile's particles in bin order
    __shared__ union {
        struct { int cnt[SORT_W], excl[SORT_W], base[SORT_W]; } w;
        struct { int32_t cell[SORT_TILE]; float off[SORT_TILE], u[SORT_TILE]; } p;
        uint64_t id[SORT_TILE];
    } sh;
    __shared__ int sDst[SORT_TILE];
    __shared__ int sRange[2 * SORT_TPB / 64], sPart[SORT_TPB / 64];
    int32_t* bins = reinterpret_cast<int32_t*>(s.bins);
    const int total = s.sort_prefix[s.nseg];
    constexpr int BPT = SORT_W / SORT_TPB;        // bins per thread of the window's scan
    static_assert(BPT == 4, "the scan reads one int4 of counts per thread");
    // Counts and particles that disagree would run into the next segment: such a run goes to
    // the segment's start and the state freezes, with its particles in the set they come from.
    bool overrun = false;
    auto checked = [&](int at, int n, int cap) {
        const bool in = slots_in(at, n, cap);
        overrun = overrun || !in;
        return in ? at : 0;
    };
    for (TileWalk tw(total); tw.t < tw.end; tw.t += tw.stride) {
        const SortTile T(s, tw.t);
        const int cb = T.L->cell_base;
        int cv[SORT_U], bin[SORT_U], dst[SORT_U], pos[SORT_U];
        float ov[SORT_U], uv[SORT_U];
        uint64_t iv[SORT_U];
        int lo = INT32_MAX, hi = -1;
#pragma unroll
        for (int q = 0; q < SORT_U; ++q) {
            const int i = T.slot(q);
            const bool in = i < T.ncur;
            cv[q] = in ? s.cell[T.base + i] : DEAD_CELL;
            ov[q] = in ? s.off[T.base + i] : 0.0f;
            uv[q] = in ? s.u[T.base + i] : 0.0f;
            iv[q] = in ? s.id[T.base + i] : 0ull;
        }
#pragma unroll
        for (int q = 0; q < SORT_U; ++q) {
            bin[q] = cv[q] != DEAD_CELL ? sort_bin(cb, cv[q], ov[q], s.sub) : -1;
            dst[q] = pos[q] = 0;
            lo = min(lo, bin[q] >= 0 ? bin[q] : INT32_MAX);
            hi = max(hi, bin[q]);
        }
        tile_range(lo, hi, sRange);
        const int windows = hi < 0 ? 0 : (hi - lo) / SORT_W + 1;
        if (windows > SORT_PASSES) {
#pragma unroll
            for (int q = 0; q < SORT_U; ++q) {
                if (bin[q] < 0) continue;
                const int64_t k = T.base + checked(atomicAdd(&bins[4 * (size_t)bin[q] + T.sp], 1), 1, T.cap);
                s.cell2[k] = cv[q];
                s.off2[k] = ov[q];
                s.u2[k] = uv[q];
                s.id2[k] = iv[q];
            }
            __syncthreads();                          // sRange is read before the next tile writes it
            continue;
        }
        int live = 0;                                 // particles in the windows so far
        for (int k = 0; k < windows; ++k) {
            const int w0 = lo + k * SORT_W;
            for (int b = threadIdx.x; b < SORT_W; b += SORT_TPB) sh.w.cnt[b] = 0;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < SORT_U; ++q) {
                const int r = bin[q] - w0;
                if (bin[q] >= 0 && r >= 0 && r < SORT_W) pos[q] = atomicAdd(&sh.w.cnt[r], 1);
            }
            __syncthreads();
            const int4 n = reinterpret_cast<const int4*>(sh.w.cnt)[threadIdx.x];
            int in_window;
            const int ex = tile_scan(n.x + n.y + n.z + n.w, in_window, sPart);
            reinterpret_cast<int4*>(sh.w.excl)[threadIdx.x] =
                make_int4(ex, ex + n.x, ex + n.x + n.y, ex + n.x + n.y + n.z);
            const int nbin = min(SORT_W, hi - w0 + 1);
            for (int b = threadIdx.x; b < nbin; b += SORT_TPB) {
                const int c = sh.w.cnt[b];
                if (c != 0) sh.w.base[b] = checked(atomicAdd(&bins[4 * (size_t)(w0 + b) + T.sp], c), c, T.cap);
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < SORT_U; ++q) {
                const int r = bin[q] - w0;
                if (bin[q] >= 0 && r >= 0 && r < SORT_W) {
                    dst[q] = sh.w.base[r] + pos[q];
                    pos[q] += live + sh.w.excl[r];
                }
            }
            live += in_window;
            __syncthreads();
        }
#pragma unroll
        for (int q = 0; q < SORT_U; ++q) {
            if (bin[q] < 0) continue;
            sDst[pos[q]] = dst[q];
            sh.p.cell[pos[q]] = cv[q];
            sh.p.off[pos[q]] = ov[q];
            sh.p.u[pos[q]] = uv[q];
        }
        __syncthreads();
        for (int i = threadIdx.x; i < live; i += SORT_TPB) {
            const int64_t k = T.base + sDst[i];
            s.cell2[k] = sh.p.cell[i];
            s.off2[k] = sh.p.off[i];
            s.u2[k] = sh.p.u[i];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < SORT_U; ++q)
            if (bin[q] >= 0) sh.id[pos[q]] = iv[q];
        __syncthreads();
        for (int i = threadIdx.x; i < live; i += SORT_TPB) s.id2[T.base + sDst[i]] = sh.id[i];
        __syncthreads();
    }
    if (overrun) set_error(&s.sc->err, -3);
}

// ---------------------------------------------------------------------------
// Initial pair plasma: pair i of a line in cell i / ppc at offset U24(w0) of the
// Philox block (0, i, line, STREAM_INIT).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_init_pairs(InitArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n_pairs) return;
    const uint4 w = philox4x32_10(make_uint4(0u, (uint32_t)i, (uint32_t)a.line, STREAM_INIT), a.key0, a.key1);
    const int cell = (int)(i / a.ppc);
    const float off = uniform24(w.x);
    float ue = 0.0f, up = 0.0f;
    if (a.mode == 1) {
        const double gam = pow(10.0, (double)uniform24(w.y) * a.log10_gmax);
        const double uu = sqrt(fmax(gam * gam - 1.0, 0.0));
        const float s = (w.z >> 31) ? -1.0f : 1.0f;
        ue = up = s * (float)uu;
    } else if (a.mode == 2) {
        up = (float)a.u_stream;
        ue = -(float)a.u_stream;
    }
    const int64_t ke = a.base_e + i, kp = a.base_p + i;
    a.cell[ke] = cell; a.off[ke] = off; a.u[ke] = ue; a.id[ke] = a.id_base + 2 * (uint64_t)i;
    a.cell[kp] = cell; a.off[kp] = off; a.u[kp] = up; a.id[kp] = a.id_base + 2 * (uint64_t)i + 1;
}

// Sum of v over the run of consecutive lanes that share this lane's key, in the
// run's first lane (head = true there).  Every lane of the wavefront must take part.
// Keys need not be sorted: equal keys that are not adjacent form runs of their own.
__device__ __forceinline__ long long wave_run_sum(int key, long long v, bool& head) {
    const int lane = threadIdx.x & 63;
    const int prev = __shfl_up(key, 1, 64);
    const int next = __shfl_down(key, 1, 64);
    head = lane == 0 || prev != key;
    const bool tail = lane == 63 || next != key;
    long long p = v;                                  // inclusive prefix sum
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long y = __shfl_up(p, o, 64);
        if (lane >= o) p += y;
    }
    const unsigned long long T = __ballot(tail);      // bit 63 always set
    const int e = lane + __builtin_ctzll(T >> lane);  // the run's last lane
    const long long pe = __shfl(p, e, 64);
    const long long pb = __shfl(p, lane > 0 ? lane - 1 : 0, 64);
    return pe - (lane > 0 ? pb : 0ll);
}

// Histogram of live particles per cell and species (after init / set_particles).
__global__ __launch_bounds__(256) void k_hist(HistArgs h) {
    const int total = h.tile_prefix[h.nseg];
    for (TileWalk tw(total); tw.t < tw.end; tw.t += tw.stride) {
        const int t = tw.t;
        const int seg = find_segment(h.tile_prefix, h.nseg, t);
        const int sp = seg & 3;
        const LineDev& L = h.lines[seg >> 2];
        const int ncur = h.n_cur[seg];
        const int64_t base = h.seg_base[seg];
        const int i0 = (t - h.tile_prefix[seg]) * h.tile;
        for (int q = 0; q < h.tile / PUSH_TPB; ++q) {
            // one atomic per run of lanes in the same cell (every lane takes part)
            const int i = i0 + q * PUSH_TPB + threadIdx.x;
            const int c = i < ncur ? h.cell[base + i] : DEAD_CELL;
            bool head;
            const long long n = wave_run_sum(c == DEAD_CELL ? -1 : c, c == DEAD_CELL ? 0 : 1, head);
            if (head && c != DEAD_CELL) atomicAdd(&h.hist[4 * (size_t)(L.cell_base + c) + sp], (int)n);
        }
    }
}

// ---------------------------------------------------------------------------
// Moments: cloud-in-cell charge on nodes (fixed point), kinetic energy.
// A block takes 256 MOM_U consecutive particles of one of the line's segments at a
// time, the chunks of the four segments dealt in turn, so that small segments share the
// blocks; neighbours in memory share cells, so a thread adds its runs of particles of
// one cell, and the block collects its charge in an LDS window of nodes before the
// global one.  Bound by the float64 arithmetic of the kinetic energy: 153 us for 3.9e7
// particles on 65,536 cells, 14 us for 1.5e5 on 512 (400 and 55 us with a segmented sum
// over every wavefront in place of the window, and atomics on three addresses for the
// kinetic energy).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_moments_particles(MomArgs m) {
    __shared__ unsigned long long sR[MOM_W];
    __shared__ unsigned long long sK[4][3];
    __shared__ int sLo[4], sHi[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int k = threadIdx.x; k < MOM_W; k += 256) sR[k] = 0ull;
    // kinetic energy sum m (gamma - 1) / m_e in fixed point: v 2^48 split exactly into
    // three 32-bit chunks, each summed as an integer, so the total does not depend on
    // the order in which particles are visited (bits below 2^-48 of a term dropped)
    unsigned long long k0 = 0, k1 = 0, k2 = 0;
    constexpr int CHUNK = 256 * MOM_U;
    // the chunks of the line's four segments are dealt to the blocks in turn
    int64_t next = blockIdx.x;
    for (int sp = 0; sp < NSPEC; ++sp) {
        const int seg = 4 * m.line + sp;
        const int ncur = m.n_cur[seg];
        const int64_t base = m.seg_base[seg];
        const long long sg = m.sign[sp] < 0.0 ? -1 : 1;
        const double mass = (sp == 3) ? m.mass_ratio : 1.0;
        const int64_t nchunk = (ncur + (int64_t)CHUNK - 1) / CHUNK;
        for (; next < nchunk; next += gridDim.x) {
            const int64_t i0 = next * CHUNK;
            int cv[MOM_U];
            float ov[MOM_U], uv[MOM_U];
            int lo = INT32_MAX, hi = -1;
#pragma unroll
            for (int h = 0; h < MOM_U / 4; ++h) {
                // four consecutive particles; a group that starts below ncur lies within the
                // segment (capacities are multiples of 256)
                const int64_t g = i0 + 4 * (h * 256 + (int)threadIdx.x);
                int4 c = make_int4(DEAD_CELL, DEAD_CELL, DEAD_CELL, DEAD_CELL);
                float4 o = make_float4(0.f, 0.f, 0.f, 0.f), u = o;
                if (g < ncur) {
                    c = *reinterpret_cast<const int4*>(m.cell + base + g);
                    o = *reinterpret_cast<const float4*>(m.off + base + g);
                    u = *reinterpret_cast<const float4*>(m.u + base + g);
                }
                const int c4[4] = {c.x, c.y, c.z, c.w};
                const float o4[4] = {o.x, o.y, o.z, o.w}, u4[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool live = g + j < ncur && c4[j] != DEAD_CELL;
                    cv[4 * h + j] = live ? c4[j] : -1;
                    ov[4 * h + j] = o4[j];
                    uv[4 * h + j] = live ? u4[j] : 0.0f;
                    lo = min(lo, live ? c4[j] : INT32_MAX);
                    hi = max(hi, live ? c4[j] : -1);
                }
            }
            lo = wave_min_i(lo);
            hi = wave_max_i(hi);
            if (lane == 0) {
                sLo[w] = lo;
                sHi[w] = hi;
            }
            __syncthreads();
            lo = min(min(sLo[0], sLo[1]), min(sLo[2], sLo[3]));
            hi = max(max(sHi[0], sHi[1]), max(sHi[2], sHi[3]));
            const bool window = hi >= 0 && hi - lo + 2 <= MOM_W;
            int key = -1;
            long long a0 = 0, a1 = 0;
            auto flush = [&] {
                if (key < 0) return;
                if (window) {
                    atomicAdd(&sR[key - lo], (unsigned long long)a0);
                    atomicAdd(&sR[key - lo + 1], (unsigned long long)a1);
                } else {
                    atomicAdd(&m.rho[key], (unsigned long long)a0);
                    atomicAdd(&m.rho[key + 1], (unsigned long long)a1);
                }
            };
#pragma unroll
            for (int q = 0; q < MOM_U; ++q) {
                if (cv[q] != key) {
                    flush();
                    key = cv[q];
                    a0 = a1 = 0;
                }
                // cloud-in-cell weights of the position quantised as in the deposit (2^-28 cell)
                const long long f = (long long)(int)(ov[q] * POS_SCALE) << POS_TO_FIX;
                a0 += sg * (4294967296ll - f);
                a1 += sg * f;
                // gamma - 1 = u^2 / (gamma + 1), free of cancellation at small u
                const double u = (double)uv[q];
                const double v = mass * (u * u / (sqrt(fma(u, u, 1.0)) + 1.0));
                const double sv = v * 0x1.0p48;
                const double h2 = floor(sv * 0x1.0p-64);
                const double r = fma(-h2, 0x1.0p64, sv);          // exact: the bits of sv below 2^64
                const double h1 = floor(r * 0x1.0p-32);
                const double h0 = floor(fma(-h1, 0x1.0p32, r));
                k0 += (unsigned long long)h0;
                k1 += (unsigned long long)h1;
                k2 += (unsigned long long)h2;
            }
            flush();
            __syncthreads();
            if (window) {
                for (int k = threadIdx.x; k < hi - lo + 2; k += 256) {
                    const unsigned long long v = sR[k];
                    if (v != 0ull) {
                        atomicAdd(&m.rho[lo + k], v);
                        sR[k] = 0ull;
                    }
                }
            }
            __syncthreads();
        }
        next -= nchunk;
    }
    for (int o = 32; o > 0; o >>= 1) {
        k0 += __shfl_xor(k0, o, 64);
        k1 += __shfl_xor(k1, o, 64);
        k2 += __shfl_xor(k2, o, 64);
    }
    if (lane == 0) {
        sK[w][0] = k0;
        sK[w][1] = k1;
        sK[w][2] = k2;
    }
    __syncthreads();
    if (threadIdx.x < 3)
        m.hdr->kin[blockIdx.x][threadIdx.x] = sK[0][threadIdx.x] + sK[1][threadIdx.x] + sK[2][threadIdx.x] + sK[3][threadIdx.x];
}

// Gauss residual on interior nodes, the per-block partial sums of E and E^2 and the live
// counts of one line (the host adds the partials in block order: the circuit potential
// and the field energy are the same bits on every run), and the per-cell arrays of the
// cells [c0, c1), straight into pinned host memory: one transfer at the link's rate
// (4 MB in 85 us) in place of a copy per array through the runtime's staging.
__global__ __launch_bounds__(256) void k_moments_grid(MomArgs m) {
    __shared__ double sE[4][3];
    __shared__ long long sC[4][4];
    const LineDev& L = m.lines[m.line];
    const int n = L.n_cells, cb = L.cell_base;
    const uint64_t step = m.sc->step;
    const int32_t* hist = m.hist[step & 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (m.first) {
        if (blockIdx.x == 0 && threadIdx.x < NCOUNT) {
            unsigned long long c = 0;
            for (int r = 0; r < CNT_REPL; ++r) c += m.counters[((size_t)m.line * CNT_REPL + r) * NCOUNT + threadIdx.x];
            m.hdr->counters[threadIdx.x] = (int64_t)c;
        }
        if (blockIdx.x == 0 && threadIdx.x == NCOUNT) {
            m.hdr->step = (int64_t)step;
            m.hdr->avg = m.avg_count[0];
        }
        double rmax = 0.0, esum = 0.0, e2 = 0.0;
        long long cnt[4] = {0, 0, 0, 0};
        const double* E = m.E + cb;
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += gridDim.x * blockDim.x) {
            if (i < n) {
                esum += E[i];
                e2 = fma(E[i], E[i], e2);
#pragma unroll
                for (int s = 0; s < 4; ++s) cnt[s] += hist[4 * (size_t)(cb + i) + s];
            }
            if (i >= 1 && i <= n - 1) {
                const double rho = (double)(long long)m.rho[i] * FIX_INV * L.Q;
                rmax = fmax(rmax, fabs(E[i] - E[i - 1] - 4.0 * 3.14159265358979323846 * rho));
            }
            m.rho[i] = 0ull;                 // for the next call
        }
        for (int o = 32; o > 0; o >>= 1) {
            rmax = fmax(rmax, __shfl_xor(rmax, o, 64));
            esum += __shfl_xor(esum, o, 64);
            e2 += __shfl_xor(e2, o, 64);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) cnt[s] = wave_sum_ll(cnt[s]);
        if (lane == 0) {
            sE[w][0] = esum;
            sE[w][1] = e2;
            sE[w][2] = rmax;
#pragma unroll
            for (int s = 0; s < 4; ++s) sC[w][s] = cnt[s];
        }
        __syncthreads();
        if (threadIdx.x < 2)
            m.hdr->part[blockIdx.x][threadIdx.x] =
                ((sE[0][threadIdx.x] + sE[1][threadIdx.x]) + sE[2][threadIdx.x]) + sE[3][threadIdx.x];
        if (threadIdx.x == 2) m.hdr->rmax[blockIdx.x] = fmax(fmax(sE[0][2], sE[1][2]), fmax(sE[2][2], sE[3][2]));
        if (threadIdx.x >= 64 && threadIdx.x < 68) {
            const int s = threadIdx.x - 64;
            m.hdr->count[blockIdx.x][s] = sC[0][s] + sC[1][s] + sC[2][s] + sC[3][s];
        }
    }
    const double na = m.average ? (double)max(m.avg_count[0], 1ll) : 1.0;
    const size_t len = (size_t)(m.c1 - m.c0);
    for (int c = m.c0 + blockIdx.x * blockDim.x + threadIdx.x; c < m.c1; c += gridDim.x * blockDim.x) {
        const size_t g = (size_t)cb + c;
        double* o = m.arr + (c - m.c0);
#pragma unroll
        for (int s = 0; s < 4; ++s)
            o[s * len] = (m.average ? (double)m.n_sum[4 * g + s] : (double)hist[4 * g + s]) / (na * m.ppc0);
        o[4 * len] = (m.average ? m.j_sum[g] : m.j_last[g]) / (na * m.jn);
        o[5 * len] = (m.average ? m.E_sum[g] : m.E[g]) / na;
        o[6 * len] = m.average ? (double)m.pair_sum[g] / na : (double)m.pair_last[g];
    }
}

// RICS backend evaluation at given points (diagnostics and surrogate error).
template <int BACKEND>
__device__ __forceinline__ void rics_eval_point(const PushArgs& a, int line, int64_t n, const float* s_cells,
                                                const float* uin, float* F, float* N, float* eps) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const LineDev L = a.lines[line];
    const float s = fminf(fmaxf(s_cells[i], 0.0f), (float)L.n_cells);
    const int c0 = min((int)floorf(s), L.n_cells - 1);
    const float o0 = s - (float)c0;
    PartGeo pg = part_geo<BACKEND>(a, L, a.nodes[L.node_base + c0], a.nodes[L.node_base + c0 + 1], c0, o0);
    const Geo& g = pg.g;
    const float u = uin[i];
    float f = 0.0f, nd = 0.0f;
    if constexpr (BACKEND != RICS_OFF) {
        f = rics_eval<BACKEND>(a, L, u, pg).F;
        nd = rics_N<BACKEND>(a, L, u, pg);
    }
    F[i] = f;
    N[i] = nd;
    eps[i] = photon_energy(fsqrt(fmaf(u, u, 1.0f)), g.b);
}
template <int BACKEND>
__global__ __launch_bounds__(256) void k_rics_eval(PushArgs a, int line, int64_t n, const float* s_cells,
                                                   const float* uin, float* F, float* N, float* eps) {
    rics_eval_point<BACKEND>(a, line, n, s_cells, uin, F, N, eps);
}
template __global__ void k_rics_eval<RICS_OFF>(PushArgs, int, int64_t, const float*, const float*, float*, float*, float*);
template __global__ void k_rics_eval<RICS_EXACT>(PushArgs, int, int64_t, const float*, const float*, float*, float*, float*);
template __global__ void k_rics_eval<RICS_TABLE>(PushArgs, int, int64_t, const float*, const float*, float*, float*, float*);

// The surrogate at n points (one per lane; the whole wavefront evaluates the
// network together, lanes past n on a dummy point).
__global__ __launch_bounds__(256) void k_rics_eval_mlp(PushArgs a, int line, int64_t n, const float* s_cells,
                                                       const float* uin, float* F, float* N, float* eps) {
    if (a.lines[line].use_table) {           // this line takes its table (uniform over the launch)
        rics_eval_point<RICS_TABLE>(a, line, n, s_cells, uin, F, N, eps);
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool ok = i < n;
    const LineDev L = a.lines[line];
    const float s = ok ? fminf(fmaxf(s_cells[i], 0.0f), (float)L.n_cells) : 0.5f;
    const int c0 = min((int)floorf(s), L.n_cells - 1);
    const float o0 = s - (float)c0;
    const double x = (double)c0 + (double)o0;
    const Geo g = geo_lerp(L, a.nodes[L.node_base + c0], a.nodes[L.node_base + c0 + 1], o0);
    const float u = ok ? uin[i] : 0.0f;
    int n_eval = 0;
    const MlpRics rr = mlp_rics(a, a.mlp_ft, a.mlp_bias, u, g, (float)(x / (double)L.n_cells), n_eval);
    if (ok) {
        F[i] = rr.F;
        N[i] = rr.N;
        eps[i] = photon_energy(fsqrt(fmaf(u, u, 1.0f)), g.b);
    }
}

// The surrogate's error estimate on each line (MLP backend with table fallback):
// every table node (log10 gamma_i, row centre s_j) of every line is evaluated by
// the network as the pusher evaluates it (float32 geometry, inputs at s_j / L) and
// by the closed forms of Eqs. contdrag and scatteringNdot in float64; the line's
// estimate is the largest relative error of F and Ndot where they are significant
// (|F| h >= 1e-9 max(u, 1) and Ndot h >= 1e-9).  One node per lane; the whole wavefront
// evaluates the network together.
__global__ __launch_bounds__(256) void k_mlp_line_error(PushArgs a, const double* row_geo, double kT_keV,
                                                        unsigned int* err) {
    __shared__ bf16x8 sW[FT_TOTAL * 64];
    __shared__ float sWb[MLP_BIAS];
    for (int e = threadIdx.x; e < FT_TOTAL * 64; e += blockDim.x) sW[e] = a.mlp_ft[e];
    for (int e = threadIdx.x; e < MLP_BIAS; e += blockDim.x) sWb[e] = a.mlp_bias[e];
    __syncthreads();
    const int nlg = a.nlg, ns = a.ns;
    const int64_t per_line = (int64_t)nlg * ns;
    const int n_lines = a.nseg >> 2;
    const int64_t total = per_line * n_lines;
    const double theta = kT_keV / 510.99895000;
    const double base = 2.8179403262e-13 * 1.0e6 / (4.0 * 3.8615926796e-11 * 3.8615926796e-11);
    const double AF = base * theta * theta * theta, AN = base * theta * theta;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    // every lane of a wavefront runs the same number of iterations (the network needs all 64)
    const int64_t rounds = (total + stride - 1) / stride;
    for (int64_t it = 0; it < rounds; ++it) {
        const int64_t e = it * stride + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
        const bool valid = e < total;
        const int64_t ee = valid ? e : 0;
        const int line = (int)(ee / per_line);
        const int rem = (int)(ee % per_line);
        const int j = rem / nlg, i = rem % nlg;
        const LineDev& L = a.lines[line];
        const double* rg = row_geo + 3 * ((size_t)line * ns + j);
        const double b = rg[0], mu = rg[1], x = rg[2];
        const double gam = pow(10.0, 8.0 * i / (nlg - 1));
        const double u = sqrt(fmax(gam * gam - 1.0, 0.0));
        Geo g;
        g.b = (float)b;
        g.mu = (float)mu;
        g.ix2 = frcp((float)x * (float)x);
        g.by = g.b * L.inv_theta;
        int dummy = 0;
        const MlpRics r = mlp_rics(a, sW, sWb, (float)u, g, (float)((j + 0.5) / ns), dummy);
        // closed forms (float64)
        const double y = b / (theta * (gam - u * mu));
        double Fe = 0.0, Ne = 0.0;
        if (y <= 80.0) {
            const double em1 = expm1(y);
            Fe = AF / (x * x) * (gam * mu - u) * y * y * y / em1;
            Ne = AN / (x * x * gam) * y * y / em1;
        }
        const double h = (double)L.h;
        double worst = 0.0;
        if (valid && fabs(Fe) * h >= 1e-9 * fmax(u, 1.0) && Fe != 0.0) worst = fabs((double)r.F - Fe) / fabs(Fe);
        if (valid && Ne * h >= 1e-9) worst = fmax(worst, fabs((double)r.N - Ne) / Ne);
        if (!(worst <= 3.0e38)) worst = 3.0e38;        // non-finite network output: no trust
        const float wf = (float)worst;
        if (valid && wf > 0.0f) atomicMax(&err[line], __float_as_uint(wf));
    }
}

}  // namespace pic1d
