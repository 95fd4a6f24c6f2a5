// blas.hip -- site-local kernels of the Krylov solvers (the paper's "zaxpy-like"
// functions, Sec. 2.3 and Sec. 4.2), compensated dot products, and the packing of
// gauge links into the 12-real formats (Sec. 2.3, Sec. 4.1).
//
// Every vector kernel fuses the axpy updates with the reduction that follows
// them (|r|^2 after x += alpha p, r -= alpha q), so a CG iteration reads each
// vector the minimum number of times.  Reductions: TwoSum per thread, wave64
// shuffle and LDS pair tree, one (sum, error) pair per block, and a finalize
// kernel (one block per system) that adds the pairs in a fixed order and runs the
// scalar step.

#include "device_common.hpp"
#include "kernels.hpp"
#include "solver_state.hpp"

namespace stg {

// The vector kernels of several fields run one block per (chunk of kBlock sites, field):
// blockIdx.y is the field, so a parked field's blocks leave at once, and a small lattice
// has as many blocks as fields times chunks to hide its latency with.  A thread loads all
// vectors of its site before it stores any (the stores may alias the loads as far as the
// compiler knows, so loads issued per colour would wait for them).  With all fields in
// one thread, one colour at a time: 16^3 x 32, 4 FP64 fields, r update 9.3 -> 7.4 us, p
// update 7.9 -> 6.5; mixed CG with 8 RHS at 16^4 34.1 -> 26.3 ms, at 32^4 253 -> 242.
struct FieldSite {
    int j;        // field
    size_t o;     // its site's first entry
    bool live;
    __device__ __forceinline__ explicit FieldSite(const VecArgs &a) {
        const uint32_t h = blockIdx.x * kBlock + threadIdx.x;
        j = (int)blockIdx.y;
        o = (size_t)j * a.fstride + h;
        live = h < a.Vh;
    }
};

template <typename T>
__device__ __forceinline__ vec3<T> ld_site(const void *f, size_t o, uint32_t Vh) {
    vec3<T> v;
#pragma unroll
    for (int c = 0; c < 3; ++c) v.c[c] = ld_c<T>(f, o + (size_t)c * Vh);
    return v;
}

template <typename T>
__device__ __forceinline__ void st_site(void *f, size_t o, uint32_t Vh, const vec3<T> &v) {
#pragma unroll
    for (int c = 0; c < 3; ++c) st_c<T>(f, o + (size_t)c * Vh, v.c[c]);
}

// the block's sum of field j into its place of the partials
__device__ __forceinline__ void field_partials(const VecArgs &a, int j, double s, double c) {
    double ps[1] = {s}, pc[1] = {c};
    block_partials<1>(ps, pc, a.partials + 2 * (size_t)j * gridDim.x);
}

// x += alpha p; r -= alpha q; block partials of |r|^2 (OP_BETA in the finalize kernel)
template <typename T>
__global__ __launch_bounds__(kBlock) void cg_update_kernel(VecArgs a) {
    const FieldSite f(a);
    const SysState &s = a.state[f.j];
    if (!(s.flags & SYS_RUNNING)) return;
    double ps = 0.0, pc = 0.0;
    if (f.live) {
        const T al = (T)s.alpha;
        vec3<T> x = ld_site<T>(a.x, f.o, a.Vh);
        const vec3<T> p = ld_site<T>(a.p, f.o, a.Vh);
        vec3<T> r = ld_site<T>(a.r, f.o, a.Vh);
        const vec3<T> q = ld_site<T>(a.q, f.o, a.Vh);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x.c[c].re += al * p.c[c].re;
            x.c[c].im += al * p.c[c].im;
            r.c[c].re -= al * q.c[c].re;
            r.c[c].im -= al * q.c[c].im;
            pair_add(ps, pc, (double)r.c[c].re * (double)r.c[c].re +
                                 (double)r.c[c].im * (double)r.c[c].im, 0.0);
        }
        st_site<T>(a.x, f.o, a.Vh, x);
        st_site<T>(a.r, f.o, a.Vh, r);
    }
    field_partials(a, f.j, ps, pc);
}

// p = r + beta p
template <typename T>
__global__ __launch_bounds__(kBlock) void p_update_kernel(VecArgs a) {
    const FieldSite f(a);
    const SysState &s = a.state[f.j];
    if (!(s.flags & SYS_RUNNING) || !f.live) return;
    const T be = (T)s.beta;
    vec3<T> p = ld_site<T>(a.p, f.o, a.Vh);
    const vec3<T> r = ld_site<T>(a.r, f.o, a.Vh);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        p.c[c].re = r.c[c].re + be * p.c[c].re;
        p.c[c].im = r.c[c].im + be * p.c[c].im;
    }
    st_site<T>(a.p, f.o, a.Vh, p);
}

// ---------------------------------------------------------------------------
// single-field CG iteration with the reductions finished by their consumers
// ---------------------------------------------------------------------------
// Sum of the n (sum, error) pairs at x by the whole block, in the fixed order of
// block_sum2_pairs, returned to every thread: every block of a launch obtains the
// bitwise same total, so each can take the scalar step itself and no finalize
// kernel runs between the producer and the consumer.
__device__ __forceinline__ double block_total(const double *x, uint32_t n) {
    __shared__ double sh_red[2 * kWaves];
    __shared__ double sh_tot;
    const double t = block_sum2_pairs(x, (int)n, sh_red);
    if (threadIdx.x == 0) sh_tot = t;
    __syncthreads();
    return sh_tot;
}

// alpha = rr / <p, q> (the hop's partials), x += alpha p, r -= alpha q, partials of
// |r|^2.  Writes no solver state.  A breakdown (<p, q> not a finite positive
// number) leaves x and r alone and writes NaN partials, which the beta step of the
// next kernel turns into SYS_BREAKDOWN.
template <typename T>
__global__ __launch_bounds__(kBlock) void cg_update_fused_kernel(VecArgs a) {
    if (block_gate_closed(a.ctl, a.gate_mask)) return;
    const double pq = block_total(a.fin_partials, a.fin_blocks);
    const SysState &s = a.state[0];
    const bool running = (s.flags & SYS_RUNNING) != 0;
    const bool ok = finite_pos(pq) && (s.rr >= 0.0 && s.rr < 1.0e300);
    const uint32_t h = blockIdx.x * kBlock + threadIdx.x;
    double ps[1] = {0.0}, pc[1] = {0.0};
    if (running && !ok) {
        ps[0] = __builtin_nan("");
    } else if (running && h < a.Vh) {
        const T al = (T)(s.rr / pq);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const size_t i = (size_t)c * a.Vh + h;
            cpx<T> x = ld_c<T>(a.x, i), p = ld_c<T>(a.p, i), r = ld_c<T>(a.r, i),
                   q = ld_c<T>(a.q, i);
            x.re += al * p.re;
            x.im += al * p.im;
            r.re -= al * q.re;
            r.im -= al * q.im;
            st_c<T>(a.x, i, x);
            st_c<T>(a.r, i, r);
            pair_add(ps[0], pc[0], (double)r.re * (double)r.re + (double)r.im * (double)r.im,
                     0.0);
        }
    }
    block_partials<1>(ps, pc, a.partials);
}

// |r_new|^2 from the partials of cg_update_fused, the beta step (solver_state.hpp)
// on a copy of the state, p = r + beta p while the system still runs.  Block 0
// stores the new state in a.state_out: the next iteration reads that buffer, so
// no block reads a state that another block of this launch is writing.  Block 0
// always runs (also when no system runs), so that a.state_out is always current.
template <typename T>
__global__ __launch_bounds__(kBlock) void p_update_fused_kernel(VecArgs a) {
    const bool closed = block_gate_closed(a.ctl, a.gate_mask);
    if (closed && blockIdx.x != 0) return;
    SysState ns = a.state[0];
    ns.flags &= ~SYS_RESUME;
    bool left = false;
    if (!closed && (ns.flags & SYS_RUNNING)) {
        const double rr = block_total(a.fin_partials, a.fin_blocks);
        left = beta_step(ns, rr);
        const uint32_t h = blockIdx.x * kBlock + threadIdx.x;
        if (!left && h < a.Vh) {
            const T be = (T)ns.beta;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const size_t i = (size_t)c * a.Vh + h;
                cpx<T> p = ld_c<T>(a.p, i), r = ld_c<T>(a.r, i);
                p.re = r.re + be * p.re;
                p.im = r.im + be * p.im;
                st_c<T>(a.p, i, p);
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.state_out[0] = ns;
        if (left) atomicAdd(&a.ctl->n_running, -1);
    }
}

int launch_cg_update_fused(const VecArgs &a, int fp64, hipStream_t stream) {
    dim3 grid(site_blocks(a.Vh));
    if (fp64)
        cg_update_fused_kernel<double><<<grid, kBlock, 0, stream>>>(a);
    else
        cg_update_fused_kernel<float><<<grid, kBlock, 0, stream>>>(a);
    return 0;
}

int launch_p_update_fused(const VecArgs &a, int fp64, hipStream_t stream) {
    dim3 grid(site_blocks(a.Vh));
    if (fp64)
        p_update_fused_kernel<double><<<grid, kBlock, 0, stream>>>(a);
    else
        p_update_fused_kernel<float><<<grid, kBlock, 0, stream>>>(a);
    return 0;
}

// ---------------------------------------------------------------------------
// single-reduction CG (Chronopoulos and Gear; solver_state.hpp cgcg_step)
// ---------------------------------------------------------------------------
// One site's vectors of one system, and their update: p = r + beta p; s = w + beta s;
// x += alpha p; r -= alpha s; returns the site's |r_new|^2 in FP64.
template <typename T>
struct CgcgSite {
    vec3<T> r, w, p, sv, x;
    __device__ __forceinline__ void load(const VecArgs &a, size_t o, uint32_t h) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const size_t i = o + (size_t)c * a.Vh + h;
            r.c[c] = ld_c<T>(a.r, i);
            w.c[c] = ld_c<T>(a.w, i);
            p.c[c] = ld_c<T>(a.p, i);
            sv.c[c] = ld_c<T>(a.s, i);
            x.c[c] = ld_c<T>(a.x, i);
        }
    }
    __device__ __forceinline__ double update(const VecArgs &a, size_t o, uint32_t h, T al, T be) {
        double rr = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const size_t i = o + (size_t)c * a.Vh + h;
            p.c[c].re = r.c[c].re + be * p.c[c].re;
            p.c[c].im = r.c[c].im + be * p.c[c].im;
            sv.c[c].re = w.c[c].re + be * sv.c[c].re;
            sv.c[c].im = w.c[c].im + be * sv.c[c].im;
            x.c[c].re += al * p.c[c].re;
            x.c[c].im += al * p.c[c].im;
            r.c[c].re -= al * sv.c[c].re;
            r.c[c].im -= al * sv.c[c].im;
            st_c<T>(a.p, i, p.c[c]);
            st_c<T>(a.s, i, sv.c[c]);
            st_c<T>(a.x, i, x.c[c]);
            st_c<T>(a.r, i, r.c[c]);
            rr = fmat((double)r.c[c].re, (double)r.c[c].re, rr);
            rr = fmat((double)r.c[c].im, (double)r.c[c].im, rr);
        }
        return rr;
    }
};

template <typename T>
__global__ __launch_bounds__(kBlock) void cgcg_update_kernel(VecArgs a) {
    const int j = (int)blockIdx.y;
    const SysState &st = a.state[j];
    if (!(st.flags & SYS_RUNNING)) return;
    const uint32_t h = blockIdx.x * kBlock + threadIdx.x;
    double ps = 0.0, pc = 0.0;
    if (h < a.Vh) {
        CgcgSite<T> v;
        v.load(a, (size_t)j * a.fstride, h);
        pair_add(ps, pc, v.update(a, (size_t)j * a.fstride, h, (T)st.alpha, (T)st.beta), 0.0);
    }
    field_partials(a, j, ps, pc);
}

// Compensated sums of n (sum, error) pairs at x and of m at y by one wave in a fixed order,
// in every lane: lane l takes pairs l, l + 64, ..., then a tree across the lanes.
__device__ __forceinline__ void wave_totals(const double *x, uint32_t n, const double *y,
                                            uint32_t m, double &sx, double &sy) {
    double s = 0.0, c = 0.0, u = 0.0, v = 0.0;
    for (uint32_t i = threadIdx.x & 63; i < n; i += 64) pair_add(s, c, x[2 * i], x[2 * i + 1]);
    for (uint32_t i = threadIdx.x & 63; i < m; i += 64) pair_add(u, v, y[2 * i], y[2 * i + 1]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double s2 = __shfl_down(s, off, 64), c2 = __shfl_down(c, off, 64);
        const double u2 = __shfl_down(u, off, 64), v2 = __shfl_down(v, off, 64);
        pair_add(s, c, s2, c2);
        pair_add(u, v, u2, v2);
    }
    sx = __shfl(s + c, 0, 64);
    sy = __shfl(u + v, 0, 64);
}

// One field, no finalize kernel: every wave sums the hop's <r, w> partials and the
// previous update's |r|^2 partials in the same fixed order (bitwise the same totals),
// takes the scalar step on a copy of the state, and updates its sites; block 0 stores
// the new state in a.state_out (the next iteration's buffer, never a.state, which the
// other blocks are reading).  Block 0 always runs, so that a.state_out stays current.
// A breakdown or a system that parks leaves the vectors alone.
//
// On a small lattice the kernel is a chain of latencies, so the waves do without the
// block's barriers up to the last reduction (a wave sums the few hundred pairs itself;
// the state of this launch is not written by it, so its flags gate without one), and the
// site's vectors are loaded before the sums are waited for: 17.1 -> 16.4 us per
// iteration of 8^4 in FP64.
template <typename T>
__global__ __launch_bounds__(kBlock) void cgcg_update_fused_kernel(VecArgs a) {
    SysState ns = a.state[0];
    const bool closed = !(ns.flags & SYS_RUNNING);
    if (closed && blockIdx.x != 0) return;
    bool left = false;
    double ps[1] = {0.0}, pc[1] = {0.0};
    if (!closed) {
        const uint32_t h = blockIdx.x * kBlock + threadIdx.x;
        CgcgSite<T> v;
        if (h < a.Vh) v.load(a, 0, h);
        // just resumed: gamma comes from the state, the partials are stale
        double delta, gamma;
        wave_totals(a.fin_partials, a.fin_blocks, a.fin_partials2,
                    (ns.flags & SYS_RESUME) ? 0 : a.fin_blocks2, delta, gamma);
        left = cgcg_step(ns, delta, gamma);
        if (!left && h < a.Vh)
            pair_add(ps[0], pc[0], v.update(a, 0, h, (T)ns.alpha, (T)ns.beta), 0.0);
        block_partials<1>(ps, pc, a.partials);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.state_out[0] = ns;
        if (left) atomicAdd(&a.ctl->n_running, -1);
    }
}

int launch_cgcg_update(const VecArgs &a, int fp64, int nr, hipStream_t stream);
int launch_cgcg_update_fused(const VecArgs &a, int fp64, hipStream_t stream) {
    dim3 grid(site_blocks(a.Vh));
    if (fp64)
        cgcg_update_fused_kernel<double><<<grid, kBlock, 0, stream>>>(a);
    else
        cgcg_update_fused_kernel<float><<<grid, kBlock, 0, stream>>>(a);
    return 0;
}

// x64 += x32; x32 = 0 for parked systems
__global__ __launch_bounds__(kBlock) void ru_accumulate_kernel(VecArgs a) {
    const FieldSite f(a);
    if (!(a.state[f.j].flags & SYS_RU_PENDING) || !f.live) return;
    const vec3<float> xs = ld_site<float>(a.x, f.o, a.Vh);
    vec3<double> xd = ld_site<double>(a.x64, f.o, a.Vh);
    vec3<float> zero;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        xd.c[c].re += (double)xs.c[c].re;
        xd.c[c].im += (double)xs.c[c].im;
        zero.c[c] = {0.0f, 0.0f};
    }
    st_site<double>(a.x64, f.o, a.Vh, xd);
    st_site<float>(a.x, f.o, a.Vh, zero);
}

// resumed systems: r_inner = r64 (rounded to T); p = r_inner + beta p
template <typename T>
__global__ __launch_bounds__(kBlock) void ru_resume_kernel(VecArgs a) {
    const FieldSite f(a);
    const SysState &s = a.state[f.j];
    if (!(s.flags & SYS_RESUME) || !f.live) return;
    const T be = (T)s.beta;
    const vec3<double> rd = ld_site<double>(a.r64, f.o, a.Vh);
    vec3<T> r, p;
    if (!a.skip_p) p = ld_site<T>(a.p, f.o, a.Vh);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        r.c[c] = {(T)rd.c[c].re, (T)rd.c[c].im};
        if (a.skip_p) continue;
        p.c[c].re = r.c[c].re + be * p.c[c].re;
        p.c[c].im = r.c[c].im + be * p.c[c].im;
    }
    if (a.r != a.r64) st_site<T>(a.r, f.o, a.Vh, r);
    if (!a.skip_p) st_site<T>(a.p, f.o, a.Vh, p);
}

// multi-shift (Sec. 2.2, Eq. shlineq): base residual r = r_in - alpha q (the next slot of
// the ring of residuals); |r|^2 -> OP_MS_BETA
template <typename T>
__global__ __launch_bounds__(kBlock) void ms_r_update_kernel(VecArgs a) {
    const FieldSite f(a);
    const SysState &s = a.state[f.j];
    if (!(s.flags & SYS_RUNNING)) return;
    double ps = 0.0, pc = 0.0;
    if (f.live) {
        const T al = (T)s.alpha;
        vec3<T> r = ld_site<T>(a.r_in, f.o, a.Vh);
        const vec3<T> q = ld_site<T>(a.q, f.o, a.Vh);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            r.c[c].re -= al * q.c[c].re;
            r.c[c].im -= al * q.c[c].im;
            pair_add(ps, pc, (double)r.c[c].re * (double)r.c[c].re +
                                 (double)r.c[c].im * (double)r.c[c].im, 0.0);
        }
        st_site<T>(a.r, f.o, a.Vh, r);
    }
    field_partials(a, f.j, ps, pc);
}

// multi-shift, every M iterations: the steps of the shifted systems that the iterations
// left in a.steps (solver_state.hpp ShiftStep), x_k += alpha_k p_k with the old p_k, then
// p_k = zeta_k r + beta_k p_k with that iteration's base residual r, one slot of the ring
// a.r after the other.  The same operations in the same order as when every iteration
// updates the shifted vectors, but x_k and p_k are read and written once for M
// iterations: the update was bound by that traffic (4 vectors per active shift and
// iteration, 68 % of the stage's bytes with 16 shifts), which M = 8 divides by eight.
// 16^3 x 32, 10 poles x 4 RHS in FP64: 37.1 us per iteration with the base directions ->
// 48.8 / 8 + 7.2 (the whole solve 68.9 -> 52.2 ms); 24^3 x 48, 16 shifts x 2 RHS in FP32:
// 58.4 -> 106 / 8 + 8.5 us.
//
// One block works on one chunk of kBlock sites of one (shift, RHS) pair; a retired pair
// costs one scalar test per block.  The shift blocks of a chunk sit next to each other in
// the XCD-ordered block sequence: they run on the same XCD, where the residuals they all
// read stay in L2.  After a full ring one more block per chunk updates the base direction
// of that iteration, p = r + beta p (a.p), which saves a small lattice the launch.
template <typename T, int M>
__global__ __launch_bounds__(kBlock) void ms_shift_update_kernel(VecArgs a) {
    const uint32_t nk = (uint32_t)a.nshift + (a.p ? 1u : 0u);
    uint32_t b = xcd_block(blockIdx.x, gridDim.x);
    const uint32_t k = b % nk;
    b /= nk;
    const uint32_t nr = (uint32_t)a.nfields;
    const uint32_t j = b % nr;
    const uint32_t h = (b / nr) * kBlock + threadIdx.x;
    if (k == (uint32_t)a.nshift) {
        const SysState &s = a.state[j];
        if (!(s.flags & SYS_RUNNING) || h >= a.Vh) return;
        const T be = (T)s.beta;
        const size_t o = (size_t)j * a.fstride + h;
        const size_t last = (size_t)(a.nsteps - 1) * a.rstride;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const size_t i = o + (size_t)c * a.Vh;
            cpx<T> p = ld_c<T>(a.p, i), r = ld_c<T>(a.r, last + i);
            p.re = r.re + be * p.re;
            p.im = r.im + be * p.im;
            st_c<T>(a.p, i, p);
        }
        return;
    }
    const Ctl &ctl = *a.ctl;
    const size_t slot = (size_t)ctl.nshift * ctl.nrhs;  // entries per slot of steps
    const ShiftStep *st = ctl.steps + k * ctl.nrhs + a.state[j].gid;
    if (st[0].mode == 0 || h >= a.Vh) return;  // the modes of a pair never rise again
    const bool both = st[0].mode == 2;
    const size_t ir = (size_t)j * a.fstride + h, i = (size_t)k * a.kstride + ir;
    vec3<T> x, p, r[M];
#pragma unroll
    for (int c = 0; c < 3; ++c) x.c[c] = ld_c<T>(a.xs, i + (size_t)c * a.Vh);
#pragma unroll
    for (int c = 0; c < 3; ++c) p.c[c] = ld_c<T>(a.ps, i + (size_t)c * a.Vh);
    // the residuals of all the steps that need one are loaded before the first step
#pragma unroll
    for (int m = 0; m < M; ++m)
        if (m < a.nsteps && st[m * slot].mode == 2) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
                r[m].c[c] = ld_c<T>(a.r, (size_t)m * a.rstride + ir + (size_t)c * a.Vh);
        }
#pragma unroll
    for (int m = 0; m < M; ++m) {
        if (m >= a.nsteps) break;
        const ShiftStep &z = st[m * slot];
        if (z.mode == 0) break;
        const T ak = (T)z.alpha, zk = (T)z.zeta, bk = (T)z.beta;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x.c[c].re += ak * p.c[c].re;
            x.c[c].im += ak * p.c[c].im;
        }
        if (z.mode == 2) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                p.c[c].re = zk * r[m].c[c].re + bk * p.c[c].re;
                p.c[c].im = zk * r[m].c[c].im + bk * p.c[c].im;
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) st_c<T>(a.xs, i + (size_t)c * a.Vh, x.c[c]);
    if (both) {
#pragma unroll
        for (int c = 0; c < 3; ++c) st_c<T>(a.ps, i + (size_t)c * a.Vh, p.c[c]);
    }
}

// one launcher per kernel template: the precision is compile-time, the fields are grid.y
#define STG_VEC_LAUNCHER(NAME, KERNEL)                                                   \
    int NAME(const VecArgs &a, int fp64, int nr, hipStream_t stream) {                  \
        const dim3 grid(site_blocks(a.Vh), (uint32_t)nr);                                \
        if (fp64)                                                                        \
            KERNEL<double><<<grid, kBlock, 0, stream>>>(a);                              \
        else                                                                             \
            KERNEL<float><<<grid, kBlock, 0, stream>>>(a);                               \
        return 0;                                                                        \
    }

STG_VEC_LAUNCHER(launch_cg_update_only, cg_update_kernel)
STG_VEC_LAUNCHER(launch_p_update, p_update_kernel)
STG_VEC_LAUNCHER(launch_ru_resume, ru_resume_kernel)
STG_VEC_LAUNCHER(launch_ms_r_update_only, ms_r_update_kernel)
STG_VEC_LAUNCHER(launch_cgcg_update, cgcg_update_kernel)

int launch_cg_update(const VecArgs &a, int fp64, int nr, hipStream_t stream) {
    if (launch_cg_update_only(a, fp64, nr, stream)) return -1;
    FinArgs f{a.partials, site_blocks(a.Vh), nr, OP_BETA, a.gate_mask, a.ctl, a.state, nullptr};
    return launch_finalize(f, stream);
}

// grid: one block per (chunk of kBlock sites, field, shift or, with a.p, base direction)
int launch_ms_shift_update(const VecArgs &a, int fp64, int slots, hipStream_t stream) {
    dim3 grid(site_blocks(a.Vh) * (uint32_t)((a.nshift + (a.p ? 1 : 0)) * a.nfields));
    switch (slots * 2 + (fp64 ? 1 : 0)) {
        case 3: ms_shift_update_kernel<double, 1><<<grid, kBlock, 0, stream>>>(a); return 0;
        case 2: ms_shift_update_kernel<float, 1><<<grid, kBlock, 0, stream>>>(a); return 0;
        case 5: ms_shift_update_kernel<double, 2><<<grid, kBlock, 0, stream>>>(a); return 0;
        case 4: ms_shift_update_kernel<float, 2><<<grid, kBlock, 0, stream>>>(a); return 0;
        case 9: ms_shift_update_kernel<double, 4><<<grid, kBlock, 0, stream>>>(a); return 0;
        case 8: ms_shift_update_kernel<float, 4><<<grid, kBlock, 0, stream>>>(a); return 0;
        case 17: ms_shift_update_kernel<double, 8><<<grid, kBlock, 0, stream>>>(a); return 0;
        case 16: ms_shift_update_kernel<float, 8><<<grid, kBlock, 0, stream>>>(a); return 0;
        default: return -1;
    }
}

int launch_ms_r_update(const VecArgs &a, int fp64, int nr, hipStream_t stream) {
    if (launch_ms_r_update_only(a, fp64, nr, stream)) return -1;
    // no gate: the iteration's slot of the deferred shift steps is written in any case
    FinArgs f{a.partials, site_blocks(a.Vh), nr, OP_MS_BETA, 0, a.ctl, a.state, nullptr};
    f.slot = a.slot;
    return launch_finalize(f, stream);
}

// ---------------------------------------------------------------------------
// finishing the reductions: one block per system, fixed order, compensated
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void finalize_kernel(FinArgs f) {
    __shared__ double sh_red[2 * kWaves];
    const int j = blockIdx.x;
    // every thread reads its block's own system before the first barrier of the sum;
    // thread 0 changes it only after the last one
    if (f.gate_mask && !(f.state[j].flags & f.gate_mask)) return;
    double tot = block_sum2_pairs(f.partials + 2 * (size_t)j * f.nblocks, (int)f.nblocks, sh_red);
    double tot2 = 0.0;
    if (f.op == OP_CGCG)
        tot2 = block_sum2_pairs(f.partials2 + 2 * (size_t)j * f.nblocks2, (int)f.nblocks2, sh_red);
    if (f.op == OP_MS_ALPHA || f.op == OP_MS_BETA)
        finalize_ms_block(f.op, f.ctl, f.state, j, tot, f.slot);
    else if (threadIdx.x == 0)
        finalize_one(f.op, f.ctl, f.state, f.out, j, tot, tot2);
}

int launch_finalize(const FinArgs &f, hipStream_t stream) {
    finalize_kernel<<<f.nr, kBlock, 0, stream>>>(f);
    return 0;
}

int launch_ru_accumulate(const VecArgs &a, int nr, hipStream_t stream) {
    ru_accumulate_kernel<<<dim3(site_blocks(a.Vh), (uint32_t)nr), kBlock, 0, stream>>>(a);
    return 0;
}

// ---------------------------------------------------------------------------
// compensated complex dot product of one vector pair
// ---------------------------------------------------------------------------
constexpr uint32_t kDotMaxBlocks = 1024;

size_t dot_blocks(size_t n) {
    size_t b = (n + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    return b > kDotMaxBlocks ? kDotMaxBlocks : b;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void dot_kernel(size_t n, const void *x, const void *y,
                                                     double *partials) {
    // per-thread compensated accumulation of the real and imaginary parts
    double sr = 0.0, cr = 0.0, si = 0.0, ci = 0.0;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (size_t)gridDim.x * kBlock) {
        cpx<T> a = ld_c<T>(x, i), b = ld_c<T>(y, i);
        // conj(a) b; products of two floats are exact in double
        double pr1 = (double)a.re * (double)b.re, pr2 = (double)a.im * (double)b.im;
        double pi1 = (double)a.re * (double)b.im, pi2 = -(double)a.im * (double)b.re;
        double e;
        two_sum(sr, pr1, sr, e);
        cr += e;
        two_sum(sr, pr2, sr, e);
        cr += e;
        two_sum(si, pi1, si, e);
        ci += e;
        two_sum(si, pi2, si, e);
        ci += e;
    }
    double ps[2] = {sr, si}, pc[2] = {cr, ci};
    block_partials<2>(ps, pc, partials);
}

int launch_dot(int fp64, int nvec, size_t n, const void *x, const void *y, double *partials,
               Ctl *ctl, int op, SysState *state, double *out, hipStream_t stream) {
    const size_t esz = fp64 ? 16 : 8;
    dim3 grid((uint32_t)dot_blocks(n));
    for (int j = 0; j < nvec; ++j) {
        const char *xj = reinterpret_cast<const char *>(x) + (size_t)j * n * esz;
        const char *yj = reinterpret_cast<const char *>(y) + (size_t)j * n * esz;
        SysState *sj = state ? state + j : nullptr;
        double *oj = out ? out + 2 * j : nullptr;
        if (fp64)
            dot_kernel<double><<<grid, kBlock, 0, stream>>>(n, xj, yj, partials);
        else
            dot_kernel<float><<<grid, kBlock, 0, stream>>>(n, xj, yj, partials);
        // OP_STORE finishes both parts (re, im); the solver ops use the real part
        FinArgs f{partials, grid.x, op == OP_STORE ? 2 : 1, op, 0, ctl, sj, oj};
        launch_finalize(f, stream);
    }
    return 0;
}

// ---------------------------------------------------------------------------
// packing (Sec. 2.3: keep rows 0 and 1; Sec. 4.1 layouts)
// ---------------------------------------------------------------------------

// double -> bfloat16, round to nearest even, via round-to-odd float: the float
// keeps 16 more bits than bfloat16, so the second rounding is the correct one.
__device__ __forceinline__ uint32_t bf16_rne(double x) {
    float f = __double2float_rz(x);
    uint32_t u = __float_as_uint(f);
    if ((double)f != x) u |= 1u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

__global__ __launch_bounds__(kBlock) void pack_links_kernel(uint32_t Vh, const double2 *src,
                                                            int fmt, void *dst) {
    const uint32_t h = blockIdx.x * kBlock + threadIdx.x;
    const int s = blockIdx.y;
    if (h >= Vh) return;
    double2 e[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) e[a][b] = src[((size_t)(s * 3 + a) * 3 + b) * Vh + h];
    if (fmt == FMT_C128_18) {
        double2 *d = reinterpret_cast<double2 *>(dst);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) d[((size_t)(s * 3 + a) * 3 + b) * Vh + h] = e[a][b];
    } else if (fmt == FMT_C128_12) {
        double2 *d = reinterpret_cast<double2 *>(dst);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) d[((size_t)(s * 2 + a) * 3 + b) * Vh + h] = e[a][b];
    } else if (fmt == FMT_C64_12) {
        float4 *d = reinterpret_cast<float4 *>(dst);
        const double2 *flat = &e[0][0];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double2 u = flat[2 * k], v = flat[2 * k + 1];
            d[(size_t)(s * 3 + k) * Vh + h] =
                make_float4((float)u.x, (float)u.y, (float)v.x, (float)v.y);
        }
    } else {  // FMT_BF16_12
        const double2 *flat = &e[0][0];
        uint32_t w[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) w[k] = bf16_rne(flat[k].x) | (bf16_rne(flat[k].y) << 16);
        uint4 *da = reinterpret_cast<uint4 *>(dst);
        uint2 *db = reinterpret_cast<uint2 *>(da + (size_t)8 * Vh);
        da[(size_t)s * Vh + h] = make_uint4(w[0], w[1], w[2], w[3]);
        db[(size_t)s * Vh + h] = make_uint2(w[4], w[5]);
    }
}

int launch_pack_links(const Geom &g, const void *src, int fmt, void *dst, hipStream_t stream) {
    dim3 grid(site_blocks(g.Vh), 8);
    pack_links_kernel<<<grid, kBlock, 0, stream>>>(g.Vh, reinterpret_cast<const double2 *>(src),
                                                   fmt, dst);
    return 0;
}

__global__ __launch_bounds__(kBlock) void f64_to_f32_kernel(size_t n, const double *src,
                                                            float *dst) {
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (size_t)gridDim.x * kBlock)
        dst[i] = (float)src[i];
}

int launch_pack_phases_f32(size_t n, const double *src, float *dst, hipStream_t stream) {
    size_t b = (n + kBlock - 1) / kBlock;
    if (b > 65536) b = 65536;
    if (b < 1) b = 1;
    f64_to_f32_kernel<<<dim3((uint32_t)b), kBlock, 0, stream>>>(n, src, dst);
    return 0;
}

int launch_c128_to_c64(size_t n, const void *src, void *dst, hipStream_t stream) {
    return launch_pack_phases_f32(2 * n, reinterpret_cast<const double *>(src),
                                  reinterpret_cast<float *>(dst), stream);
}

__global__ __launch_bounds__(kBlock) void f32_to_f64_kernel(size_t n, const float *src,
                                                            double *dst) {
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (size_t)gridDim.x * kBlock)
        dst[i] = (double)src[i];
}

int launch_c64_to_c128(size_t n, const void *src, void *dst, hipStream_t stream) {
    size_t b = (2 * n + kBlock - 1) / kBlock;
    if (b > 65536) b = 65536;
    if (b < 1) b = 1;
    f32_to_f64_kernel<<<dim3((uint32_t)b), kBlock, 0, stream>>>(
        2 * n, reinterpret_cast<const float *>(src), reinterpret_cast<double *>(dst));
    return 0;
}

__global__ __launch_bounds__(kBlock) void zero_kernel(size_t n4, uint32_t *dst) {
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n4;
         i += (size_t)gridDim.x * kBlock)
        dst[i] = 0u;
}

int launch_zero(void *dst, size_t bytes, hipStream_t stream) {
    size_t n4 = bytes / 4;
    if (n4 == 0) return 0;
    size_t b = (n4 + kBlock - 1) / kBlock;
    if (b > 65536) b = 65536;
    zero_kernel<<<dim3((uint32_t)b), kBlock, 0, stream>>>(n4, reinterpret_cast<uint32_t *>(dst));
    return 0;
}

// ---------------------------------------------------------------------------
// rational function: y = a0 b + sum_k a_k x_k (FP64), one pass over the x_k
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void rational_sum_kernel(size_t n, int nshift, double a0,
                                                              const double *coeffs, const void *b,
                                                              const void *xs, void *y) {
    const size_t stride = (size_t)gridDim.x * kBlock;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        const cpx<double> bi = ld_c<double>(b, i);
        cpx<double> acc{a0 * bi.re, a0 * bi.im};
        for (int k = 0; k < nshift; ++k) {
            const double a = coeffs[k];
            const cpx<double> x = ld_c<double>(xs, (size_t)k * n + i);
            acc.re = fmat(a, x.re, acc.re);
            acc.im = fmat(a, x.im, acc.im);
        }
        st_c<double>(y, i, acc);
    }
}

int launch_rational_sum(size_t n, int nshift, double a0, const double *coeffs, const void *b,
                        const void *xs, void *y, hipStream_t stream) {
    size_t blocks = (n + kBlock - 1) / kBlock;
    if (blocks > 8192) blocks = 8192;
    if (blocks == 0) return 0;
    rational_sum_kernel<<<dim3((uint32_t)blocks), kBlock, 0, stream>>>(n, nshift, a0, coeffs, b,
                                                                      xs, y);
    return 0;
}

}  // namespace stg
