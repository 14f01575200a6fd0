// pt_grad.hip -- gradients of the window cost and the elite refinement built
// on them.
//
//   k_window_fwd      one wavefront per listed simulation: runs the window
//                     from a given start with the step code of the other
//                     kernels (same bits), the cost and optionally the end
//                     state; with a checkpoint buffer it records, before every
//                     step, the body and after the step's solve the kept
//                     contact keys and their impulses (float64)
//   k_window_bwd      the reverse sweep over those checkpoints: each step's
//                     contacts are rebuilt from the recorded keys (no narrow
//                     phase, no Newton solve), then the step adjoint runs
//                     (implicit differentiation of the contact solve).
//                     Output: the gradient of the window cost with respect
//                     to the start (x, q, v, w, m, mu, f)
//   (the elites come from the resampler's own ranking, k_rank)
//   k_refine_gather   the elites' window starts; the scaled gradient step is
//                     the reverse sweep's last act and keep-or-halve the
//                     forward sweep's (kernels of their own waited behind the
//                     sweeps that fill the GPU, 130 us a gradient step in
//                     parts that overlap: the real-time window 9.81 -> 9.72 ms)
#include <algorithm>

#include "pt_adjoint.hpp"
#include "pt_internal.h"
#include "pt_io.hpp"

namespace pt {

__device__ __forceinline__ void load_start(const float *__restrict__ xi, int n, int i, Body &B)
{
    B.x[0] = xi[0 * (size_t)n + i]; B.x[1] = xi[1 * (size_t)n + i]; B.x[2] = xi[2 * (size_t)n + i];
    B.q[0] = xi[3 * (size_t)n + i]; B.q[1] = xi[4 * (size_t)n + i]; B.q[2] = xi[5 * (size_t)n + i];
    B.q[3] = xi[6 * (size_t)n + i];
    B.v[0] = xi[7 * (size_t)n + i]; B.v[1] = xi[8 * (size_t)n + i]; B.v[2] = xi[9 * (size_t)n + i];
    B.w[0] = xi[10 * (size_t)n + i]; B.w[1] = xi[11 * (size_t)n + i]; B.w[2] = xi[12 * (size_t)n + i];
    B.m = xi[13 * (size_t)n + i]; B.mu = xi[14 * (size_t)n + i];
    B.f[0] = xi[15 * (size_t)n + i]; B.f[1] = xi[16 * (size_t)n + i]; B.f[2] = xi[17 * (size_t)n + i];
}

// xi is [18][n]: x(3) q(4) v(3) w(3) m mu f(3); warm0 is [n][C_max][4]
// One launch covers `count` listed simulations i0 .. i0+count-1 of arrays
// with row stride n; the checkpoint buffer holds `count` simulations.
template <typename SR, bool PT>
__global__ __launch_bounds__(WAVE) void k_window_fwd(Consts P, Tables tb, const float *__restrict__ seg_win, int n,
                                                     int i0, int count,
                                                     const int32_t *__restrict__ env, const float *__restrict__ xi,
                                                     const float *__restrict__ warm0,
                                                     const float *__restrict__ obs_gt_win, float *__restrict__ cost_out,
                                                     float *__restrict__ end_state, float *__restrict__ end_warm,
                                                     float *__restrict__ ckpt, float *__restrict__ resid_out,
                                                     RefineKeep keep)
{
    extern __shared__ __align__(16) char smem[];
    const int c = blockIdx.x;
    if (c >= count) return;
    const int i = i0 + c;
    const int lane = lane_id();
    const int e = env[i];
    if (e < 0 || e >= P.K) {
        // not a simulation of this batch
        if (lane == 0 && cost_out) cost_out[i] = __int_as_float(0x7fc00000);
        return;
    }
    WaveLds lds = carve_lds(smem, 0, P.max_cand, 0);
    float *stage = contact_stage(lds);
    const int type = tb.env_type[e];
    const int g = tb.group_of[e];
    const int S = tb.n_spheres[type];
    const float *sph = tb.spheres + (size_t)type * P.S_max * 4;
    const float reach = tb.reach[type];
    const float inv[3] = {tb.inv_inertia[3 * type], tb.inv_inertia[3 * type + 1], tb.inv_inertia[3 * type + 2]};
    const size_t LG = (size_t)P.L * P.G;
    const size_t CK = ckpt_step_floats(P.C_max);

    Body B;
    load_start(xi, n, i, B);
    int wkey;
    float wr[3];
    load_warm(warm0, P.C_max, i, wkey, wr);
    StepStats stt = {0, 0, 0};

    // cost summed in the order of the other paths; the largest final merit
    // of the window's contact solves (how far they are from the root the
    // reverse sweep assumes)
    float cost = 0.f, resid = 0.f;
    for (int t = 0; t < P.T; ++t) {
        float *ck = ckpt ? ckpt + ((size_t)c * P.T + t) * CK : nullptr;
        if (ck) save_body(ck, B);
        const float *seg = seg_win + (size_t)t * P.L * SEG_STRIDE;
        StepState<SR> st;
        step_setup<SR>(P, seg, sph, S, inv, B, reach, wkey, wr, lds, stt, st);
        step_solve<SR, PT>(P, st, B.mu, inv, reinterpret_cast<SR *>(lds.cand));
        resid = fmaxf(resid, (float)st.psi_end);
        if (ck) save_contact<SR>(ck, P.C_max, st);
        int link;
        float imp[3];
        step_finish<SR>(P, st, inv, B, wkey, wr, link, imp);
        uniform_body(B);
        *reinterpret_cast<float4 *>(stage + 4 * lane) = make_float4(__int_as_float(link), imp[0], imp[1], imp[2]);
        wave_sync();
        float o[4];
        float cl = 0.f;
        if (sensor_force(P, stage, link, o)) {
            const float *gt = obs_gt_win + (size_t)t * 4 * LG;
            float gv[4] = {gt[0 * LG + (size_t)lane * P.G + g], gt[1 * LG + (size_t)lane * P.G + g],
                           gt[2 * LG + (size_t)lane * P.G + g], gt[3 * LG + (size_t)lane * P.G + g]};
            cl = sensor_cost(P, o, gv);
        }
        wave_sync();
        cost += step_cost_wave(P, cl);
    }
    if (keep.cost) {
        // an elite's trial: kept where its window cost is lower (the batch
        // slot then takes the replay's end of window, the trial's mass and
        // friction, and its cost; flag = 1 asks for the gradient at the new
        // start), otherwise the step is halved (flag = 0)
        const bool kept = cost < keep.cost[i];
        if (lane == 0) {
            keep.flag[i] = kept ? 1 : 0;
            if (kept) {
                keep.cost[i] = cost;
                keep.cost_sum[e] = cost;
                keep.params[e] = B.m;
                keep.params[(size_t)P.K + e] = B.mu;
            } else {
                keep.rho[i] *= 0.5f;
            }
        }
        if (kept) {
            if (lane < XI_ROWS) keep.xi[(size_t)lane * n + i] = xi[(size_t)lane * n + i];
            store_body(keep.state, keep.params, P.K, e, B);   // f is 0 after a step
            store_warm(keep.warm, P.C_max, e, wkey, wr);
        }
        return;
    }
    if (lane == 0) {
        cost_out[i] = cost;
        if (resid_out) resid_out[i] = resid;
        if (end_state) {
            const float v13[13] = {B.x[0], B.x[1], B.x[2], B.q[0], B.q[1], B.q[2], B.q[3],
                                   B.v[0], B.v[1], B.v[2], B.w[0], B.w[1], B.w[2]};
            for (int r = 0; r < 13; ++r) end_state[(size_t)r * n + i] = v13[r];
        }
    }
    if (end_warm) store_warm(end_warm, P.C_max, i, wkey, wr);
}

// trial start of elite i: xi - rho (s o s o g) / |s o g| over (x, q, v, w, m,
// mu), then q renormalised and m, mu clamped; the one-step force is kept
__device__ __forceinline__ void refine_propose(const RefineTry &R, const float *__restrict__ xi,
                                               const float (&grad)[XI_ROWS], int n, int i)
{
    const RefineArgs &A = R.args;
    float x[XI_ROWS];
    for (int r = 0; r < XI_ROWS; ++r) x[r] = xi[(size_t)r * n + i];
    float sg2 = 0.f;
    for (int r = 0; r < 15; ++r) {
        float v = A.scale[r] * grad[r];
        sg2 += v * v;
    }
    const float nrm = sqrtf(sg2);
    if (nrm > 0.f && nrm < __int_as_float(0x7f800000)) {
        const float f = R.rho[i] / nrm;
        for (int r = 0; r < 15; ++r) x[r] -= f * A.scale[r] * A.scale[r] * grad[r];
        const float qn = sqrtf(x[3] * x[3] + x[4] * x[4] + x[5] * x[5] + x[6] * x[6]);
        if (qn > 0.f)
            for (int r = 3; r < 7; ++r) x[r] /= qn;
        x[13] = fminf(fmaxf(x[13], A.m_lo), A.m_hi);
        x[14] = fminf(fmaxf(x[14], A.mu_lo), A.mu_hi);
    }
    if (lane_id() == 0)
        for (int r = 0; r < XI_ROWS; ++r) R.xi_try[(size_t)r * n + i] = x[r];
}

// reverse sweep over the checkpoints k_window_fwd wrote for the same n, env
// and xi (ckpt_by_env = 0: slot c of the launch), or that the population's
// window wrote (ckpt_by_env = 1: slot env[i]); simulations with flag[i] == 0
// keep their gradient (flag may be NULL); with refine.xi_try the next trial
// start is proposed from it, swept or kept
template <typename SR>
__global__ __launch_bounds__(WAVE) void k_window_bwd(Consts P, Tables tb, const float *__restrict__ seg_win, int n,
                                                     int i0, int count,
                                                     const int32_t *__restrict__ env, const float *__restrict__ xi,
                                                     const float *__restrict__ obs_gt_win,
                                                     const float *__restrict__ ckpt, int ckpt_by_env,
                                                     const int32_t *__restrict__ flag, float *__restrict__ grad,
                                                     RefineTry refine)
{
    extern __shared__ __align__(16) char smem[];
    const int c = blockIdx.x;
    if (c >= count) return;
    const int i = i0 + c;
    if (flag && flag[i] == 0) {
        if (refine.xi_try) {
            float g[XI_ROWS];
            for (int r = 0; r < XI_ROWS; ++r) g[r] = grad[(size_t)r * n + i];
            refine_propose(refine, xi, g, n, i);
        }
        return;
    }
    const int lane = lane_id();
    const int e = env[i];
    if (e < 0 || e >= P.K) {
        if (lane == 0)
            for (int r = 0; r < XI_ROWS; ++r) grad[(size_t)r * n + i] = 0.f;
        return;
    }
    // the sum rows whole in the list: the adjoint stages data in the words after it
    WaveLds lds = carve_lds(smem, 0, P.max_cand_rows, 0);
    float *stage = contact_stage(lds);
    const int type = tb.env_type[e];
    const int g = tb.group_of[e];
    const float *sph = tb.spheres + (size_t)type * P.S_max * 4;
    const float inv[3] = {tb.inv_inertia[3 * type], tb.inv_inertia[3 * type + 1], tb.inv_inertia[3 * type + 2]};
    const size_t LG = (size_t)P.L * P.G;
    const size_t CK = ckpt_step_floats(P.C_max);
    const float m0 = xi[13 * (size_t)n + i], mu0 = xi[14 * (size_t)n + i];

    BodyBar<SR> bar;
#pragma unroll
    for (int k = 0; k < 3; ++k) bar.x[k] = bar.v[k] = bar.w[k] = SR(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) bar.q[k] = SR(0);
    SR mbar = 0, mubar = 0, fbar[3] = {0, 0, 0};
    for (int t = P.T - 1; t >= 0; --t) {
        const float *ck = ckpt + ((size_t)(ckpt_by_env ? e : c) * P.T + t) * CK;
        Body B;
        load_body_ckpt(ck, B);
        B.m = m0;
        B.mu = mu0;
        SR r[3];
        const int key = load_contact<SR>(ck, P.C_max, r);
        const float *seg = seg_win + (size_t)t * P.L * SEG_STRIDE;
        // the step as the forward sweep left it: same contacts, same impulses
        StepState<SR> st;
        step_pose<SR>(P, inv, B, st);
        contact_setup<SR>(P, seg, sph, B, key, st);
        const int C = __popcll(__ballot(st.act));
        st.C = C;
        st.ncand = C;
        st.span = lane_span(C);
        st.r[0] = r[0]; st.r[1] = r[1]; st.r[2] = r[2];
        body_dv(st, st.r, st.nu);
        st.nu[0] += st.vs[0]; st.nu[1] += st.vs[1]; st.nu[2] += st.vs[2];
        st.nu[3] += st.ws[0]; st.nu[4] += st.ws[1]; st.nu[5] += st.ws[2];
        step_adjoint<SR>(P, seg, sph, inv, B, st, obs_gt_win + (size_t)t * 4 * LG, g, stage, lds.wr,
                         reinterpret_cast<SR *>(lds.cand), bar, mbar, mubar, t == 0 ? fbar : nullptr);
    }
    const float gv[XI_ROWS] = {(float)bar.x[0], (float)bar.x[1], (float)bar.x[2], (float)bar.q[0], (float)bar.q[1],
                               (float)bar.q[2], (float)bar.q[3], (float)bar.v[0], (float)bar.v[1], (float)bar.v[2],
                               (float)bar.w[0], (float)bar.w[1], (float)bar.w[2], (float)mbar,     (float)mubar,
                               (float)fbar[0],  (float)fbar[1],  (float)fbar[2]};
    if (lane == 0)
        for (int r = 0; r < XI_ROWS; ++r) grad[(size_t)r * n + i] = gv[r];
    if (refine.xi_try) refine_propose(refine, xi, gv, n, i);
}

// start of each listed simulation from the window-start snapshot (and, if
// cost_sum is given, its window cost): one row entry or warm-cache slot per
// thread
__global__ __launch_bounds__(256) void k_refine_gather(int n, int K, int C_max, const int32_t *__restrict__ env,
                                                       const float *__restrict__ state, const float *__restrict__ params,
                                                       const float *__restrict__ warm, const float *__restrict__ cost_sum,
                                                       float *__restrict__ xi, float *__restrict__ warm0,
                                                       float *__restrict__ cost, float *__restrict__ rho, float rho0)
{
    const int rows = XI_ROWS * n, total = rows + n * C_max;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < total; x += gridDim.x * blockDim.x) {
        const bool row = x < rows;
        const int i = row ? x % n : (x - rows) / C_max, r = row ? x / n : x - rows - i * C_max;
        const int e = env[i];
        if (e < 0 || e >= K) continue;
        if (!row) {
            reinterpret_cast<float4 *>(warm0)[(size_t)i * C_max + r] =
                reinterpret_cast<const float4 *>(warm)[(size_t)e * C_max + r];
            continue;
        }
        xi[x] = r < 13 ? state[(size_t)r * K + e] : params[(size_t)(r - 13) * K + e];
        if (r == 0) {
            rho[i] = rho0;
            if (cost_sum) cost[i] = cost_sum[e];
        }
    }
}

}  // namespace pt

using namespace pt;

size_t ckpt_floats(const Consts &P, int n) { return (size_t)n * P.T * ckpt_step_floats(P.C_max); }

hipError_t launch_window_fwd(const Consts &P, const Tables &tb, const float *seg_win, int n, int i0, int count,
                             const int32_t *env, const float *xi, const float *warm0, const float *obs_gt_win,
                             float *cost, float *end_state, float *end_warm, float *ckpt, hipStream_t s,
                             float *resid, const RefineKeep *keep)
{
    if (count <= 0) return hipSuccess;
    size_t lds = wave_lds_bytes(P.max_cand, 0);
    // paired line-search trials when no step can hold more than 32 contacts
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(count), dim3(WAVE), lds, s, P, tb, seg_win, n, i0, count, env, xi, warm0,
                           obs_gt_win, cost, end_state, end_warm, ckpt, resid, keep ? *keep : RefineKeep());
        return hipGetLastError();
    };
    const bool pt = P.C_max <= 32;
    if (P.solve_fp64) return pt ? go(k_window_fwd<double, true>) : go(k_window_fwd<double, false>);
    return pt ? go(k_window_fwd<float, true>) : go(k_window_fwd<float, false>);
}

hipError_t launch_window_bwd(const Consts &P, const Tables &tb, const float *seg_win, int n, int i0, int count,
                             const int32_t *env, const float *xi, const float *obs_gt_win, const float *ckpt,
                             bool ckpt_by_env, const int32_t *flag, float *grad, hipStream_t s, const RefineTry *refine)
{
    if (count <= 0) return hipSuccess;
    size_t lds = wave_lds_bytes(P.max_cand_rows, 0);
    const int by_env = ckpt_by_env ? 1 : 0;
    const RefineTry next = refine ? *refine : RefineTry();
    if (P.solve_fp64)
        hipLaunchKernelGGL(k_window_bwd<double>, dim3(count), dim3(WAVE), lds, s, P, tb, seg_win, n, i0, count, env,
                           xi, obs_gt_win, ckpt, by_env, flag, grad, next);
    else
        hipLaunchKernelGGL(k_window_bwd<float>, dim3(count), dim3(WAVE), lds, s, P, tb, seg_win, n, i0, count, env,
                           xi, obs_gt_win, ckpt, by_env, flag, grad, next);
    return hipGetLastError();
}

hipError_t launch_refine_gather(int n, int K, int C_max, const int32_t *env, const float *state, const float *params,
                                const float *warm, const float *cost_sum, float *xi, float *warm0, float *cost,
                                float *rho, float rho0, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_refine_gather, dim3(std::min<size_t>(((size_t)n * (XI_ROWS + C_max) + 255) / 256, 4096)),
                       dim3(256), 0, s, n, K, C_max, env, state, params, warm,
                       cost_sum, xi, warm0, cost, rho, rho0);
    return hipGetLastError();
}

hipError_t set_grad_lds_limits(size_t bytes)
{
    const void *fs[] = {reinterpret_cast<const void *>(k_window_fwd<float, false>),
                        reinterpret_cast<const void *>(k_window_fwd<double, false>),
                        reinterpret_cast<const void *>(k_window_fwd<float, true>),
                        reinterpret_cast<const void *>(k_window_fwd<double, true>),
                        reinterpret_cast<const void *>(k_window_bwd<float>),
                        reinterpret_cast<const void *>(k_window_bwd<double>)};
    for (const void *f : fs) {
        hipError_t e = set_dynamic_lds_limit(f, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
