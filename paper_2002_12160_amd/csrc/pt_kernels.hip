// pt_kernels.hip -- HIP kernels of libpt for CDNA4 (gfx950).
//
//   k_hand_fk      forward kinematics of the kinematic hand, once per step
//                  (shared by every simulation: the same command u_t drives
//                  all of them, Alg. 1)
//   k_step         plain path: one simulation step per wavefront; contacts
//                  written to HBM for the observation kernel
//   k_observe      per-sensor contact force of the last step
//   k_cost         step cost against the observed force, running sum (Eq. 1)
//   k_argmin       per-group argmin of the running cost (Eq. 2)
//   k_rank         the groups' simulations ranked by running cost
//   k_resample     population-based resampling with Philox4x32-10 (Sec. III-D.3)
//   k_window       batched path: persistent kernel running T steps with the
//                  observation and cost fused, state kept on chip
#include <algorithm>

#include "pt_internal.h"
#include "pt_io.hpp"

namespace pt {

// ---------------------------------------------------------------------
// hand kinematics (double precision: it runs once per step for the whole
// population, and the link velocities are differences of positions)
// ---------------------------------------------------------------------
// Joint rotation of a link for joint vector u, Rot(axis0, u[j0]) Rot(axis1,
// u[j1]) (identity for a joint index < 0), by a pair of adjacent lanes: lane
// j of the pair (j = 0, 1) evaluates the half-angle rotation of joint j, the
// odd lane's moves to the even one (DPP, quad_perm [1,0,3,2]), which composes
// the two and writes them to qj.  Both lanes of the pair must be active.
__device__ __forceinline__ void fk_joint_pair(const float *__restrict__ h, const float *__restrict__ u, int j,
                                              double *qj)
{
    const int jx = (int)h[1 + j];
    const float *ax = h + 3 + 3 * j;
    double q[4] = {1, 0, 0, 0};
    if (jx >= 0) {
        double s, c;
        sincos(0.5 * (double)u[jx], &s, &c);
        q[0] = c; q[1] = s * ax[0]; q[2] = s * ax[1]; q[3] = s * ax[2];
    }
    double r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = dpp_f<0xb1, 0xf>(q[i]);
    if (j == 0) {
        if ((int)h[2] >= 0) {
            double t[4];
            quat_mul_d(q, r, t);
            for (int i = 0; i < 4; ++i) q[i] = t[i];
        }
        for (int i = 0; i < 4; ++i) qj[i] = q[i];
    }
}

// pose of link l in configuration w from its parent's (already computed):
// origin, orientation and the segment [a, b] along the link's local +x axis
__device__ __forceinline__ void fk_link(const float *__restrict__ h, int parent, const double *qj, double *tq, double *tp,
                        double *seg_a, double *seg_b, int l)
{
    double pq[4] = {1, 0, 0, 0}, pp[3] = {0, 0, 0};
    if (parent >= 0) {
        for (int i = 0; i < 4; ++i) pq[i] = tq[4 * parent + i];
        for (int i = 0; i < 3; ++i) pp[i] = tp[3 * parent + i];
    }
    double Rp[9];
    quat_to_mat_d(pq, Rp);
    double off[3] = {h[9], h[10], h[11]};
    double o[3] = {pp[0] + Rp[0] * off[0] + Rp[1] * off[1] + Rp[2] * off[2],
                   pp[1] + Rp[3] * off[0] + Rp[4] * off[1] + Rp[5] * off[2],
                   pp[2] + Rp[6] * off[0] + Rp[7] * off[1] + Rp[8] * off[2]};
    double qo[4] = {h[12], h[13], h[14], h[15]};
    double q0[4], q[4];
    quat_mul_d(pq, qo, q0);
    quat_mul_d(q0, qj + 4 * l, q);
    double len = h[16];
    // local +x axis of the link frame
    double xa[3] = {1 - 2 * (q[2] * q[2] + q[3] * q[3]), 2 * (q[1] * q[2] + q[0] * q[3]),
                    2 * (q[1] * q[3] - q[0] * q[2])};
    double b[3] = {o[0] + len * xa[0], o[1] + len * xa[1], o[2] + len * xa[2]};
    for (int i = 0; i < 4; ++i) tq[4 * l + i] = q[i];
    for (int i = 0; i < 3; ++i) {
        tp[3 * l + i] = b[i];
        seg_a[3 * l + i] = o[i];
        seg_b[3 * l + i] = b[i];
    }
}

// LDS of one evaluation of the hand kinematics: the link table, the link
// depths, and for both configurations the joint rotations, link frames and
// segment ends (double)
struct FkLds {
    float *hs;
    int *depth;
    float *su;       // [2][Ds] staged joint commands (u_prev, u), Ds = fk_staged_joints(D)
    double *cf;      // per configuration w: cf + 17 L w = [qj 4L | tq 4L | tp 3L | sa 3L | sb 3L]
    int L;
    __device__ double *qj(int w) const { return cf + (size_t)17 * L * w; }
    __device__ double *tq(int w) const { return cf + (size_t)17 * L * w + 4 * L; }
    __device__ double *tp(int w) const { return cf + (size_t)17 * L * w + 8 * L; }
    __device__ double *sa(int w) const { return cf + (size_t)17 * L * w + 11 * L; }
    __device__ double *sb(int w) const { return cf + (size_t)17 * L * w + 14 * L; }
};

// joint commands staged in LDS (every command, read before the link table
// says which ones are used); past 2 MAX_LINKS of them they are read from
// global memory where needed
__host__ __device__ constexpr int fk_staged_joints(int D) { return D <= 2 * MAX_LINKS ? D : 0; }

__host__ __device__ constexpr size_t fk_head_bytes(int L, int D)
{
    return ((size_t)L * (4 * HAND_STRIDE + 4) + (size_t)8 * fk_staged_joints(D) + 7) & ~(size_t)7;
}

__host__ __device__ constexpr size_t fk_lds_bytes(int L, int D) { return fk_head_bytes(L, D) + (size_t)L * 2 * 17 * 8; }

__device__ __forceinline__ FkLds carve_fk(char *p, int L, int D)
{
    FkLds s;
    s.hs = reinterpret_cast<float *>(p);
    s.depth = reinterpret_cast<int *>(s.hs + (size_t)L * HAND_STRIDE);
    s.su = reinterpret_cast<float *>(s.depth + L);
    s.cf = reinterpret_cast<double *>(p + fk_head_bytes(L, D));
    s.L = L;
    return s;
}

// Hand kinematics of one step by nt cooperating threads (tid in [0, nt), nt
// even, a wavefront's lanes in order): the link table staged in LDS, the joint
// rotations (the transcendental part) one thread per (configuration, link,
// joint), the chains composed level by
// level of the link tree (links at one depth in parallel, both
// configurations at once), then the segment record of every link: a,
// b - a, the radius, 1/|b - a|^2 and the end-point velocities
// (FK(u) - FK(u_prev)) / dt.  sync() orders the LDS between the stages.
// Every value is computed by the same code whichever threads run it, so a
// workgroup and a wavefront produce the same bits.
template <typename Sync>
__device__ __forceinline__ void hand_kinematics(const float *__restrict__ hand, int L, int D, float dt,
                                                const float *__restrict__ u_prev, const float *__restrict__ u,
                                                const FkLds &s, float *seg_out, int tid, int nt, Sync sync)
{
    const int Ds = fk_staged_joints(D);
    // the loads in flight together before their LDS writes: the commands,
    // then the link table eight per thread at a time (one round trip to
    // memory for a table of up to 8 nt floats, not one per element)
    float up0 = 0.f, uu0 = 0.f;
    if (tid < Ds) {
        up0 = u_prev[tid];
        uu0 = u[tid];
    }
    const int nh = L * HAND_STRIDE;
    for (int i0 = tid; i0 < nh; i0 += 8 * nt) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = hand[min(i0 + k * nt, nh - 1)];   // in bounds, no branch
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (i0 + k * nt < nh) s.hs[i0 + k * nt] = v[k];
    }
    if (tid < Ds) {
        s.su[tid] = up0;
        s.su[Ds + tid] = uu0;
    }
    for (int i = tid + nt; i < Ds; i += nt) {
        s.su[i] = u_prev[i];
        s.su[Ds + i] = u[i];
    }
    sync();
    for (int l = tid; l < L; l += nt) {
        // parents precede children (checked at batch creation), so the walk ends
        int d = 0, p = (int)s.hs[l * HAND_STRIDE];
        while (p >= 0) {
            ++d;
            p = (int)s.hs[p * HAND_STRIDE];
        }
        s.depth[l] = d;
    }
    // thread pairs (2m, 2m + 1) share an iteration (4 L and nt are even)
    for (int i = tid; i < 4 * L; i += nt) {
        const int w = i / (2 * L), r = i - w * 2 * L, l = r >> 1;
        const float *uw = Ds > 0 ? s.su + w * Ds : (w == 0 ? u_prev : u);
        fk_joint_pair(s.hs + l * HAND_STRIDE, uw, r & 1, s.qj(w) + 4 * l);
    }
    sync();
    int dmax = 0;
    for (int l = 0; l < L; ++l) dmax = max(dmax, s.depth[l]);
    for (int d = 0; d <= dmax; ++d) {
        for (int i = tid; i < 2 * L; i += nt) {
            int w = i / L, l = i - w * L;
            if (s.depth[l] == d)
                fk_link(s.hs + l * HAND_STRIDE, (int)s.hs[l * HAND_STRIDE], s.qj(w), s.tq(w), s.tp(w), s.sa(w),
                        s.sb(w), l);
        }
        sync();
    }
    const double idt = 1.0 / (double)dt;
    for (int l = tid; l < L; l += nt) {
        float *o = seg_out + (size_t)l * SEG_STRIDE;
        float a0[3], ab[3];
        const double *sa0 = s.sa(0), *sb0 = s.sb(0), *sa1 = s.sa(1), *sb1 = s.sb(1);
        for (int i = 0; i < 3; ++i) {
            a0[i] = (float)sa0[3 * l + i];
            ab[i] = (float)(sb0[3 * l + i] - sa0[3 * l + i]);
        }
        float L2 = ab[0] * ab[0] + ab[1] * ab[1] + ab[2] * ab[2];
        float inv = sqrtf(L2) >= 1e-9f ? 1.f / L2 : 0.f;
        for (int i = 0; i < 3; ++i) {
            o[i] = a0[i];
            o[4 + i] = ab[i];
            o[8 + i] = (float)((sa1[3 * l + i] - sa0[3 * l + i]) * idt);
            o[12 + i] = (float)((sb1[3 * l + i] - sb0[3 * l + i]) * idt);
        }
        o[3] = s.hs[l * HAND_STRIDE + 17];
        o[7] = inv;
        o[11] = 0.f;
        o[15] = 0.f;
    }
}

// grid: one block per step; u_prev/u for step t at u_prev + t*stride
__global__ __launch_bounds__(128) void k_hand_fk(const float *__restrict__ hand, int L, int D, float dt,
                                                 const float *__restrict__ u_prev, const float *__restrict__ u,
                                                 int stride, float *__restrict__ seg_out)
{
    __shared__ __align__(16) char fk[fk_lds_bytes(MAX_LINKS, 2 * MAX_LINKS)];
    const int t = blockIdx.x;
    const FkLds s = carve_fk(fk, L, D);
    hand_kinematics(hand, L, D, dt, u_prev + (size_t)t * stride, u + (size_t)t * stride, s,
                    seg_out + (size_t)t * L * SEG_STRIDE, threadIdx.x, blockDim.x, [] { __syncthreads(); });
}


// ---------------------------------------------------------------------
// plain path
// ---------------------------------------------------------------------
// float64 solves need more registers than a 512-thread block leaves a wave
template <typename SR>
struct StepBounds {
    static constexpr int threads = sizeof(SR) == 8 ? 256 : 512;
};

// EQ3: the observation of Eq. 3 (cost_mode 1) compiled in; the default
// force-only kernels carry none of its registers.  SDF: links against the
// object's distance field (collision_mode 1).  SEGIN: the step's hand
// segments come from k_hand_fk (in seg_out) instead of every wavefront's own
// hand kinematics -- the same bits, one evaluation per step instead of one
// per simulation, for launches that fill the GPU
template <typename SR, bool EQ3, bool SDF = false, bool SEGIN = false>
__global__ __launch_bounds__(StepBounds<SR>::threads) void k_step(Consts P, Tables tb,
                                               const float *__restrict__ u_prev, const float *__restrict__ u,
                                               float *__restrict__ state, float *__restrict__ params,
                                               float *__restrict__ warm, float *__restrict__ contacts,
                                               float *__restrict__ cslip, float *__restrict__ seg_out,
                                               int64_t *__restrict__ stats)
{
    extern __shared__ __align__(16) char smem[];
    // the simulation index is wave-uniform: its per-simulation loads go
    // through scalar registers
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int e = xcd_block(blockIdx.x, gridDim.x) * (blockDim.x / WAVE) + wib;
    if (e >= P.K) return;
    WaveLds lds = carve_lds(smem, wib, P.max_cand, SEGIN ? 0 : P.L);
    const int type = tb.env_type[e];
    const int S = tb.n_spheres[type];
    const float *sph = tb.spheres + (size_t)type * P.S_max * 4;
    const float reach = tb.reach[type];
    const float inv[3] = {tb.inv_inertia[3 * type], tb.inv_inertia[3 * type + 1], tb.inv_inertia[3 * type + 2]};
    const float rows = load_body_rows(state, params, P.K, e);
    int wkey;
    float wr[3];
    load_warm(warm, P.C_max, e, wkey, wr);
    // otherwise every wavefront evaluates the step's hand kinematics itself
    // (the candidate list's LDS as scratch), while its state loads are in
    // flight: no launch of its own on the per-step path, and the same bits
    // as k_hand_fk
    if (!SEGIN)
        hand_kinematics(tb.hand, P.L, P.D, P.dt, u_prev, u,
                        carve_fk(reinterpret_cast<char *>(lds.cand), P.L, P.D), lds.seg, lane_id(), WAVE,
                        [] { wave_sync(); });
    Body B;
    body_from_rows(rows, B);
    const float *seg = SEGIN ? seg_out : lds.seg;
    StepStats st = {0, 0, 0};
    int link;
    float imp[3];
    StepState<SR> sst;
    SdfRef sdf;
    if (SDF) {
        sdf.v = tb.sdf + (size_t)type * P.sdf_n * P.sdf_n * P.sdf_n;
        sdf.box = tb.sdf_box + 4 * type;
        sdf.n = P.sdf_n;
        sdf.M = P.link_samples;
    }
    step_setup<SR, SDF>(P, seg, sph, S, inv, B, reach, wkey, wr, lds, st, sst, sdf);
    step_solve<SR, true>(P, sst, B.mu, inv, reinterpret_cast<SR *>(lds.cand));
    step_finish<SR>(P, sst, inv, B, wkey, wr, link, imp);
    const int lane = lane_id();
    if (EQ3) {
        // Eq. 3's slip data of every contact, and the step's segments (one
        // wavefront) for the observation kernel
        float rec[SLIP_STRIDE];
        slip_record<SR>(sst, seg, B.w, rec);
        if (lane < P.C_max) {
            float4 *o = reinterpret_cast<float4 *>(cslip + ((size_t)e * P.C_max + lane) * SLIP_STRIDE);
            o[0] = make_float4(rec[0], rec[1], rec[2], rec[3]);
            o[1] = make_float4(rec[4], rec[5], rec[6], rec[7]);
        }
        if (!SEGIN && e == 0)
            for (int i = lane; i < P.L * SEG_STRIDE; i += WAVE) seg_out[i] = seg[i];
    }
    store_body(state, params, P.K, e, B);
    store_warm(warm, P.C_max, e, wkey, wr);
    if (lane < P.C_max)
        *reinterpret_cast<float4 *>(contacts + ((size_t)e * P.C_max + lane) * 4) =
            make_float4(__int_as_float(link), imp[0], imp[1], imp[2]);
    flush_stats(stats, st, 1, e);
}

// The observation of the last step: a workgroup stages the contacts of SIMS
// simulations in LDS, a thread per (simulation, sensor) sums its own in
// contact order.  cost_mode 1 (EQ3): the seven rows of Eq. 3, from the
// contacts' slip records and the step's segments.  PD hand: J rows of joint
// angles from hstate follow the force rows.  Bound by the walk over all
// contact slots; a simulation's records are offset by 16 bytes from the last
// one's, so that the lanes' reads at one slot fall in different banks.
// SIMS: 16 where that still gives every compute unit a workgroup, past
// OBS_FEW simulations, as their rows are written 64 bytes at a time (64 slots,
// 20 sensors; a wavefront per simulation with its lanes over sensors, 4 and 16
// simulations: 8192 of them 7.9, 6.1 and 5.0 us, 16384 12.8 us and, with 16,
// 6.8); up to there 4, whose slots are staged in one go (9 sensors, 256
// simulations: 4.4, 3.4 and 4.9 us).
constexpr int OBS_FEW = 4096;
template <bool EQ3, int SIMS>
__global__ __launch_bounds__(1024) void k_observe(Consts P, const float *__restrict__ contacts,
                                                  const float *__restrict__ cslip, const float *__restrict__ seg,
                                                  const float *__restrict__ hstate, int J, float *__restrict__ obs)
{
    extern __shared__ __align__(16) float4 obs_lds[];
    const int C = P.C_max, fs = C + 1, ss = 2 * C + 1;
    float4 *force = obs_lds, *slip = obs_lds + SIMS * fs;
    const int e0 = xcd_block(blockIdx.x, gridDim.x) * SIMS, n = min(SIMS, P.K - e0);
    const float4 *src = reinterpret_cast<const float4 *>(contacts) + (size_t)e0 * C;
    for (int i = threadIdx.x; i < n * C; i += blockDim.x) force[i + i / C] = src[i];
    if constexpr (EQ3) {
        const float4 *from = reinterpret_cast<const float4 *>(cslip) + (size_t)e0 * C * 2;
        for (int i = threadIdx.x; i < n * C * 2; i += blockDim.x) slip[i + i / (2 * C)] = from[i];
    }
    const size_t K = P.K, LK = P.L * K;
    for (int i = threadIdx.x; i < J * SIMS; i += blockDim.x) {
        const int s = i % SIMS, j = i / SIMS;
        if (s < n) obs[4 * LK + j * K + e0 + s] = hstate[j * K + e0 + s];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < P.L * SIMS; i += blockDim.x) {
        const int s = i % SIMS, l = i / SIMS;
        if (s >= n) continue;
        const float4 *f = force + s * fs, *w = slip + s * ss;
        SensorSums m;
#pragma unroll 8
        for (int c = 0; c < C; ++c) {
            const float4 r = f[c];
            if (__float_as_int(r.x) == l) {
                m.add_force(r);
                if constexpr (EQ3) m.add_slip(w[2 * c], w[2 * c + 1]);
            }
        }
        constexpr int R = EQ3 ? 7 : 4;
        float o[R];
        if constexpr (EQ3) eq3_obs(P, m, seg, l, o);
        else force_obs(P, m.f0, m.f1, m.f2, o);
#pragma unroll
        for (int j = 0; j < R; ++j) obs[j * LK + l * K + e0 + s] = o[j];
    }
}

// The step cost: a thread per (simulation, sensor) makes the terms, COST_ROWS
// sensors of SIMS simulations at a time through LDS, a thread per simulation
// sums them in sensor order (the order of step_cost_wave, so the plain and
// batched paths add the same bits); obs_gt is [R][L][G] (the observed
// batch's own observation layout; R = 4: force rows; R = 7: the rows of
// Eq. 3).  PD hand: J joint rows follow, their w_q (q_j - q_gt_j)^2 in joint
// order.  Latency-bound: a thread per simulation that walks its sensors has
// few wavefronts and a chain of loads (16384 simulations: 9.3 -> 5.0 us; with
// the PD hand's joints 14.3 -> 5.3 us; 256 simulations, with the ranking:
// 7.5 -> 5.6 us).
// SIMS: 256 where the launch also ranks (`best`), so that up to 256
// simulations are one workgroup, which needs no counter (4.8 us of 256; 257
// and its counter 8.6 us), and beyond that few workgroups take part in the
// counting: only the wavefronts that wrote sums flush them first (one group of
// 512: 12.4 us when all 16 did, 9.1 us; a thread per simulation in 256-thread
// workgroups 8.9 us, of 4096 11.3 against 10.0 us).  Otherwise 16, which gives
// 16384 simulations four workgroups a compute unit.
constexpr int COST_ROWS = 32;
template <int R, int SIMS>
__global__ __launch_bounds__(1024) void k_cost(Consts P, const int32_t *__restrict__ group_of,
                                               const int32_t *__restrict__ group_start,
                                               const float *__restrict__ obs, const float *__restrict__ obs_gt,
                                               float w_q, int J, float *cost_sum, int32_t *__restrict__ best,
                                               int32_t *done)
{
    __shared__ float term[COST_ROWS][SIMS];
    __shared__ float csum[SIMS];
    const int e0 = blockIdx.x * SIMS, nt = blockDim.x;
    const size_t LK = (size_t)P.L * P.K, LG = (size_t)P.L * P.G;
    // a thread's simulation is the same in every item: nt is a multiple of SIMS
    const int s = threadIdx.x % SIMS, e = min(e0 + s, P.K - 1), r0 = threadIdx.x / SIMS, dr = nt / SIMS;
    const int g = P.G == 1 ? 0 : group_of[e];
    const bool sums = threadIdx.x < SIMS && e0 + s < P.K;
    const float prev = sums ? cost_sum[e] : 0.f;
    float cs = 0.f;
    for (int l0 = 0; l0 < P.L; l0 += COST_ROWS) {
        const int n = min(COST_ROWS, P.L - l0);
        // CH sensors' loads in flight at a time
        constexpr int CH = SIMS < 256 ? 1 : 4;
        for (int r = r0; r < n; r += CH * dr) {
            float o[CH][R], gt[CH][R];
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const size_t l = l0 + min(r + c * dr, n - 1);
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    o[c][j] = obs[j * LK + l * P.K + e];
                    gt[c][j] = obs_gt[j * LG + l * P.G + g];
                }
            }
#pragma unroll
            for (int c = 0; c < CH; ++c)
                if (r + c * dr < n) {
                    if constexpr (R == 7) term[r + c * dr][s] = sensor_cost_eq3(P, o[c], gt[c]);
                    else term[r + c * dr][s] = sensor_cost(P, o[c], gt[c]);
                }
        }
        __syncthreads();
        if (sums) {
#pragma unroll 8
            for (int r = 0; r < n; ++r) cs += term[r][s];
        }
        __syncthreads();
    }
    for (int j0 = 0; j0 < J; j0 += COST_ROWS) {
        const int n = min(COST_ROWS, J - j0);
        for (int r = r0; r < n; r += dr)
            term[r][s] = obs[R * LK + (size_t)(j0 + r) * P.K + e] - obs_gt[R * LG + (size_t)(j0 + r) * P.G + g];
        __syncthreads();
        if (sums) {
#pragma unroll 8
            for (int r = 0; r < n; ++r) cs = pd_joint_cost(cs, w_q, term[r][s]);
        }
        __syncthreads();
    }
    if (sums) {
        cost_sum[e] = prev + cs;
        csum[s] = prev + cs;
    }
    // with `best`: the workgroup that finishes last ranks every group (Eq. 2);
    // a single workgroup ranks its own sums from LDS, with no counter
    __shared__ float sv[16];
    __shared__ int si[17];
    if (!best) return;
    if (gridDim.x == 1) {
        __syncthreads();
        team_argmin(P.G, group_start, csum, best, sv, si);
    } else if (last_block(done, si + 16, sums)) {
        team_argmin(P.G, group_start, cost_sum, best, sv, si);
        if (threadIdx.x == 0) *done = 0;
    }
}

// one block per group: lowest index of the minimum, NaN ranked as +inf
__global__ void k_argmin(const int32_t *__restrict__ group_start, const float *__restrict__ cost,
                         int32_t *__restrict__ best)
{
    __shared__ float sv[16];
    __shared__ int si[16];
    team_argmin(1, group_start + blockIdx.x, cost, best + blockIdx.x, sv, si);
}

// ---------------------------------------------------------------------
// population-based resampling
// ---------------------------------------------------------------------
// Ranks by counting: a workgroup takes 64 simulations of a group, one per
// lane, and its wavefronts each count the lower entries in their share of
// the group's costs.  n^2 / 64 broadcast reads and n^2 compares a group, but
// over the whole GPU and with one barrier, where a bitonic sort in one
// workgroup per group has log^2 n dependent stages.  Bound by latency: 8 us
// for 16 groups of 1024 (the sort: 22).
__global__ __launch_bounds__(1024) void k_rank(float elite_frac, const int2 *__restrict__ piece,
                                               const int32_t *__restrict__ group_start,
                                               const int32_t *__restrict__ elite_start,
                                               const float *__restrict__ cost_sum, int32_t *__restrict__ rank,
                                               int32_t *__restrict__ order, int32_t *__restrict__ elite0,
                                               int32_t *__restrict__ elite1)
{
    extern __shared__ __align__(16) float cs[];
    __shared__ int part[1024 / WAVE][WAVE];
    const int2 pc = piece[blockIdx.x];
    const int lo = group_start[pc.x], n = group_start[pc.x + 1] - lo, i0 = pc.y;
    stage_costs(cost_sum + lo, n, cs);
    __syncthreads();
    const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), nw = blockDim.x / WAVE;
    const int n4 = (n + 3) & ~3, share = (n4 / 4 + nw - 1) / nw * 4;
    const int i = i0 + lane;
    const float ci = i < n ? cs[i] : 0.f;
    part[w][lane] = rank_count(cs, w * share, min((w + 1) * share, n4), i, i0, min(i0 + RANK_CHUNK, n4), ci);
    __syncthreads();
    if (w > 0 || i >= n) return;
    int r = 0;
    for (int k = 0; k < nw; ++k) r += part[k][lane];
    if (rank) rank[lo + i] = r;
    if (order) order[lo + r] = lo + i;
    if (elite_start && r < elite_count(n, elite_frac)) {
        if (elite0) elite0[elite_start[pc.x] + r] = lo + i;
        if (elite1) elite1[elite_start[pc.x] + r] = lo + i;
    }
}

// Copies and exploration.  ONE: a workgroup takes a whole group of at most
// RESAMPLE_ONE simulations and ranks it first, four threads per simulation;
// otherwise a workgroup takes COPY_CHUNK simulations of a group that k_rank
// has ranked.  The parents are elites, which nothing here writes, so the
// copies need no order among themselves; the running costs (read by the
// ranking alone) are cleared.  Bound by the copies' latency and, for large
// populations, their bytes: 16 groups of 1024 with 64-slot warm caches (13 MB
// copied) take 53 us in one workgroup per group, 8 + 10 us like this; one
// group of 16384 777 and 46; a group of 256 is 1 to 3 us faster in one
// workgroup (one launch) than in two kernels.
// A workgroup per group, sized for the largest, has four threads per
// simulation and four wavefronts at least: a group's latency.  Past
// RESAMPLE_MANY groups these no longer run side by side, so groups of up to 16
// get one wavefront (4096 groups of 4: 15.4 us with four, 12.4 with one; 1024
// groups of 4: 6.8 and 8.6), and where the largest is more than four times the
// mean they are cut into pieces (3000 groups of 4 and one of 256: 32.7 us with
// 1024 threads for each, 19.1 in pieces; 1000 of 4 and one of 100: 11.2, 11.8).
constexpr int RESAMPLE_MANY = 1536;
template <bool ONE>
__global__ __launch_bounds__(1024) void k_resample(Consts P, ResampleArgs R, const int2 *__restrict__ piece,
                                                   const int32_t *__restrict__ group_start, uint32_t window_idx,
                                                   float *__restrict__ cost_sum, const int32_t *__restrict__ rank,
                                                   const int32_t *__restrict__ order, float *__restrict__ state,
                                                   float *__restrict__ params, float *__restrict__ warm,
                                                   int32_t *__restrict__ parent)
{
    constexpr int M = ONE ? RESAMPLE_ONE : COPY_CHUNK;
    __shared__ __align__(16) float cs[ONE ? RESAMPLE_ONE : 4];
    __shared__ int rk[M], ord[ONE ? RESAMPLE_ONE : 1], par[M];
    const int tid = threadIdx.x, nt = blockDim.x;
    const int g = ONE ? blockIdx.x : piece[blockIdx.x].x;
    const int i0 = ONE ? 0 : piece[blockIdx.x].y;
    const int lo = group_start[g], n = group_start[g + 1] - lo;
    const int m = min(n - i0, M);   // simulations of this workgroup
    const int kb = elite_count(n, R.elite_frac);
    const size_t K = P.K;
    if (kb >= n) {   // all elites: nothing is copied
        for (int s = tid; s < m; s += nt) {
            if (parent) parent[lo + i0 + s] = -1;
            cost_sum[lo + i0 + s] = 0.f;
        }
        return;
    }
    if constexpr (ONE) {
        stage_costs(cost_sum + lo, n, cs);
        __syncthreads();
        // four adjacent lanes per simulation, a quarter of the group each
        const int n4 = (n + 3) & ~3, share = (n4 / 4 + 3) / 4 * 4, q = tid & 3;
        for (int i = tid >> 2; i - (tid >> 2) < n; i += nt >> 2) {
            int r = 0;
            if (i < n)
                for (int j = q * share; j < min((q + 1) * share, n); ++j)
                    r += cs[j] < cs[i] || (cs[j] == cs[i] && j < i) ? 1 : 0;
            r += __shfl_xor(r, 1);
            r += __shfl_xor(r, 2);
            if (q == 0 && i < n) {
                rk[i] = r;
                ord[r] = lo + i;
            }
        }
        __syncthreads();
    }
    for (int s = tid; s < m; s += nt) {
        const int j = lo + i0 + s, t = ONE ? rk[s] : rank[j];
        int p = -1;
        if (t >= kb) {
            uint32_t w[4];
            philox4x32_10((uint32_t)j, window_idx, 0u, 0u, (uint32_t)(R.seed & 0xffffffffu), (uint32_t)(R.seed >> 32), w);
            const int prank = (int)(((uint64_t)w[0] * (uint64_t)kb) >> 32);
            p = ONE ? ord[prank] : order[lo + prank];
        }
        par[s] = p;
        if (parent) parent[j] = p;
    }
    __syncthreads();
    // exploration by the block's last wavefronts, copies by the others: the
    // draws are a chain as long as a wavefront's share of the copies
    const int nx = (min(m, nt / 2) + WAVE - 1) / WAVE * WAVE, nc = nt > nx ? nt - nx : nt;
    if (tid >= nt - nx) {
        for (int s = tid - (nt - nx); s < m; s += nx) {
            const int j = lo + i0 + s, p = par[s];
            cost_sum[j] = 0.f;
            if (p < 0) continue;
            float e[5];
            explore(R, (uint32_t)j, window_idx, params[p], params[K + p], e);
            for (int c = 0; c < 5; ++c) params[(size_t)c * K + j] = e[c];
        }
        if (nc < nt) return;
    }
    // warm-cache slots, four of a thread's loaded before any is stored
    float4 *w4 = reinterpret_cast<float4 *>(warm);
    const int C = P.C_max;
    const int items = m * C;
    // x / C and x / m by the reciprocal: x below 2^14 and the divisor at most
    // 256, so (x + 1/2) / d is farther from an integer than its rounding
    const float per_slot = 1.f / (float)C, per_row = 1.f / (float)m;
    auto sim = [&](int x) { return (int)(((float)x + 0.5f) * per_slot); };
    auto source = [&](int x) {
        const int y = min(x, items - 1), s = sim(y), p = par[s];
        return w4[(size_t)(p < 0 ? lo + i0 + s : p) * C + (y - s * C)];
    };
    auto copy = [&](int x, const float4 &v) {
        if (x < items && par[sim(x)] >= 0) w4[(size_t)(lo + i0) * C + x] = v;
    };
    for (int x = tid; x < items; x += 4 * nc) {
        const float4 a = source(x), b = source(x + nc), c = source(x + 2 * nc), d = source(x + 3 * nc);
        copy(x, a);
        copy(x + nc, b);
        copy(x + 2 * nc, c);
        copy(x + 3 * nc, d);
    }
    // state rows, a row's simulations in order
    for (int x = tid; x < 13 * m; x += nc) {
        const int c = (int)(((float)x + 0.5f) * per_row), s = x - c * m, p = par[s];
        if (p >= 0) state[(size_t)c * K + lo + i0 + s] = state[(size_t)c * K + p];
    }
}

// ---------------------------------------------------------------------
// batched path: persistent kernel over a window of T steps
// ---------------------------------------------------------------------
// (the Eq. 3 kernel for large caps, a few registers over what two
// wavefronts per SIMD leave, is held to two with a small spill: ~12% more
// throughput on the 16384-simulation workload)
// SDF: links against the object's distance field (collision_mode 1)
template <typename SR, bool EQ3, bool PT, bool SDF = false>
__global__ __launch_bounds__(StepBounds<SR>::threads) __attribute__((amdgpu_waves_per_eu(!PT ? 2 : 1))) void
k_window(Consts P, Tables tb, const float *__restrict__ seg_win, float *__restrict__ state,
         float *__restrict__ params, float *__restrict__ warm, const float *__restrict__ obs_gt_win,
         float *__restrict__ cost_sum, float *__restrict__ obs_out, const int32_t *__restrict__ env_order,
         int32_t *queue, int64_t *__restrict__ stats, float *__restrict__ ckpt,
         const int32_t *__restrict__ group_start, int32_t *__restrict__ best)
{
    extern __shared__ __align__(16) char smem[];
    const int wib = threadIdx.x / WAVE;
    const int lane = lane_id();
    WaveLds lds = carve_lds(smem, wib, P.max_cand, 0);
    float *stage = contact_stage(lds);
    StepStats st = {0, 0, 0};
    int64_t done = 0;
    const size_t LK = (size_t)P.L * P.K, LG = (size_t)P.L * P.G;
    for (;;) {
        int slot = 0;
        if (lane == 0) slot = atomicAdd(queue, 1);
        slot = __builtin_amdgcn_readfirstlane(slot);
        if (slot >= P.K) break;
        const int e = env_order[slot];
        const int type = tb.env_type[e];
        const int g = tb.group_of[e];
        const int S = tb.n_spheres[type];
        const float *sph = tb.spheres + (size_t)type * P.S_max * 4;
        const float reach = tb.reach[type];
        const float inv[3] = {tb.inv_inertia[3 * type], tb.inv_inertia[3 * type + 1], tb.inv_inertia[3 * type + 2]};
        SdfRef sdf;
        if (SDF) {
            sdf.v = tb.sdf + (size_t)type * P.sdf_n * P.sdf_n * P.sdf_n;
            sdf.box = tb.sdf_box + 4 * type;
            sdf.n = P.sdf_n;
            sdf.M = P.link_samples;
        }
        Body B;
        load_body(state, params, P.K, e, B);
        int wkey;
        float wr[3];
        load_warm(warm, P.C_max, e, wkey, wr);
        // running sum continued step by step, in the order the plain path adds
        float cost = cost_sum[e];
        for (int t = 0; t < P.T; ++t) {
            int link;
            float imp[3];
            // with a checkpoint buffer: the body before the step and the kept
            // contacts' keys and impulses after its solve, per simulation
            const float *seg = seg_win + (size_t)t * P.L * SEG_STRIDE;
            float *ck = ckpt ? ckpt + ((size_t)e * P.T + t) * ckpt_step_floats(P.C_max) : nullptr;
            if (ck) save_body(ck, B);
            StepState<SR> sst;
            step_setup<SR, SDF>(P, seg, sph, S, inv, B, reach, wkey, wr, lds, st, sst, sdf);
            step_solve<SR, PT>(P, sst, B.mu, inv, reinterpret_cast<SR *>(lds.cand));
            if (ck) save_contact<SR>(ck, P.C_max, sst);
            step_finish<SR>(P, sst, inv, B, wkey, wr, link, imp);
            uniform_body(B);
            *reinterpret_cast<float4 *>(stage + 4 * lane) = make_float4(__int_as_float(link), imp[0], imp[1], imp[2]);
            // Eq. 3 (cost_mode 1): the contacts' slip records staged in the
            // candidate list's LDS, free between the solve and the next
            // step's narrow phase
            float *slip = reinterpret_cast<float *>(lds.cand);
            if constexpr (EQ3) {
                float rec[SLIP_STRIDE];
                slip_record<SR>(sst, seg, B.w, rec);
                *reinterpret_cast<float4 *>(slip + SLIP_STRIDE * lane) = make_float4(rec[0], rec[1], rec[2], rec[3]);
                *reinterpret_cast<float4 *>(slip + SLIP_STRIDE * lane + 4) = make_float4(rec[4], rec[5], rec[6], rec[7]);
            }
            wave_sync();
            float cl = 0.f;
            if constexpr (EQ3) {
                float o[7];
                if (sensor_obs_eq3(P, stage, slip, seg, link, o)) {
                    const float *gt = obs_gt_win + (size_t)t * 7 * LG;
                    float gv[7];
#pragma unroll
                    for (int j = 0; j < 7; ++j) gv[j] = gt[j * LG + (size_t)lane * P.G + g];
                    cl = sensor_cost_eq3(P, o, gv);
                    if (obs_out) {
                        float *ob = obs_out + (size_t)t * 7 * LK;
#pragma unroll
                        for (int j = 0; j < 7; ++j) ob[j * LK + (size_t)lane * P.K + e] = o[j];
                    }
                }
            } else {
                float o[4];
                if (sensor_force(P, stage, link, o)) {
                    const float *gt = obs_gt_win + (size_t)t * 4 * LG;
                    float gv[4] = {gt[0 * LG + (size_t)lane * P.G + g], gt[1 * LG + (size_t)lane * P.G + g],
                                   gt[2 * LG + (size_t)lane * P.G + g], gt[3 * LG + (size_t)lane * P.G + g]};
                    cl = sensor_cost(P, o, gv);
                    if (obs_out) {
                        float *ob = obs_out + (size_t)t * 4 * LK;
                        ob[0 * LK + (size_t)lane * P.K + e] = o[0];
                        ob[1 * LK + (size_t)lane * P.K + e] = o[1];
                        ob[2 * LK + (size_t)lane * P.K + e] = o[2];
                        ob[3 * LK + (size_t)lane * P.K + e] = o[3];
                    }
                }
            }
            wave_sync();
            // step cost summed over sensors in sensor order
            cost += step_cost_wave(P, cl);
        }
        store_body(state, params, P.K, e, B);
        store_warm(warm, P.C_max, e, wkey, wr);
        if (lane == 0) cost_sum[e] = cost;
        done += P.T;
    }
    flush_stats(stats, st, done, blockIdx.x * (blockDim.x / WAVE) + wib);
    // the workgroup that finishes last ranks every group (Eq. 2) and puts the
    // work queue back to 0 for the next window
    // (the block's dynamic LDS is free once every wave has left the loop)
    float *sv = reinterpret_cast<float *>(smem);
    int *si = reinterpret_cast<int *>(smem) + 16;
    if (last_block(queue + 1, si + 16)) {
        if (best) block_argmin(P.G, group_start, cost_sum, best, sv, si);
        if (threadIdx.x == 0) { queue[0] = 0; queue[1] = 0; }
    }
}

}  // namespace pt

// ---------------------------------------------------------------------
// launch wrappers (host side)
// ---------------------------------------------------------------------
using namespace pt;

size_t hand_fk_lds_bytes(int L, int D) { return fk_lds_bytes(L, D); }

hipError_t launch_hand_fk(const float *hand, int L, int D, float dt, const float *u_prev, const float *u,
                          int stride, int nsteps, float *seg_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_hand_fk, dim3(nsteps), dim3(128), 0, s, hand, L, D, dt, u_prev, u, stride, seg_out);
    return hipGetLastError();
}

hipError_t launch_step(const Consts &P, const Tables &tb, const float *u_prev, const float *u, float *state,
                       float *params, float *warm, float *contacts, float *cslip, float *seg_out, int64_t *stats,
                       int waves_per_block, bool seg_in, hipStream_t s)
{
    int blocks = (P.K + waves_per_block - 1) / waves_per_block;
    seg_in = seg_in && P.solve_fp64;
    size_t lds = (size_t)waves_per_block * wave_lds_bytes(P.max_cand, seg_in ? 0 : P.L);
    const dim3 grid(blocks), block(WAVE * waves_per_block);
    const bool eq3 = P.cost_mode == 1;
    if (seg_in) {
        if (P.collision_mode == 1)
            hipLaunchKernelGGL((k_step<double, false, true, true>), grid, block, lds, s, P, tb, u_prev, u, state,
                               params, warm, contacts, cslip, seg_out, stats);
        else if (!eq3)
            hipLaunchKernelGGL((k_step<double, false, false, true>), grid, block, lds, s, P, tb, u_prev, u, state,
                               params, warm, contacts, cslip, seg_out, stats);
        else
            hipLaunchKernelGGL((k_step<double, true, false, true>), grid, block, lds, s, P, tb, u_prev, u, state,
                               params, warm, contacts, cslip, seg_out, stats);
    } else if (P.collision_mode == 1)   // float64 solve and force terms only (checked at batch creation)
        hipLaunchKernelGGL((k_step<double, false, true>), grid, block, lds, s, P, tb, u_prev, u, state, params,
                           warm, contacts, cslip, seg_out, stats);
    else if (P.solve_fp64 && !eq3)
        hipLaunchKernelGGL((k_step<double, false>), grid, block, lds, s, P, tb, u_prev, u, state, params, warm,
                           contacts, cslip, seg_out, stats);
    else if (P.solve_fp64)
        hipLaunchKernelGGL((k_step<double, true>), grid, block, lds, s, P, tb, u_prev, u, state, params, warm,
                           contacts, cslip, seg_out, stats);
    else if (!eq3)
        hipLaunchKernelGGL((k_step<float, false>), grid, block, lds, s, P, tb, u_prev, u, state, params, warm,
                           contacts, cslip, seg_out, stats);
    else
        hipLaunchKernelGGL((k_step<float, true>), grid, block, lds, s, P, tb, u_prev, u, state, params, warm,
                           contacts, cslip, seg_out, stats);
    return hipGetLastError();
}

hipError_t launch_observe(const Consts &P, const float *contacts, const float *cslip, const float *seg,
                          const float *hstate, int n_joint, float *obs, hipStream_t s)
{
    auto go = [&](auto kernel, int sims) {
        const int threads = std::max(256, std::min(1024, (P.L * sims + WAVE - 1) / WAVE * WAVE));
        const size_t lds = sizeof(float4) * sims * (P.C_max + 1 + (P.cost_mode == 1 ? 2 * P.C_max + 1 : 0));
        hipLaunchKernelGGL(kernel, dim3((P.K + sims - 1) / sims), dim3(threads), lds, s, P, contacts, cslip, seg, hstate,
                           n_joint, obs);
    };
    const bool few = P.K <= OBS_FEW;
    if (P.cost_mode == 1)
        few ? go(k_observe<true, 4>, 4) : go(k_observe<true, 16>, 16);
    else
        few ? go(k_observe<false, 4>, 4) : go(k_observe<false, 16>, 16);
    return hipGetLastError();
}

hipError_t launch_cost(const Consts &P, const int32_t *group_of, const int32_t *group_start, const float *obs,
                       const float *obs_gt, float w_q, int n_joint, float *cost_sum, int32_t *best, int32_t *done,
                       hipStream_t s)
{
    // threads: a multiple of the simulations of a workgroup, a row of sensors
    // or joints for each
    auto go = [&](auto kernel, int sims) {
        const int rows = std::max(1, std::min(COST_ROWS, std::max(P.L, n_joint)));
        const int threads = std::min(1024, (rows * sims + WAVE - 1) / WAVE * WAVE);
        hipLaunchKernelGGL(kernel, dim3((P.K + sims - 1) / sims), dim3(threads), 0, s, P, group_of, group_start, obs,
                           obs_gt, w_q, n_joint, cost_sum, best, done);
    };
    if (P.cost_mode == 1)
        best ? go(k_cost<7, 256>, 256) : go(k_cost<7, 16>, 16);
    else
        best ? go(k_cost<4, 256>, 256) : go(k_cost<4, 16>, 16);
    return hipGetLastError();
}

hipError_t launch_argmin(int G, const int32_t *group_start, const float *cost, int32_t *best, hipStream_t s)
{
    hipLaunchKernelGGL(k_argmin, dim3(G), dim3(1024), 0, s, group_start, cost, best);
    return hipGetLastError();
}

hipError_t launch_rank(const Pieces &rank_pieces, int max_group, float elite_frac, const int32_t *group_start,
                       const int32_t *elite_start, const float *cost_sum, int32_t *rank, int32_t *order,
                       int32_t *elite0, int32_t *elite1, hipStream_t s)
{
    const int waves = std::min(16, (max_group + WAVE - 1) / WAVE);
    hipLaunchKernelGGL(k_rank, dim3(rank_pieces.count), dim3(WAVE * waves), sizeof(float) * ((max_group + 3) & ~3), s,
                       elite_frac, rank_pieces.piece, group_start, elite_start, cost_sum, rank, order, elite0, elite1);
    return hipGetLastError();
}

hipError_t launch_resample(const Consts &P, const ResampleArgs &R, const int32_t *group_start, int max_group,
                           const Pieces &rank_pieces, const Pieces &copy_pieces, uint32_t window_idx, float *cost_sum,
                           int32_t *rank, int32_t *order, float *state, float *params, float *warm, int32_t *parent,
                           hipStream_t s)
{
    const bool many = P.G > RESAMPLE_MANY, mixed = max_group > 64 && (size_t)max_group * P.G > 4 * (size_t)P.K;
    if (max_group <= RESAMPLE_ONE && !(many && mixed)) {
        const int per = many && max_group <= 16 ? 1 : 4;
        const int threads = std::max(WAVE * per, std::min(1024, (per * max_group + WAVE - 1) / WAVE * WAVE));
        hipLaunchKernelGGL(k_resample<true>, dim3(P.G), dim3(threads), 0, s, P, R, nullptr, group_start, window_idx,
                           cost_sum, nullptr, nullptr, state, params, warm, parent);
        return hipGetLastError();
    }
    hipError_t e = launch_rank(rank_pieces, max_group, R.elite_frac, group_start, nullptr, cost_sum, rank, order,
                               nullptr, nullptr, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_resample<false>, dim3(copy_pieces.count), dim3(256), 0, s, P, R, copy_pieces.piece, group_start,
                       window_idx, cost_sum, rank, order, state, params, warm, parent);
    return hipGetLastError();
}

// the window kernel for a batch: solve precision, cost mode, and the paired
// line-search trials when no step can hold more than 32 contacts (C_max <=
// 32: latency-bound populations, where the extra registers cost nothing);
// the distance-field collision with the float64 solve and the force terms
// only (checked at batch creation)
template <typename F>
static hipError_t with_window_kernel(const Consts &P, F f)
{
    const bool eq3 = P.cost_mode == 1, pt = P.C_max <= 32;
    if (P.collision_mode == 1) return pt ? f(k_window<double, false, true, true>) : f(k_window<double, false, false, true>);
    if (P.solve_fp64) {
        if (eq3) return pt ? f(k_window<double, true, true>) : f(k_window<double, true, false>);
        return pt ? f(k_window<double, false, true>) : f(k_window<double, false, false>);
    }
    if (eq3) return pt ? f(k_window<float, true, true>) : f(k_window<float, true, false>);
    return pt ? f(k_window<float, false, true>) : f(k_window<float, false, false>);
}

hipError_t launch_window(const Consts &P, const Tables &tb, const float *seg_win, float *state, float *params,
                         float *warm, const float *obs_gt_win, float *cost_sum, float *obs_out,
                         const int32_t *env_order, int32_t *queue, int64_t *stats, int waves_per_block, int blocks,
                         float *ckpt, const int32_t *group_start, int32_t *best, hipStream_t s)
{
    size_t lds = (size_t)waves_per_block * wave_lds_bytes(P.max_cand, 0);
    const dim3 grid(blocks), block(WAVE * waves_per_block);
    return with_window_kernel(P, [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, lds, s, P, tb, seg_win, state, params, warm, obs_gt_win, cost_sum,
                           obs_out, env_order, queue, stats, ckpt, group_start, best);
        return hipGetLastError();
    });
}

hipError_t window_occupancy(const Consts &P, int waves_per_block, int *blocks_per_cu)
{
    size_t lds = (size_t)waves_per_block * wave_lds_bytes(P.max_cand, 0);
    return with_window_kernel(P, [&](auto kern) {
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, reinterpret_cast<const void *>(kern),
                                                            WAVE * waves_per_block, lds);
    });
}

hipError_t set_lds_limits(size_t bytes)
{
    const void *fs[] = {reinterpret_cast<const void *>(k_window<float, false, false>),
                        reinterpret_cast<const void *>(k_window<double, false, false>),
                        reinterpret_cast<const void *>(k_window<float, true, false>),
                        reinterpret_cast<const void *>(k_window<double, true, false>),
                        reinterpret_cast<const void *>(k_window<float, false, true>),
                        reinterpret_cast<const void *>(k_window<double, false, true>),
                        reinterpret_cast<const void *>(k_window<float, true, true>),
                        reinterpret_cast<const void *>(k_window<double, true, true>),
                        reinterpret_cast<const void *>(k_window<double, false, false, true>),
                        reinterpret_cast<const void *>(k_window<double, false, true, true>),
                        reinterpret_cast<const void *>(k_step<float, false>),
                        reinterpret_cast<const void *>(k_step<double, false>),
                        reinterpret_cast<const void *>(k_step<float, true>),
                        reinterpret_cast<const void *>(k_step<double, true>),
                        reinterpret_cast<const void *>(k_step<double, false, true>),
                        reinterpret_cast<const void *>(k_rank)};
    for (const void *f : fs) {
        hipError_t e = set_dynamic_lds_limit(f, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
