// gs_deform_lbs kernels: linear blend skinning of canonical avatar Gaussians.
//
// One thread per Gaussian.  The blended 3x4 matrix A = sum_k w_k M_{j_k} is
// formed from four joint matrices read through the cache (all avatars'
// matrices are a few KB; in clip mode eight, two frames per joint); the
// Gaussian streams 60 B in and 36 B out, so the kernel is HBM-bound.
#include "gs_internal.hpp"

namespace gs {



// A += wk * M for one row-major 3x4 matrix M
__device__ __forceinline__ void add_matrix(float *A, float wk, const float *Mp) {
    const float4 *M = reinterpret_cast<const float4 *>(Mp);
    const float4 r0 = M[0], r1 = M[1], r2 = M[2];
    A[0] += wk * r0.x;
    A[1] += wk * r0.y;
    A[2] += wk * r0.z;
    A[3] += wk * r0.w;
    A[4] += wk * r1.x;
    A[5] += wk * r1.y;
    A[6] += wk * r1.z;
    A[7] += wk * r1.w;
    A[8] += wk * r2.x;
    A[9] += wk * r2.y;
    A[10] += wk * r2.z;
    A[11] += wk * r2.w;
}

// The blended matrix A = sum_k w_k M_{j_k}.  In clip mode M_j is avatar a's
// joint matrix at its current time: the linear interpolation
// (1 - s) M_j[f] + s M_j[f + 1] of the two clip frames around the
// fractional frame position p (f = floor(p), s = p - f; p clamped to the
// clip, a clip of one frame holds its pose).  Interpolation and blend are
// both linear, so they are fused: A = sum_k w_k (1 - s) M_{j_k}[f] +
// w_k s M_{j_k}[f + 1], eight matrices read through the cache.
template <bool CLIP>
__device__ __forceinline__ void blend_matrix(const LbsArgs &a, int64_t i, float *A) {
    const uchar4 ji = reinterpret_cast<const uchar4 *>(a.joint_idx)[i];
    const float4 w = reinterpret_cast<const float4 *>(a.weights)[i];
    int av = a.avatar_of[i];
    av = av < 0 ? 0 : (av >= a.n_avatars ? a.n_avatars - 1 : av);
    const int j[4] = {min((int)ji.x, a.n_joints - 1), min((int)ji.y, a.n_joints - 1), min((int)ji.z, a.n_joints - 1),
                      min((int)ji.w, a.n_joints - 1)};
    const float wk[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 12; ++e) A[e] = 0.0f;
    if (!CLIP) {
        const float *base = a.skin + (size_t)av * a.n_joints * 12;
#pragma unroll
        for (int k = 0; k < 4; ++k) add_matrix(A, wk[k], base + (size_t)j[k] * 12);
        return;
    }
    // the avatar's clip, clamped into the clip array
    const int first = min(max(a.clip_first[av], 0), a.clip_total - 1);
    const int frames = min(max(a.clip_frames[av], 1), a.clip_total - first);
    const float p = a.frame_pos[av];
    const float pc = p > 0.0f ? fminf(p, (float)(frames - 1)) : 0.0f;  // NaN -> 0
    const int f0 = frames > 1 ? min((int)floorf(pc), frames - 2) : 0;
    const int f1 = frames > 1 ? f0 + 1 : 0;
    const float s = frames > 1 ? pc - (float)f0 : 0.0f;
    const float *b0 = a.clip + (size_t)(first + f0) * a.n_joints * 12;
    const float *b1 = a.clip + (size_t)(first + f1) * a.n_joints * 12;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        add_matrix(A, wk[k] * (1.0f - s), b0 + (size_t)j[k] * 12);
        add_matrix(A, wk[k] * s, b1 + (size_t)j[k] * 12);
    }
}

template <bool CLIP>
__global__ void __launch_bounds__(256) lbs_kernel(const LbsArgs a) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= a.n) return;
    float A[12];
    blend_matrix<CLIP>(a, i, A);
    const float mx = a.means[3 * i], my = a.means[3 * i + 1], mz = a.means[3 * i + 2];
#pragma unroll
    for (int r = 0; r < 3; ++r) a.means_out[3 * i + r] = A[4 * r] * mx + A[4 * r + 1] * my + A[4 * r + 2] * mz + A[4 * r + 3];
    const float4 q = reinterpret_cast<const float4 *>(a.quats)[i];
    const Rot rot = quat_rot(q.x, q.y, q.z, q.w);
    float s[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) s[k] = expf(a.log_scales[3 * i + k]);
    // A3 M with M = R S; Sigma' = (A3 M)(A3 M)^T
    float N[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            N[3 * r + c] = (A[4 * r] * rot.R[c] + A[4 * r + 1] * rot.R[3 + c] + A[4 * r + 2] * rot.R[6 + c]) * s[c];
    float *o = a.cov6_out + 6 * i;
    o[0] = N[0] * N[0] + N[1] * N[1] + N[2] * N[2];
    o[1] = N[0] * N[3] + N[1] * N[4] + N[2] * N[5];
    o[2] = N[0] * N[6] + N[1] * N[7] + N[2] * N[8];
    o[3] = N[3] * N[3] + N[4] * N[4] + N[5] * N[5];
    o[4] = N[3] * N[6] + N[4] * N[7] + N[5] * N[8];
    o[5] = N[6] * N[6] + N[7] * N[7] + N[8] * N[8];
}

template <bool CLIP>
__global__ void __launch_bounds__(256) lbs_backward_kernel(const LbsArgs a) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= a.n) return;
    float A[12];
    blend_matrix<CLIP>(a, i, A);
    const float gx = a.d_means_out[3 * i], gy = a.d_means_out[3 * i + 1], gz = a.d_means_out[3 * i + 2];
#pragma unroll
    for (int c = 0; c < 3; ++c) a.d_means[3 * i + c] = A[c] * gx + A[4 + c] * gy + A[8 + c] * gz;
    // dSigma = A3^T G A3 with G the full symmetric adjoint of Sigma'
    const float *d = a.d_cov6_out + 6 * i;
    const float G[9] = {d[0], 0.5f * d[1], 0.5f * d[2], 0.5f * d[1], d[3], 0.5f * d[4], 0.5f * d[2], 0.5f * d[4], d[5]};
    float GA[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) GA[3 * r + c] = G[3 * r] * A[c] + G[3 * r + 1] * A[4 + c] + G[3 * r + 2] * A[8 + c];
    float dS[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) dS[3 * r + c] = A[r] * GA[c] + A[4 + r] * GA[3 + c] + A[8 + r] * GA[6 + c];
    const float4 q = reinterpret_cast<const float4 *>(a.quats)[i];
    const Rot rot = quat_rot(q.x, q.y, q.z, q.w);
    float s[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) s[k] = expf(a.log_scales[3 * i + k]);
    float dls[3], dq[4];
    cov_backward(rot, s, dS, dls, dq);
#pragma unroll
    for (int k = 0; k < 3; ++k) a.d_log_scales[3 * i + k] = dls[k];
    reinterpret_cast<float4 *>(a.d_quats)[i] = make_float4(dq[0], dq[1], dq[2], dq[3]);
}

// Adjoint w.r.t. the joint matrices (fixed-matrix mode): with dL/dA_g =
// (g mean^T + 2 G A3 Sigma | g) the 3x4 adjoint of Gaussian g's blended
// matrix, joint j of an avatar gets the sum over its Gaussians of w_gj dL/dA_g.
constexpr int kJointLds = 4096;

__device__ __forceinline__ void gaussian_matrix_adjoint(const LbsArgs &a, int64_t i, const float *A, float *dA) {
    const float gx = a.d_means_out[3 * i], gy = a.d_means_out[3 * i + 1], gz = a.d_means_out[3 * i + 2];
    const float mx = a.means[3 * i], my = a.means[3 * i + 1], mz = a.means[3 * i + 2];
    const float *d = a.d_cov6_out + 6 * i;
    const float G[9] = {d[0], 0.5f * d[1], 0.5f * d[2], 0.5f * d[1], d[3], 0.5f * d[4], 0.5f * d[2], 0.5f * d[4], d[5]};
    // Sigma = (R S)(R S)^T from the canonical scales and rotation
    const float4 q = reinterpret_cast<const float4 *>(a.quats)[i];
    const Rot rot = quat_rot(q.x, q.y, q.z, q.w);
    float M[9];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float sk = expf(a.log_scales[3 * i + k]);
#pragma unroll
        for (int r = 0; r < 3; ++r) M[3 * r + k] = rot.R[3 * r + k] * sk;
    }
    float S[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) S[3 * r + c] = M[3 * r] * M[3 * c] + M[3 * r + 1] * M[3 * c + 1] + M[3 * r + 2] * M[3 * c + 2];
    // GA = G A3, then dA3 = 2 GA Sigma + g mean^T
    float GA[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) GA[3 * r + c] = G[3 * r] * A[c] + G[3 * r + 1] * A[4 + c] + G[3 * r + 2] * A[8 + c];
    const float g[3] = {gx, gy, gz}, m[3] = {mx, my, mz};
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
            dA[4 * r + c] = 2.0f * (GA[3 * r] * S[c] + GA[3 * r + 1] * S[3 + c] + GA[3 * r + 2] * S[6 + c]) + g[r] * m[c];
        dA[4 * r + 3] = g[r];
    }
}

// the four joints, weights and avatar of Gaussian i, clamped as in the blend
struct Blend4 {
    int av, j[4];
    float w[4];
};
__device__ __forceinline__ Blend4 blend_of(const LbsArgs &a, int64_t i) {
    const uchar4 ji = reinterpret_cast<const uchar4 *>(a.joint_idx)[i];
    const float4 w = reinterpret_cast<const float4 *>(a.weights)[i];
    const int av = a.avatar_of[i], jl = a.n_joints - 1;
    return {av < 0 ? 0 : (av >= a.n_avatars ? a.n_avatars - 1 : av),
            {min((int)ji.x, jl), min((int)ji.y, jl), min((int)ji.z, jl), min((int)ji.w, jl)},
            {w.x, w.y, w.z, w.w}};
}

// Up to 16 MB joints: the sum is a matrix product, D[joint][element] =
// sum_g W[joint][g] dA[g][element], and the matrix cores take it.  A wave
// owns a contiguous run of Gaussians, 64 at a time: each lane scatters its
// four weights into its column of W (zero elsewhere) and its twelve elements
// into dA, both in LDS with the Gaussian fastest, and MB x 16
// v_mfma_f32_16x16x4_f32 add them to the wave's sums.  The sums stay in
// registers until the avatar changes, then go to the workgroup's copy of the
// output in LDS (where it fits, kJointLds floats), whose nonzero entries end
// in float atomics.  A group that spans avatars takes one product per avatar,
// up to four; the Gaussians of further ones add their 48 terms themselves
// (avatars mixed at random would take a product per Gaussian), and in small
// calls, where the products' chain is the time, all of a group of more than
// sixteen avatars (1000 Gaussians of 64 avatars of 55 joints mixed 36 us with
// them, 32 without).  So does a Gaussian whose dA is not finite, which would
// reach every joint of the product through the zero weights.  Bound by its 140
// B of reads per Gaussian and their latency; adding every element to LDS with
// atomics (48 per Gaussian, a few lanes of a wave on the same joint each time)
// took 114 us for 400k Gaussians of 8 avatars with 24 joints, this takes 25 us.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kFewGroups = 64;  // groups of a small call
constexpr int kJgStride = 68;  // floats per row of 64 Gaussians: rows on different banks
template <int MB, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) lbs_joint_mfma_kernel(const LbsArgs a, float *d_skin) {
    __shared__ __attribute__((aligned(16))) float s_w[WAVES][16 * MB][kJgStride];
    __shared__ __attribute__((aligned(16))) float s_da[WAVES][12][kJgStride];
    __shared__ float s_acc[kJointLds];
    const int64_t n_mats = (int64_t)a.n_avatars * a.n_joints * 12;
    const bool lds = n_mats <= kJointLds;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int mi = lane & 15, mk = lane >> 4;  // operand row / column, k block
    float(*W)[kJgStride] = s_w[wave];
    float(*dAs)[kJgStride] = s_da[wave];
    for (int k = lane; k < 16 * MB * kJgStride; k += 64) (&W[0][0])[k] = 0.0f;
    if (lds)
        for (int k = threadIdx.x; k < n_mats; k += 64 * WAVES) s_acc[k] = 0.0f;
    __syncthreads();
    f32x4 acc[MB];
    int acc_av = -1;  // avatar of the sums held in acc (uniform)
    auto add = [&](int64_t at, float v) {
        if (lds) atomicAdd(&s_acc[at], v);
        else atomicAdd(&d_skin[at], v);
    };
    auto flush = [&](int next) {  // D row 4 mk + r, column mi
        if (acc_av >= 0 && mi < 12) {
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int j = 16 * b + 4 * mk + r;
                    if (j < a.n_joints && acc[b][r] != 0.0f)
                        add(((int64_t)acc_av * a.n_joints + j) * 12 + mi, acc[b][r]);
                }
        }
#pragma unroll
        for (int b = 0; b < MB; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        acc_av = next;
    };
    flush(-1);
    const int64_t groups = (a.n + 63) / 64, w0 = (int64_t)blockIdx.x * WAVES + wave, nw = (int64_t)gridDim.x * WAVES;
    for (int64_t gr = groups * w0 / nw; gr < groups * (w0 + 1) / nw; ++gr) {
        const int64_t i = gr * 64 + lane;
        const bool valid = i < a.n;
        float A[12], dA[12];
#pragma unroll
        for (int e = 0; e < 12; ++e) dA[e] = 0.0f;
        Blend4 bl = {-1, {0, 0, 0, 0}, {0.0f, 0.0f, 0.0f, 0.0f}};
        if (valid) {
            bl = blend_of(a, i);
            blend_matrix<false>(a, i, A);
            gaussian_matrix_adjoint(a, i, A, dA);
        }
        bool finite = true;
#pragma unroll
        for (int e = 0; e < 12; ++e) finite = finite && isfinite(dA[e]);
        lds_wave_sync();
#pragma unroll
        for (int e = 0; e < 12; ++e) dAs[e][lane] = finite ? dA[e] : 0.0f;
        uint64_t left = __ballot(valid && finite);
        int turns = 4;
        if (groups <= kFewGroups) {  // uniform
            uint64_t m = left;
            for (int k = 0; m && k < 16; ++k)
                m &= ~__ballot(bl.av == __builtin_amdgcn_readlane(bl.av, __ffsll((unsigned long long)m) - 1));
            if (m) turns = 0;
        }
        for (int turn = 0; left && turn < turns; ++turn) {  // one avatar at a time
            const int av = __builtin_amdgcn_readlane(bl.av, __ffsll((unsigned long long)left) - 1);
            const bool mine = valid && finite && bl.av == av;
            left &= ~__ballot(mine);
            if (av != acc_av) flush(av);
            if (mine)
#pragma unroll
                for (int k = 0; k < 4; ++k) atomicAdd(&W[bl.j[k]][lane], bl.w[k]);  // a joint may come twice
            lds_wave_sync();
            f32x4 bv[4];
#pragma unroll
            for (int m = 0; m < 4; ++m)
                bv[m] = mi < 12 ? *reinterpret_cast<const f32x4 *>(&dAs[mi][16 * mk + 4 * m])
                                : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                const f32x4 *row = reinterpret_cast<const f32x4 *>(&W[16 * b + mi][16 * mk]);
                const f32x4 wv[4] = {row[0], row[1], row[2], row[3]};
#pragma unroll
                for (int st = 0; st < 16; ++st)
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[st >> 2][st & 3], bv[st >> 2][st & 3], acc[b], 0,
                                                                  0, 0);
            }
            lds_wave_sync();
            if (mine)
#pragma unroll
                for (int k = 0; k < 4; ++k) W[bl.j[k]][lane] = 0.0f;
            lds_wave_sync();
        }
        if (valid && (!finite || ((left >> lane) & 1ull)))
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 12; ++e)
                    add(((int64_t)bl.av * a.n_joints + bl.j[k]) * 12 + e, bl.w[k] * dA[e]);
    }
    flush(-1);
    if (lds) {
        __syncthreads();
        for (int k = threadIdx.x; k < n_mats; k += 64 * WAVES)
            if (s_acc[k] != 0.0f) atomicAdd(&d_skin[k], s_acc[k]);
    }
}

// More joints than that: a persistent grid walks the Gaussians, each thread
// adding w_k dA to the four joints it blends, first in the workgroup's LDS
// copy of the output (when it fits), whose nonzero entries end in float
// atomics.
__global__ void __launch_bounds__(256) lbs_joint_grad_kernel(const LbsArgs a, float *d_skin) {
    __shared__ float s_acc[kJointLds];
    const int64_t n_mats = (int64_t)a.n_avatars * a.n_joints * 12;
    const bool lds = n_mats <= kJointLds;
    if (lds) {
        for (int k = threadIdx.x; k < n_mats; k += 256) s_acc[k] = 0.0f;
        __syncthreads();
    }
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < a.n; i += stride) {
        float A[12], dA[12];
        blend_matrix<false>(a, i, A);
        gaussian_matrix_adjoint(a, i, A, dA);
        const Blend4 bl = blend_of(a, i);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t base = ((int64_t)bl.av * a.n_joints + bl.j[k]) * 12;
#pragma unroll
            for (int e = 0; e < 12; ++e) {
                if (lds) atomicAdd(&s_acc[base + e], bl.w[k] * dA[e]);
                else atomicAdd(&d_skin[base + e], bl.w[k] * dA[e]);
            }
        }
    }
    if (lds) {
        __syncthreads();
        for (int k = threadIdx.x; k < n_mats; k += 256)
            if (s_acc[k] != 0.0f) atomicAdd(&d_skin[k], s_acc[k]);
    }
}

hipError_t launch_lbs_joint_grad(const LbsArgs &a, float *d_skin, int n_cu, hipStream_t s) {
    const int64_t n_mats = (int64_t)a.n_avatars * a.n_joints * 12;
    hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t *>(d_skin), 0u, n_mats, s);
    if (e != hipSuccess || a.n == 0) return e;
    // one workgroup per CU: few flushes to HBM.  The joint count decides how
    // many 16-row blocks of W a wave keeps in LDS; 64 joints are what four
    // waves of a CU have room for.
    auto grid = [&](int waves) {
        const int64_t g = ((a.n + 63) / 64 + waves - 1) / waves;
        return dim3((unsigned)(g < n_cu ? g : n_cu));
    };
    // Half as many while that leaves a wave for every group on as many CUs: eight
    // contend for a CU's LDS while others are idle (24 joints, 8 avatars, 20 k
    // Gaussians 19.0 / 15.8 us, mixed at random 40.4 / 27.4; 60 k 18.5 / 15.8).
    const bool few = (a.n + 63) / 64 <= 4 * (int64_t)n_cu;
    if (a.n_joints <= 16 && !few) return launch_kernel(lbs_joint_mfma_kernel<1, 8>, grid(8), dim3(512), s, a, d_skin);
    if (a.n_joints <= 32 && !few) return launch_kernel(lbs_joint_mfma_kernel<2, 8>, grid(8), dim3(512), s, a, d_skin);
    if (a.n_joints <= 16) return launch_kernel(lbs_joint_mfma_kernel<1, 4>, grid(4), dim3(256), s, a, d_skin);
    if (a.n_joints <= 32) return launch_kernel(lbs_joint_mfma_kernel<2, 4>, grid(4), dim3(256), s, a, d_skin);
    if (a.n_joints <= 64) return launch_kernel(lbs_joint_mfma_kernel<4, 4>, grid(4), dim3(256), s, a, d_skin);
    return launch_kernel(lbs_joint_grad_kernel, grid(4), dim3(256), s, a, d_skin);
}

// Forward kinematics: one thread per avatar walks its joints parent first.
// Joint k's world transform G_k = G_parent [R(w_k) | rest_k - rest_parent]
// (the root transform in place of G_parent for a root) is written to the
// output and read back by its children; a second walk turns every G_k into
// the skinning matrix G_k [I | -rest_k].  R(w) = I + a [w]x + b [w]x^2 with
// a = sin t / t and b = (1 - cos t) / t^2 = (sin(t/2) / (t/2))^2 / 2.
__global__ void __launch_bounds__(64) fk_kernel(const FkArgs f) {
    const int a = blockIdx.x * 64 + threadIdx.x;
    if (a >= f.n_avatars) return;
    float *out = f.out + (size_t)a * f.n_joints * 12;
    const float *root = f.root + (size_t)a * 12;
    for (int k = 0; k < f.n_joints; ++k) {
        const float *w = f.pose + ((size_t)a * f.n_joints + k) * 3;
        const float wx = w[0], wy = w[1], wz = w[2];
        const float t = sqrtf(wx * wx + wy * wy + wz * wz);
        float sa = 1.0f, sb = 0.5f;
        if (t > 0.0f) {
            sa = sinf(t) / t;
            const float h = sinf(0.5f * t) / (0.5f * t);
            sb = 0.5f * h * h;
        }
        // [w]x^2 = w w^T - |w|^2 I
        const float R[9] = {1.0f + sb * (wx * wx - t * t), sb * wx * wy - sa * wz, sb * wx * wz + sa * wy,
                            sb * wx * wy + sa * wz, 1.0f + sb * (wy * wy - t * t), sb * wy * wz - sa * wx,
                            sb * wx * wz - sa * wy, sb * wy * wz + sa * wx, 1.0f + sb * (wz * wz - t * t)};
        const int p = f.parents[k];
        float lt[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) lt[c] = f.rest[3 * k + c] - (p >= 0 ? f.rest[3 * p + c] : 0.0f);
        const float *P = p >= 0 ? out + (size_t)p * 12 : root;
        float G[12];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const float p0 = P[4 * r], p1 = P[4 * r + 1], p2 = P[4 * r + 2];
#pragma unroll
            for (int c = 0; c < 3; ++c) G[4 * r + c] = p0 * R[c] + p1 * R[3 + c] + p2 * R[6 + c];
            G[4 * r + 3] = p0 * lt[0] + p1 * lt[1] + p2 * lt[2] + P[4 * r + 3];
        }
#pragma unroll
        for (int e = 0; e < 12; ++e) out[(size_t)k * 12 + e] = G[e];
    }
    for (int k = 0; k < f.n_joints; ++k) {
        float *G = out + (size_t)k * 12;
        const float rx = f.rest[3 * k], ry = f.rest[3 * k + 1], rz = f.rest[3 * k + 2];
#pragma unroll
        for (int r = 0; r < 3; ++r) G[4 * r + 3] -= G[4 * r] * rx + G[4 * r + 1] * ry + G[4 * r + 2] * rz;
    }
}

hipError_t launch_fk(const FkArgs &f, hipStream_t s) {
    if (f.n_avatars <= 0) return hipSuccess;
    return launch_kernel(fk_kernel, dim3((unsigned)((f.n_avatars + 63) / 64)), dim3(64), s, f);
}

hipError_t launch_lbs(const LbsArgs &a, bool backward, hipStream_t s) {
    if (a.n == 0) return hipSuccess;
    const unsigned grid = (unsigned)((a.n + 255) / 256);
    if (a.clip) {
        if (backward) return launch_kernel(lbs_backward_kernel<true>, dim3(grid), dim3(256), s, a);
        return launch_kernel(lbs_kernel<true>, dim3(grid), dim3(256), s, a);
    }
    if (backward) return launch_kernel(lbs_backward_kernel<false>, dim3(grid), dim3(256), s, a);
    return launch_kernel(lbs_kernel<false>, dim3(grid), dim3(256), s, a);
}

}  // namespace gs
