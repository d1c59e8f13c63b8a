// gs_project kernel: per (view, Gaussian) EWA projection, SH colour and tile
// rect, scene-major: the cameras of the launch sit in LDS and a scene drawn by
// many views is read from HBM once.
//
// Most (view, Gaussian) pairs are culled -- behind the camera or outside its
// frustum: 85 % of a room for one camera inside it -- and they are spread over
// the lanes at random, so a kernel of one Gaussian per lane spends nearly the
// whole cost of the visible ones (covariance, projection, spherical harmonics:
// about 330 VALU instructions) on every wave and view, and its lanes read the
// SH rows of scattered Gaussians 16 B at a time, again for every view.  In large
// launches of many views of degree 3 each wave therefore works in two steps.
// Step 1, one Gaussian per lane, 64 at a time: a bound from the position and the largest scale alone (cannot_draw) rejects the
// pairs that surely touch no tile.  The SH rows of the Gaussians that keep a
// view are copied to LDS once, whole rows at a time (consecutive lanes on
// consecutive 16 B), and the kept pairs are listed there.  Step 2, one pair per
// lane, whenever 64 are listed or the rows in LDS are to be replaced: the exact
// projection decides, and the records leave through LDS too, 48 contiguous
// bytes by three neighbouring lanes.  A rejected Gaussian's rotation and SH
// rows are never fetched.  PLANES: the same reads from a segment stored
// component-major (plane k of an attribute at k n); its SH is read from HBM by
// each pair, there are no rows to copy.
// Waves are independent: no barrier after the cameras are staged.  Bound by
// HBM traffic (64 views of 8 scenes: 2.2 GB, 3.0 TB/s).
#include <algorithm>

#include "gs_ewa.hpp"

namespace gs {

constexpr int kRowsLds = 32;   // SH rows a wave holds in LDS

// What step 1 needs of a camera beside its matrix: the norms of the rows of R,
// the tangent limits, and a bound m1 * ka + kb of the rounding of a
// camera-space coordinate for a mean of 1-norm m1.
struct CamBound {
    float r0, r1, r2, limx, limy, ka, kb, pad;
};

__device__ __forceinline__ CamBound cam_bound(const float *c, const ProjectArgs &a) {
    CamBound b;
    b.r0 = sqrtf(c[0] * c[0] + c[1] * c[1] + c[2] * c[2]);
    b.r1 = sqrtf(c[3] * c[3] + c[4] * c[4] + c[5] * c[5]);
    b.r2 = sqrtf(c[6] * c[6] + c[7] * c[7] + c[8] * c[8]);
    b.limx = a.fov_clamp * (0.5f * (float)a.W / c[12]);
    b.limy = a.fov_clamp * (0.5f * (float)a.H / c[13]);
    // |R| <= its row norms; 16 roundings of 2^-24.  A mirrored or degenerate
    // camera is left to the exact projection.
    b.ka = c[12] > 0.0f && c[13] > 0.0f ? 1e-6f * (b.r0 + b.r1 + b.r2) : INFINITY;
    b.kb = 1e-6f * (fabsf(c[9]) + fabsf(c[10]) + fabsf(c[11]));
    b.pad = 0.0f;
    return b;
}

// True only if the pair surely draws nothing: behind the near plane, or the
// tile rect of the largest radius it can have outside the image.  lam bounds
// the covariance's largest eigenvalue, so the 2D covariance has a + c <=
// (|T0|^2 + |T1|^2) lam + 2 lowpass with |T0| <= fx/z (|R0| + |xr| |R2|), and
// the radius is at most ceil(cut sqrt(a + c + sqrt(0.1))).  Every term is
// widened far beyond the rounding of the exact projection, and a comparison
// with a not-a-number keeps the pair.
__device__ __forceinline__ bool cannot_draw(const ProjectArgs &a, const float *cam, const CamBound &b, float mx,
                                            float my, float mz, float m1, float lam) {
    const float tx = cam[0] * mx + cam[1] * my + cam[2] * mz + cam[9];
    const float ty = cam[3] * mx + cam[4] * my + cam[5] * mz + cam[10];
    const float tz = cam[6] * mx + cam[7] * my + cam[8] * mz + cam[11];
    const float err = fmaf(m1, b.ka, b.kb);
    if (tz <= a.near_plane - err) return true;
    const float fx = cam[12], fy = cam[13];
    const float iz = __builtin_amdgcn_rcpf(tz);
    const float xz = tx * iz, yz = ty * iz;
    const float u = fmaf(fx, xz, cam[14]), v = fmaf(fy, yz, cam[15]);
    const float n0 = fx * iz * fmaf(fminf(fabsf(xz), b.limx), b.r2, b.r0);
    const float n1 = fy * iz * fmaf(fminf(fabsf(yz), b.limy), b.r2, b.r1);
    const float ac = fmaf(fmaf(n0, n0, n1 * n1), lam, 2.0f * a.lowpass + 0.32f);
    const float r = 1.002f * a.sigma_cut * __builtin_amdgcn_sqrtf(ac) + 2.0f +
                    2e-3f * (fmaxf(fx, fy) + fabsf(u) + fabsf(v));
    const float uc = fminf(fmaxf(u, -kCoordClamp), kCoordClamp), vc = fminf(fmaxf(v, -kCoordClamp), kCoordClamp);
    const bool outside = uc + r < 0.0f || uc - r > (float)(kTile * a.TX) || vc + r < 0.0f ||
                         vc - r > (float)(kTile * a.TY);
    // near the plane the coordinates' rounding could move u by more than the
    // margin: the exact projection decides there
    return outside && tz > a.near_plane + 1000.0f * err;
}

// a wave's part of the LDS
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kShVecs = 3 * 16 / 4;         // 16-byte pieces of an SH row of degree 3
constexpr int kShStride = kShVecs | 1;      // odd: rows start on different banks
struct ProjectLds {
    f32x4 rec[32 * 3];                      // records on their way out, half a wave at a time
    f32x4 sh[kRowsLds * kShStride];
    uint2 list[128];     // kept pairs: Gaussian, view of the launch | row << 8
    uint32_t gid[kRowsLds];
    uint32_t inst[32];   // instance of a record, ~0: none
};
// of the workgroup: cameras, their bounds and first instances
struct ProjectCams {
    float cam[kCamStride];
    CamBound bound;
    int64_t base;
};

// The segment of this workgroup and its cameras, staged in LDS (ends with a
// barrier).  ONE: the launch has one segment, at fixed places in the arguments
// (a lookup would head the chain of loads); BOUND: with the cameras' bounds.
struct ProjectBlock {
    int k, nv;       // segment of the launch, its views
    uint32_t block;  // workgroup within the segment
    ProjectCams *cams;
};
template <bool ONE, bool BOUND>
__device__ __forceinline__ ProjectBlock project_block(const ProjectArgs &a, char *dyn) {
    ProjectBlock B;
    B.k = 0;
    if (!ONE)
        while (B.k + 1 < a.n_segs && blockIdx.x >= a.first_block[B.k + 1]) ++B.k;
    B.block = ONE ? blockIdx.x : blockIdx.x - a.first_block[B.k];
    const int p0 = ONE ? 0 : a.first_pair[B.k];
    B.nv = a.first_pair[B.k + 1] - p0;
    B.cams = reinterpret_cast<ProjectCams *>(dyn);
    for (int k = threadIdx.x; k < B.nv * 16; k += 256)
        B.cams[k >> 4].cam[k & 15] = reinterpret_cast<const float *>(a.cams + a.view[p0 + (k >> 4)])[k & 15];
    __syncthreads();
    for (int vi = threadIdx.x; vi < B.nv; vi += 256) {
        float *c = B.cams[vi].cam;
        // camera centre -R^T t
#pragma unroll
        for (int j = 0; j < 3; ++j) c[16 + j] = -(c[j] * c[9] + c[3 + j] * c[10] + c[6 + j] * c[11]);
        c[19] = __int_as_float(a.view[p0 + vi]);
        if (BOUND) B.cams[vi].bound = cam_bound(c, a);
        B.cams[vi].base = a.base[p0 + vi];
    }
    __syncthreads();
    return B;
}

// Unit direction in world space from the camera centre to the mean, and the
// SH basis there.
template <int D>
__device__ __forceinline__ void view_basis(const float *cam, float mx, float my, float mz, float *Y) {
    float dx = mx - cam[16], dy = my - cam[17], dz = mz - cam[18];
    const float inv = 1.0f / sqrtf(dx * dx + dy * dy + dz * dz);
    dx *= inv;
    dy *= inv;
    dz *= inv;
    sh_basis<D>(dx, dy, dz, Y);
}

template <bool PLANES>
__global__ void __launch_bounds__(256) project_kernel(const ProjectArgs a) {
    constexpr int D = 3, K = 16;
    extern __shared__ __attribute__((aligned(16))) char s_dyn[];  // ProjectCams[nv]
    __shared__ __attribute__((aligned(16))) ProjectLds s_wave[4];
    const ProjectBlock B = project_block<false, true>(a, s_dyn);
    const gs_gaussians &seg = a.seg[B.k];
    const ProjectCams *s_cams = B.cams;
    const int nv = B.nv;

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    const int64_t n = seg.n;
    ProjectLds &W = s_wave[wave];
    int listed = 0, rows = 0, copied = 0;  // pairs; rows taken, rows copied
    // component k of Gaussian i in an attribute of w components
    auto at = [&](const float *p, int64_t i, int w, int k) { return PLANES ? p[(int64_t)k * n + i] : p[w * i + k]; };

    // step 2: lanes [0, m) take the last m listed pairs
    auto project = [&](int m) {
        lds_wave_sync();
        listed -= m;
        const uint2 pair = W.list[listed + min(lane, m - 1)];
        const int64_t i = (int64_t)pair.x;
        const int vi = (int)(pair.y & 255u);
        // the rows not copied yet: every load in flight before the first is stored
        constexpr int IT = (kRowsLds * kShVecs + 63) / 64;
        const int todo = PLANES ? 0 : (rows - copied) * kShVecs;
        f32x4 t[IT];
        if (todo > 0) {
#pragma unroll
            for (int k = 0; k < IT; ++k) {
                const int f = min(k * 64 + lane, todo - 1);
                t[k] = reinterpret_cast<const f32x4 *>(seg.sh + (size_t)(3 * K) * W.gid[copied + f / kShVecs])[f % kShVecs];
            }
        }
        const uint32_t inst = (uint32_t)(s_cams[vi].base + i);
        const float *cam = s_cams[vi].cam;
        const float mx = at(seg.means, i, 3, 0), my = at(seg.means, i, 3, 1), mz = at(seg.means, i, 3, 2);
        const float opac = seg.opacity[i];
        float S[6];
        if (seg.cov6) {
#pragma unroll
            for (int k = 0; k < 6; ++k) S[k] = at(seg.cov6, i, 6, k);
        } else {
            float4 q4;
            if (PLANES)
                q4 = make_float4(at(seg.quats, i, 4, 0), at(seg.quats, i, 4, 1), at(seg.quats, i, 4, 2),
                                 at(seg.quats, i, 4, 3));
            else
                q4 = reinterpret_cast<const float4 *>(seg.quats)[i];
            const Rot rot = quat_rot(q4.x, q4.y, q4.z, q4.w);
            float s[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) s[k] = expf(at(seg.log_scales, i, 3, k));
            cov_from_rot_scale(rot.R, s, S);
        }
        if (todo > 0) {
#pragma unroll
            for (int k = 0; k < IT; ++k) {
                const int f = k * 64 + lane;
                if (f < todo) W.sh[(copied + f / kShVecs) * kShStride + f % kShVecs] = t[k];
            }
            copied = rows;
            lds_wave_sync();
        }
        ViewProj p;
        const bool draws = ewa_project(cam, mx, my, mz, S, a.W, a.H, a.TX, a.TY, a.near_plane, a.lowpass, a.sigma_cut,
                                       a.fov_clamp, p);
        uint32_t count = 0u;
        f32x4 r0 = {0.0f, 0.0f, 0.0f, 0.0f}, r1 = r0, r2 = r0;
        if (draws) {
            float Y[K];
            view_basis<D>(cam, mx, my, mz, Y);
            // colour, accumulated per channel in basis order
            float col[3] = {0.0f, 0.0f, 0.0f};
            if (PLANES) {
                const float *shp = seg.sh + i;
#pragma unroll
                for (int f = 0; f < 3 * K; ++f) col[f % 3] += Y[f / 3] * shp[(int64_t)f * n];
            } else {
                const f32x4 *shp = W.sh + (pair.y >> 8) * kShStride;
#pragma unroll
                for (int v = 0; v < kShVecs; ++v) {
                    const f32x4 t4 = shp[v];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int f = 4 * v + e;  // coefficient f = 3 k + ch
                        col[f % 3] += Y[f / 3] * t4[e];
                    }
                }
            }
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) col[ch] = fmaxf(col[ch] + 0.5f, 0.0f);
            r0 = f32x4{p.u, p.v, p.tz, __int_as_float(p.radius)};
            r1 = f32x4{p.A, p.B, p.C, opac};
            r2 = f32x4{col[0], col[1], col[2], cam[19]};
            count = (uint32_t)((p.rect.x1 - p.rect.x0) * (p.rect.y1 - p.rect.y0));
        }
        if (lane < m) a.tiles_touched[inst] = count;
        // three neighbouring lanes write a record's 48 bytes, half the wave's
        // records at a time
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (32 * h >= m) break;  // uniform
            if ((lane >> 5) == h) {
                W.rec[3 * (lane & 31)] = r0;
                W.rec[3 * (lane & 31) + 1] = r1;
                W.rec[3 * (lane & 31) + 2] = r2;
                W.inst[lane & 31] = lane < m && draws ? inst : ~0u;
            }
            lds_wave_sync();
            for (int q = lane; q < 96; q += 64) {
                const uint32_t to = W.inst[q / 3];
                if (to != ~0u) reinterpret_cast<f32x4 *>(a.rec)[3 * (size_t)to + q % 3] = W.rec[q];
            }
            lds_wave_sync();
        }
    };

    // step 1
    const int64_t c = (int64_t)B.block * 4 + wave;  // this wave's 64 Gaussians
    if (c * 64 >= n) return;                        // uniform per wave, no barrier follows
    const bool valid = c * 64 + lane < n;
    const int64_t i = valid ? c * 64 + lane : n - 1;
    const float mx = at(seg.means, i, 3, 0), my = at(seg.means, i, 3, 1), mz = at(seg.means, i, 3, 2);
    const bool drawable = valid && isfinite(seg.opacity[i]);  // non-finite input is culled, never rendered
    float lam;  // bounds the covariance's largest eigenvalue
    if (seg.cov6) {
        float S[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) S[k] = at(seg.cov6, i, 6, k);
        lam = 1.01f * sqrtf(S[0] * S[0] + S[3] * S[3] + S[5] * S[5] +
                            2.0f * (S[1] * S[1] + S[2] * S[2] + S[4] * S[4]));
    } else {
        const float l = fmaxf(fmaxf(at(seg.log_scales, i, 3, 0), at(seg.log_scales, i, 3, 1)),
                              at(seg.log_scales, i, 3, 2));
        lam = 1.01f * __builtin_amdgcn_exp2f(2.0f * kLog2e * l);
    }
    const float m1 = fabsf(mx) + fabsf(my) + fabsf(mz);
    uint64_t kept = 0u;  // views
    for (int vi = 0; vi < nv; ++vi) {
        const bool keep = drawable && !cannot_draw(a, s_cams[vi].cam, s_cams[vi].bound, mx, my, mz, m1, lam);
        if (valid && !keep) a.tiles_touched[s_cams[vi].base + i] = 0u;
        kept |= (uint64_t)keep << vi;
    }
    // the Gaussians with a view, as many at a time as rows are left
    const uint64_t any = __ballot(kept != 0u);
    const int rank = __popcll(any & lt_mask), total = __popcll(any);
    for (int b = 0; b < total;) {  // uniform
        if (rows == kRowsLds) {  // the pairs listed still read the rows in LDS
            while (listed > 0) project(min(listed, 64));
            rows = copied = 0;
        }
        const int r = min(total - b, kRowsLds - rows);
        const bool in = kept != 0u && rank >= b && rank < b + r;
        const int row = rows + rank - b;
        if (in) W.gid[row] = (uint32_t)i;
        rows += r;
        b += r;
        for (int vi = 0; vi < nv; ++vi) {
            const bool keep = in && ((kept >> vi) & 1ull);
            const uint64_t m = __ballot(keep);
            if (keep)
                W.list[listed + __popcll(m & lt_mask)] = make_uint2((uint32_t)i, (uint32_t)vi | (uint32_t)row << 8);
            listed += __popcll(m);
            if (listed >= 64) project(64);
        }
    }
    while (listed > 0) project(min(listed, 64));
}

// The same for few views, low degrees and smaller launches, where the two steps' chain
// of latencies costs more than the lanes and the traffic they save (the rule
// is in launch_project): one Gaussian per lane and every view in turn.
// (Degree 3 in planes holds all 48 coefficients in flight: three waves, else it
// spills 18 registers and writes 70 MB of scratch per million Gaussians.)
template <int D, bool PLANES, bool ONE>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(PLANES && D == 3 ? 3 : 4, 6))) project_direct_kernel(const ProjectArgs a) {
    constexpr int K = (D + 1) * (D + 1);
    extern __shared__ __attribute__((aligned(16))) char s_dyn[];  // ProjectCams[nv]
    const ProjectBlock B = project_block<ONE, false>(a, s_dyn);
    const gs_gaussians &seg = a.seg[ONE ? 0 : B.k];
    const int64_t i = (int64_t)B.block * 256 + threadIdx.x, n = seg.n;
    if (i >= n) return;
    // component k of Gaussian i in an attribute of w components
    auto at = [&](const float *p, int w, int k) { return PLANES ? p[(int64_t)k * n + i] : p[w * i + k]; };
    const float mx = at(seg.means, 3, 0), my = at(seg.means, 3, 1), mz = at(seg.means, 3, 2);
    // the small attribute rows (rotation, scales, opacity: 32 B) are requested
    // together with the mean, so their latency overlaps; the SH rows are read
    // only once the Gaussian is known to land in a view
    const float opac = seg.opacity[i];
    float4 q4 = make_float4(1.0f, 0.0f, 0.0f, 0.0f);
    float ls[3] = {0.0f, 0.0f, 0.0f};
    float S[6];
    if (seg.cov6) {
#pragma unroll
        for (int k = 0; k < 6; ++k) S[k] = at(seg.cov6, 6, k);
    } else {
        if (PLANES)
            q4 = make_float4(at(seg.quats, 4, 0), at(seg.quats, 4, 1), at(seg.quats, 4, 2), at(seg.quats, 4, 3));
        else
            q4 = reinterpret_cast<const float4 *>(seg.quats)[i];
#pragma unroll
        for (int k = 0; k < 3; ++k) ls[k] = at(seg.log_scales, 3, k);
    }
    // near-plane test from the mean alone: a Gaussian behind every camera of
    // the launch is done
    bool any_front = false;
    for (int vi = 0; vi < B.nv; ++vi) {
        const float *c = B.cams[vi].cam;
        any_front |= c[6] * mx + c[7] * my + c[8] * mz + c[11] > a.near_plane;
    }
    if (!any_front || !isfinite(opac)) {  // non-finite input is culled, never rendered
        for (int vi = 0; vi < B.nv; ++vi) a.tiles_touched[B.cams[vi].base + i] = 0u;
        return;
    }
    if (!seg.cov6) {
        const Rot rot = quat_rot(q4.x, q4.y, q4.z, q4.w);
        float s[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) s[k] = expf(ls[k]);
        cov_from_rot_scale(rot.R, s, S);
    }
    const float *shp = seg.sh + (PLANES ? (size_t)i : (size_t)(3 * K) * i);
    for (int vi = 0; vi < B.nv; ++vi) {
        const int64_t inst = B.cams[vi].base + i;
        const float *cam = B.cams[vi].cam;
        ViewProj p;
        if (!ewa_project(cam, mx, my, mz, S, a.W, a.H, a.TX, a.TY, a.near_plane, a.lowpass, a.sigma_cut, a.fov_clamp,
                         p)) {
            a.tiles_touched[inst] = 0u;
            continue;
        }
        float Y[K];
        view_basis<D>(cam, mx, my, mz, Y);
        float col[3] = {0.0f, 0.0f, 0.0f};  // accumulated per channel in basis order
        if (PLANES) {
#pragma unroll
            for (int f = 0; f < 3 * K; ++f) col[f % 3] += Y[f / 3] * shp[(int64_t)f * n];
        } else if ((3 * K) % 4 == 0) {
#pragma unroll
            for (int k4 = 0; k4 < 3 * K / 4; ++k4) {
                const float4 t = reinterpret_cast<const float4 *>(shp)[k4];
                const float v4[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) col[(4 * k4 + e) % 3] += Y[(4 * k4 + e) / 3] * v4[e];
            }
        } else {
#pragma unroll
            for (int f = 0; f < 3 * K; ++f) col[f % 3] += Y[f / 3] * shp[f];
        }
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) col[ch] = fmaxf(col[ch] + 0.5f, 0.0f);
        float4 *r = a.rec + 3 * inst;
        r[0] = make_float4(p.u, p.v, p.tz, __int_as_float(p.radius));
        r[1] = make_float4(p.A, p.B, p.C, opac);
        r[2] = make_float4(col[0], col[1], col[2], cam[19]);
        a.tiles_touched[inst] = (uint32_t)((p.rect.x1 - p.rect.x0) * (p.rect.y1 - p.rect.y0));
    }
}

hipError_t launch_project(ProjectArgs a, hipStream_t s) {
    if (a.n_segs == 0) return hipSuccess;
    int64_t bytes = 0;  // attributes, records and counts
    int64_t n = 0, pairs = 0;
    int nv = 0;
    const int K = (a.seg[0].sh_degree + 1) * (a.seg[0].sh_degree + 1);
    const bool planes = a.seg[0].layout == GS_LAYOUT_PLANES;
    for (int k = 0; k < a.n_segs; ++k) {
        const int views = a.first_pair[k + 1] - a.first_pair[k];
        bytes += a.seg[k].n * (44 + 12 * K + 52 * (int64_t)views);
        n += a.seg[k].n;
        pairs += a.seg[k].n * views;
        nv = std::max(nv, views);
    }
    // Two steps trade a longer chain of latencies for lanes and for the SH rows'
    // traffic, so they win where there is much of that: at degree 3, with eight to
    // twenty-four views a Gaussian (with more, nearly every Gaussian is kept by some
    // view and the direct kernel's reads serve many), planes with several, whose
    // scattered columns cost it most; and once the launch has left the 256 MB cache
    // well behind.  Measured in two rooms, direct / two steps, us: 8 views of 0.8M
    // 134 / 110 and 101 / 92, 16 of 0.8M 217 / 209 and 172 / 162, 24 of 0.4M 141 /
    // 111 and 148 / 121, 64 views of 8 scenes of very different sizes 842 / 741; 32
    // of 0.4M 178 / 165 and 211 / 222, 48 of 0.4M 273 / 291 and 310 / 334, 64 of 0.4M
    // 371 / 407 and 402 / 445; below 400 MB 8 views of 0.4M 50 / 53 and 42 / 48, 16 of
    // 0.2M 51 / 48 and 45 / 40; 2 views of 1.3M 45 / 56, 4 of 1.4M 135 / 140, 6 of 2.3M
    // 285 / 290, 32 views of 8 equal scenes 169 / 189; degree 2: 4 views of 1.2M 85 /
    // 98, 16 of 0.45M 73 / 85, 48 of 0.3M 153 / 180; degree 0: 16 views of 0.5M 54 / 68.
    // Planes of degree 3: 2 views of 1.3M 251 / 82, 16 of 0.4M 495 / 104, 64 of 0.35M
    // 1602 / 342; of degree 1: 8 of 0.9M 84 / 88.
    const bool two_steps = K == 16 && bytes >= (int64_t)400 << 20 &&
                           (planes ? nv > 1 : pairs >= 8 * n && pairs <= 24 * n);
    a.first_block[0] = 0;
    for (int k = 0; k < a.n_segs; ++k)
        a.first_block[k + 1] = a.first_block[k] + (uint32_t)((a.seg[k].n + 255) / 256);
    const dim3 grid(a.first_block[a.n_segs]);
    const size_t lds = sizeof(ProjectCams) * (size_t)nv;
    if (two_steps)
        return planes ? launch_kernel_lds(project_kernel<true>, grid, dim3(256), lds, s, a)
                      : launch_kernel_lds(project_kernel<false>, grid, dim3(256), lds, s, a);
#define GS_PROJECT(D, PLANES)                                                                                \
    (a.n_segs == 1 ? launch_kernel_lds(project_direct_kernel<D, PLANES, true>, grid, dim3(256), lds, s, a)   \
                   : launch_kernel_lds(project_direct_kernel<D, PLANES, false>, grid, dim3(256), lds, s, a))
    if (planes) {
        switch (a.seg[0].sh_degree) {
            case 0: return GS_PROJECT(0, true);
            case 1: return GS_PROJECT(1, true);
            case 2: return GS_PROJECT(2, true);
            default: return GS_PROJECT(3, true);
        }
    }
    switch (a.seg[0].sh_degree) {
        case 0: return GS_PROJECT(0, false);
        case 1: return GS_PROJECT(1, false);
        case 2: return GS_PROJECT(2, false);
        default: return GS_PROJECT(3, false);
    }
#undef GS_PROJECT
}

}  // namespace gs
