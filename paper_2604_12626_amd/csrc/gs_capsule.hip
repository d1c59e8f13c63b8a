// gs_capsule_queries kernel: clearance to the nearest avatar capsule and
// swept-step blocking for a batch of agents (Sec. 3.3, Sec. 3.4).
//
// One wave64 per agent: the lanes take the capsules of the agent's avatars
// in turn (capsule j on lane j mod 64), interpolate each in its avatar's
// clip, and keep their smallest gaps; a butterfly of lane exchanges then
// gives the wave minimum (smallest capsule index on ties).  The agent is a
// vertical capsule (axis from its base point up `height`); a step sweeps
// that axis into the parallelogram {p0 + a (p1 - p0) + b height z}.
#include "gs_internal.hpp"

namespace gs {

struct V3 {
    float x, y, z;
};
__device__ __forceinline__ V3 v3(float x, float y, float z) { return {x, y, z}; }
__device__ __forceinline__ V3 operator+(V3 a, V3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ V3 operator-(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3 operator*(float s, V3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ float dot(V3 a, V3 b) { return fmaf(a.x, b.x, fmaf(a.y, b.y, a.z * b.z)); }
__device__ __forceinline__ V3 cross(V3 a, V3 b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ float clamp01(float t) { return fminf(fmaxf(t, 0.0f), 1.0f); }

// squared distance between segments p0 + s u and q0 + t v, s, t in [0, 1]:
// the parameter of one segment is found for the other's, clamped, and the
// first refit to the clamped second (the standard closest-point sequence)
__device__ float seg_seg_dist2(V3 p0, V3 u, V3 q0, V3 v) {
    const V3 w = p0 - q0;
    const float a = dot(u, u), c = dot(v, v), e = dot(v, w);
    float s, t;
    if (a <= 1e-20f && c <= 1e-20f) {
        s = t = 0.0f;
    } else if (a <= 1e-20f) {
        s = 0.0f;
        t = clamp01(e / c);
    } else {
        const float d = dot(u, w);
        if (c <= 1e-20f) {
            t = 0.0f;
            s = clamp01(-d / a);
        } else {
            const float b = dot(u, v);
            const float den = a * c - b * b;
            s = den > 1e-7f * a * c ? clamp01((b * e - c * d) / den) : 0.0f;
            t = (b * s + e) / c;
            if (t < 0.0f) {
                t = 0.0f;
                s = clamp01(-d / a);
            } else if (t > 1.0f) {
                t = 1.0f;
                s = clamp01((b - d) / a);
            }
        }
    }
    const V3 r = (w + s * u) - t * v;
    return dot(r, r);
}

// distance between the segment s0 + l sd (l in [0, 1]) and the
// parallelogram o + a U + b V: zero where the segment crosses it, else the
// least of the segment against the four edges and of the two end points
// against the interior
__device__ float seg_parallelogram_dist(V3 s0, V3 sd, V3 o, V3 U, V3 V) {
    float best = seg_seg_dist2(s0, sd, o, U);
    best = fminf(best, seg_seg_dist2(s0, sd, o + V, U));
    best = fminf(best, seg_seg_dist2(s0, sd, o, V));
    best = fminf(best, seg_seg_dist2(s0, sd, o + U, V));
    best = sqrtf(best);
    const float g11 = dot(U, U), g12 = dot(U, V), g22 = dot(V, V);
    const float gd = g11 * g22 - g12 * g12;
    if (gd > 1e-7f * g11 * g22) {
        const V3 n = cross(U, V);
        const float rn = 1.0f / sqrtf(dot(n, n));
        const V3 ends[2] = {s0, s0 + sd};
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const V3 r = ends[k] - o;
            const float ru = dot(r, U), rv = dot(r, V);
            const float a = (g22 * ru - g12 * rv) / gd, b = (g11 * rv - g12 * ru) / gd;
            if (a >= 0.0f && a <= 1.0f && b >= 0.0f && b <= 1.0f) best = fminf(best, fabsf(dot(r, n)) * rn);
        }
        // crossing: s0 + l sd = o + a U + b V, by Cramer's rule on
        // [sd, -U, -V] (l, a, b) = o - s0
        const V3 mu = -1.0f * U, mv = -1.0f * V, rhs = o - s0;
        const float det = dot(sd, cross(mu, mv));
        const float scale = sqrtf(dot(sd, sd) * g11 * g22);
        if (fabsf(det) > 1e-6f * scale) {
            const float l = dot(rhs, cross(mu, mv)) / det;
            const float a = dot(sd, cross(rhs, mv)) / det;
            const float b = dot(sd, cross(mu, rhs)) / det;
            if (l >= 0.0f && l <= 1.0f && a >= 0.0f && a <= 1.0f && b >= 0.0f && b <= 1.0f) best = 0.0f;
        }
    }
    return best;
}

// (gap, index) lexicographic minimum
__device__ __forceinline__ void take_min(float &g, int &i, float g2, int i2) {
    if (g2 < g || (g2 == g && i2 < i)) {
        g = g2;
        i = i2;
    }
}

// The swept step is asked only of the capsules that can attain its minimum.
// Every point of the step's parallelogram lies within |step| of the agent's
// axis at its start, which is itself part of the parallelogram, so a capsule's
// step gap is at least its clearance less |step|, and the least step gap is
// at most the least clearance: a capsule whose clearance exceeds the least by
// more than |step| (and a margin for rounding) cannot attain it.  The few that
// remain are compacted over the wave, so that one round of lanes usually takes
// them all instead of one per 64 capsules.  Bound by the VALU and the chain of
// loads to the capsules; 4096 agents against 184 capsules each 17.9 ->
// 12.1 us.
constexpr int kCapChunk = 512;  // capsules of an agent looked at before their steps

// ROUND: no agent has more capsules than lanes, and there are many agents: each
// lane asks its capsule for both, which saves the second round and registers
// (launch_capsule_queries).
template <bool ROUND>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(ROUND ? 7 : 6)))
capsule_query_kernel(const CapsuleArgs a) {
    __shared__ float s_least[4][ROUND ? 1 : kCapChunk];
    __shared__ uint16_t s_list[4][ROUND ? 1 : kCapChunk];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t e = (int64_t)blockIdx.x * 4 + wave;
    if (e >= a.n_agents) return;  // whole waves leave together
    const V3 p0 = v3(a.agent_pos[3 * e], a.agent_pos[3 * e + 1], a.agent_pos[3 * e + 2]);
    const bool step = a.agent_next != nullptr;
    V3 sd = v3(0.0f, 0.0f, 0.0f);
    if (step) sd = v3(a.agent_next[3 * e], a.agent_next[3 * e + 1], a.agent_next[3 * e + 2]) - p0;
    const V3 up = v3(0.0f, 0.0f, a.height);
    int first = a.agent_avatars[2 * e], count = a.agent_avatars[2 * e + 1];
    const int lo = max(first, 0), hi = min(first + max(count, 0), a.n_avatars);
    const int n = hi > lo ? (hi - lo) * a.n_caps : 0;
    float best = INFINITY, best_step = INFINITY;
    int best_i = -1;
    const float sdl = sqrtf(dot(sd, sd));
    // what the clearances may be off by: near-parallel axes are taken as
    // parallel, and far coordinates round
    const float far = 1e-5f * (fabsf(p0.x) + fabsf(p0.y) + fabsf(p0.z));
    // a chunk holds capsules of at most 64 avatars, whose clip frames lie one
    // avatar per lane
    const int chunk = (int)min((int64_t)kCapChunk, 63 * (int64_t)a.n_caps);
    const float inv_caps = 1.0f / (float)a.n_caps;
    for (int base = 0; base < n; base += chunk) {  // uniform
        const int m = min(n - base, chunk);
        const int av0 = base / a.n_caps, off = base - av0 * a.n_caps;
        int row0 = 0, row1 = 0;  // first capsule of the avatar's two frames
        float sp = 0.0f;
        if (lo + av0 + lane < hi) {
            // the avatar's clip frames around its position (clamped like the skinning clips)
            const int av = lo + av0 + lane;
            const int cf = min(max(a.clip_first[av], 0), a.clip_total - 1);
            const int frames = min(max(a.clip_frames[av], 1), a.clip_total - cf);
            const float p = a.frame_pos[av];
            const float pc = p > 0.0f ? fminf(p, (float)(frames - 1)) : 0.0f;
            const int f0 = frames > 1 ? min((int)floorf(pc), frames - 2) : 0;
            row0 = cf + f0;
            row1 = cf + (frames > 1 ? f0 + 1 : 0);
            sp = frames > 1 ? pc - (float)f0 : 0.0f;
        }
        // avatar (of the chunk's) of its capsule j.  Below 2^20 the quotient
        // by way of floats is exact: j + 1/2 is at least 1 / (2 n_caps) from
        // a multiple, far above the rounding.
        auto avatar = [&](int j) {
            return a.n_caps < (1 << 20) ? (int)(((float)(j + off) + 0.5f) * inv_caps) : (j + off) / a.n_caps;
        };
        // capsule j of the chunk, interpolated in its clip (every lane takes
        // part in the exchange)
        auto capsule = [&](int j, V3 &ca, V3 &cd, float &r) {
            const int t = avatar(j), c = j + off - t * a.n_caps;
            const int r0 = __shfl(row0, t, 64), r1 = __shfl(row1, t, 64);
            const float s = __shfl(sp, t, 64);
            const float4 *c0 = reinterpret_cast<const float4 *>(a.caps + ((size_t)r0 * a.n_caps + c) * 8);
            const float4 *c1 = reinterpret_cast<const float4 *>(a.caps + ((size_t)r1 * a.n_caps + c) * 8);
            const float4 x0 = c0[0], y0 = c0[1], x1 = c1[0], y1 = c1[1];
            const float t1 = 1.0f - s;
            // Fused as written, so that the last bit, which decides the nearest of
            // two equally near capsules, stays what it has always been: that is
            // how the compiler once fused the plain expression, cb.z alone with
            // the other product inside.  It is no slip: with that component like
            // its neighbours, 1 of 4096 nearest capsules was another one.
            ca = v3(fmaf(s, x1.x, t1 * x0.x), fmaf(s, x1.y, t1 * x0.y), fmaf(s, x1.z, t1 * x0.z));
            const V3 cb = v3(fmaf(s, y1.x, t1 * y0.x), fmaf(s, y1.y, t1 * y0.y), fmaf(t1, y0.z, s * y1.z));
            r = fmaf(s, x1.w, t1 * x0.w);
            cd = cb - ca;
        };
        for (int j0 = 0; j0 < m; j0 += 64) {
            const int j = j0 + lane;
            V3 ca, cd;
            float r;
            capsule(min(j, m - 1), ca, cd, r);
            if (j >= m) continue;
            const float g = sqrtf(seg_seg_dist2(p0, up, ca, cd)) - a.radius - r;
            take_min(best, best_i, g, lo * a.n_caps + base + j);
            if (ROUND && step)
                best_step = fminf(best_step, seg_parallelogram_dist(ca, cd, p0, sd, up) - a.radius - r);
            if (!ROUND && step)  // the least gap its swept step can have
                s_least[wave][j] = g - 1.001f * sdl - 2e-3f * (a.height + sqrtf(dot(cd, cd)) + sdl) -
                                   1e-5f * fabsf(g) - far;
        }
        if (ROUND || !step) continue;  // uniform
        float least = best;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) least = fminf(least, __shfl_xor(least, off, 64));
        lds_wave_sync();
        int cnt = 0;
        for (int j0 = 0; j0 < m; j0 += 64) {
            const int j = j0 + lane;
            const bool in = j < m && !(s_least[wave][j] > least);  // not-a-number stays in
            const uint64_t bal = __ballot(in);
            if (in) s_list[wave][cnt + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)j;
            cnt += __popcll(bal);
        }
        lds_wave_sync();
        for (int k0 = 0; k0 < cnt; k0 += 64) {
            V3 ca, cd;
            float r;
            capsule(s_list[wave][min(k0 + lane, cnt - 1)], ca, cd, r);
            if (k0 + lane < cnt)
                best_step = fminf(best_step, seg_parallelogram_dist(ca, cd, p0, sd, up) - a.radius - r);
        }
        lds_wave_sync();  // the list is read: the next chunk may overwrite it
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float g2 = __shfl_xor(best, off, 64);
        const int i2 = __shfl_xor(best_i, off, 64);
        take_min(best, best_i, g2, i2);
        best_step = fminf(best_step, __shfl_xor(best_step, off, 64));
    }
    if (lane == 0) {
        a.clearance[e] = best;
        if (a.nearest) a.nearest[e] = best_i;
        if (step) {
            a.step_gap[e] = best_step;
            a.blocked[e] = best_step < 0.0f ? 1 : 0;
        }
    }
}

hipError_t launch_capsule_queries(const CapsuleArgs &a, hipStream_t s) {
    if (a.n_agents <= 0) return hipSuccess;
    const unsigned grid = (unsigned)((a.n_agents + 3) / 4);
    // With more agents than the CUs hold at once the second round's work counts,
    // with fewer only its latency, which the steps of a few lanes make up for (one
    // round / two, 23 capsules: 65536 agents 77 / 88 us, 16384 23.7 / 26.8, 4096 11.0
    // / 11.0, 1024 11.5 / 9.3; 46 capsules 80 / 88, 24.8 / 26.9, 11.0 / 11.1).
    if ((int64_t)a.n_avatars * a.n_caps <= 64 && a.n_agents >= 8192)
        return launch_kernel(capsule_query_kernel<true>, dim3(grid), dim3(256), s, a);
    return launch_kernel(capsule_query_kernel<false>, dim3(grid), dim3(256), s, a);
}

}  // namespace gs
