// gs_render_backward kernels.
//
// B1 (one wave64 per 8 x 8 quadrant of a tile): walks the tile's list back
// to front from the last composited entry of the quadrant, 64 entries at a
// time, recomputing each alpha with exactly the forward's FP32 expression (so
// every skip/stop/clamp decision repeats), recovering the transmittance by
// T_i = T_{i+1} / (1 - alpha_i), and forming the screen-space adjoint of each
// entry (u, v, conic, opacity, colour, depth).  Entries that cannot reach the
// quadrant are dropped by the same conservative bound as the forward; the
// sums over the 64 pixels of the remaining ones are taken by the matrix cores
// (below) and leave with FP64 atomics.
// With the forward's segment checkpoints a list is cut into segments of
// kSegment entries (a multiple of that for lists longer than kMaxSegments
// segments), popped by a persistent grid, every segment's walk starting from
// the transmittance and the normalised colour still to come that the forward
// recorded at its end; the last segment of a list starts from t_final and
// the background, as the whole list does without them.
//
// B2 (per Gaussian of a segment, scene-major): chains the screen-space
// adjoints of every view that drew the Gaussian through the projection to the
// 3D parameters and writes the dense gradients once (no atomics).  A first
// pass over the segment (B2a) writes zeros plane by plane and lists the
// Gaussians a view of the launch draws; the chain (B2b) then runs over that
// list only.
#include "gs_ewa.hpp"

namespace gs {

// Sum over the wave, complete in lane 63 only, with DPP lane moves fused
// into the adds (no LDS traffic): pairs, quads, half rows, rows (these leave
// every lane of a 16-lane row holding the row sum), then row 0 into row 1
// and row 2 into row 3, then rows 0-1 into row 3.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float v) {
    // rows outside ROW_MASK add `old` = 0
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}

__device__ __forceinline__ float wave_sum_to_last(float v) {
    v = dpp_add<0xB1, 0xF>(v);   // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E, 0xF>(v);   // quad_perm [2, 3, 0, 1]
    v = dpp_add<0x141, 0xF>(v);  // row_half_mirror
    v = dpp_add<0x140, 0xF>(v);  // row_mirror
    v = dpp_add<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// zeros for p[0, n) by the whole grid: 16-byte stores on the 16-byte aligned
// stretch, the single floats at its ends by workgroup 0
__device__ __forceinline__ void zero_span_grid(float *p, int64_t n) {
    const uint64_t base = (uint64_t)(uintptr_t)p;  // 4-byte aligned (floats)
    int64_t v0 = 0, v1 = n;
    while (((base + 4u * (uint64_t)v0) & 15u) && v0 < n) ++v0;
    while (((base + 4u * (uint64_t)v1) & 15u) && v1 > v0) --v1;
    if (blockIdx.x == 0) {
        for (int64_t f = threadIdx.x; f < v0; f += blockDim.x) p[f] = 0.0f;
        for (int64_t f = v1 + threadIdx.x; f < n; f += blockDim.x) p[f] = 0.0f;
    }
    float4 *q = reinterpret_cast<float4 *>(p + v0);
    const int64_t m = (v1 - v0) / 4, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < m; k += stride)
        q[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

// The screen-space sums of one entry over the 64 pixels of a quadrant are
// products of small matrices, and the matrix cores take them.  With
//   g(e, p) = dL/dalpha * G   (0 where the entry is skipped or clamped)
//   w(e, p) = alpha * T       (0 where it is skipped)
// and (dx, dy) the pixel relative to the entry's centre, the adjoints of entry
// e are combinations of the six sums of g dx^a dy^b, a + b <= 2, and of four
// sums of w times dL/dred, green, blue, depth of the pixel.  A batch of kBatch
// entries writes its g and w rows to LDS (lane = pixel) and reads them back
// transposed:
//  - g: a column of eight pixels a lane.  v_mfma_f32_4x4x1_16b_f32 multiplies
//    sixteen pairs of matrices at once, one for each entry and half of the
//    quadrant: rows are the half's four columns of pixels, k the image rows,
//    columns 1, dy, dy^2 of the entry.  The four columns are then summed with
//    1, dx, dx^2 in the lane.
//  - w: rows are the entries' halves, k the pixels of a half, columns the
//    pixels' adjoints (in registers for the whole walk): v_mfma_f32_16x16x4_f32.
// Every term is about the entry's own centre: taken about the quadrant's and
// shifted afterwards, with features common to all entries, sum g dx^2 of an
// entry of about a pixel at the quadrant's corner was the difference of terms
// some forty times its size, and lost seven bits.  Chains of FP32 roundings
// are short (eight image rows and two pairs of columns; four times eight
// pixels and two pairs), halves and quadrants are added in FP64.  RMS errors
// of one quadrant's sums, of the sum of magnitudes, against 64 bits -- a sum
// over the lanes by DPP adds / moments about the quadrant's centre / this --
// for entries of 0.35 px^2: conic 3.4e-8 / 4.4e-6 / 3.2e-8, position 3.2e-8 /
// 3.2e-7 / 3.0e-8; of 40 px^2: conic 1.5e-8 / 3.6e-8 / 1.5e-8.
// (Ten sums over the lanes took 60 of 165 VALU instructions per entry, and the
// products they summed another 30; this takes about 42 in all.)
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kBatch = 8;      // entries per batch: rows 0..7 are their g, rows 8..15 their w
constexpr int kGwStride = 68;  // floats per row: the b128 reads of 16 lanes fall on different banks
enum { kS0 = 0, kSx, kSxx, kSy, kSxy, kSyy, kSums };  // sums of g dx^a dy^b

// One wave per workgroup walks one 8 x 8 quadrant of a (view, tile) list, or
// with checkpoints of one segment of one, one pixel per lane; no wave waits
// for another.  The four quadrants of an item are neighbours in one XCD's
// share of the workgroups, so its list is gathered through one L2.  10 KB of
// LDS and 128 registers: four waves per SIMD.
// The adjoints of a chunk leave with one FP64 atomic per surviving (entry,
// adjoint), consecutive lanes on consecutive adjoints of an entry: an entry's
// ten meet in one or two cache lines (one entry per lane took twice as long
// as the rest of the kernel).
// Bound by the VALU (86 % of its issue; the matrix cores 15 %).  Against a
// 256-thread workgroup per tile whose quadrants walked in step and summed with
// DPP adds: 16 views of 640 x 480 over 1.4M Gaussians 3577 -> 1640 us, a 1280
// x 720 view of 1M 341 -> 195 us, a 256 x 256 view of 500k in segments 52.7 ->
// 34.9 us (with the FP32 moments about the quadrant's centre 1571, 192, 34.3).
__global__ void __launch_bounds__(64, 4) backward_tile_kernel(const BackwardTileArgs a) {
    // the chunk's staged survivors (u, v, a, b) (c, o, z, r) (g, b) and their
    // list positions inside the chunk, back to front; the batch's g and w
    // rows.  A batch's sums of g replace the first two of its survivors; after
    // the walk the adjoints replace all of Stage, and the survivors' rows of
    // the accumulators their positions
    struct Stage {
        float4 e0[64], e1[64], e3[64];  // e3: sums only
        float gw[2 * kBatch][kGwStride];
    };
    __shared__ __attribute__((aligned(16))) Stage s_st;
    __shared__ float2 s_e2[64];
    __shared__ __attribute__((aligned(16))) uint32_t s_pos[64];
    __shared__ float s_w[2][4][64];  // sums of w over each half, times red, green, blue, depth
    static_assert(sizeof(Stage) >= 64 * kG2D * sizeof(double), "the adjoints of a chunk fit over the staging");
    static_assert(sizeof(s_st) + sizeof(s_e2) + sizeof(s_pos) + sizeof(s_w) <= 160 * 1024 / 16,
                  "sixteen workgroups share a CU's LDS");
    double *out = reinterpret_cast<double *>(&s_st);
    // sum c of half h of survivor p, in floats: in e0, e1 (halves) and e3
    auto sum_at = [](int h, int c, int p) { return (c < 4 ? 256 * h + c : 512 + 2 * h + c - 4) + 4 * p; };
    float *sums = reinterpret_cast<float *>(&s_st);
    float4 *e0s = s_st.e0, *e1s = s_st.e1;
    float2 *e2s = s_e2;
    float(*gw)[kGwStride] = s_st.gw;
    const int lane = threadIdx.x;
    const uint64_t gt_mask = lane == 63 ? 0ull : ~0ull << (lane + 1);
    // a row of g or w holds pixel (x, y) of the quadrant at 8 x + y
    const int slot_px = ((lane & 7) << 3) | (lane >> 3);
    // v_mfma_f32_4x4x1_16b_f32: block lane / 4 (entry lane / 8 of the batch, half
    // lane / 4 % 2); A row lane % 4 (so pixel column lane % 8), B column lane % 4;
    // D row = register, column lane % 4.  Lane's B: 1, dy, dy^2 (columns 0, 1, 2)
    const int g_at = (lane >> 3) * kGwStride + ((lane & 7) << 3), half = (lane >> 2) & 1, col = lane & 3;
    const int at0 = sum_at(half, col == 0 ? kS0 : col == 1 ? kSy : kSyy, 0), at1 = sum_at(half, col == 0 ? kSx : kSxy, 0);
    const float b1 = col == 0 ? 0.0f : 1.0f, b2 = col == 2 ? 1.0f : 0.0f, b3 = 1.0f - b2;
    // v_mfma_f32_16x16x4_f32: A row / B column lane % 16, k = lane / 16, D row 4
    // (lane / 16) + register, column lane % 16.  A row: entry row % 8 over half
    // row / 8; columns 0..3 are the adjoints of the first half's pixels, 8..11
    // of the second's (set per walk)
    const int mi = lane & 15, mk = lane >> 4;
    const int w_at = (mi & 7) * kGwStride + 32 * (mi >> 3) + 8 * mk;
    const bool d_col = (mi & 7) < 4;
    float feat_d[8] = {};
    // work: quadrant (k & 3) of the (k >> 2)-th item of queue q, for workgroup
    // 8 k + q: a (view, tile) list, or with checkpoints a listed segment of one
    const uint32_t n_work = a.seg_list ? a.seg_list[0] : (uint32_t)a.n_items;
    const uint32_t xq = blockIdx.x % kOrderQueues;
    for (uint32_t k = blockIdx.x / kOrderQueues;; k += a.n_groups / kOrderQueues) {
    const uint32_t wk = (k >> 2) * kOrderQueues + xq;
    const int wave = (int)(k & 3u);  // the quadrant
    if (wk >= n_work) break;
    const uint32_t entry = a.seg_list ? a.seg_list[1 + wk] : 0u;
    // whole lists with the work order: queue q holds the lists t = q mod 8,
    // longest first
    const int64_t item = a.seg_list ? (int64_t)(entry >> 6)
                         : a.order  ? (int64_t)a.order[(int64_t)xq * order_stride(a.n_items) + (k >> 2)]
                                    : (int64_t)wk;
    const uint32_t s = a.seg_list ? (entry & 63u) : 0u;
    const int view = (int)(item / a.T);
    const int tile = (int)(item - (int64_t)view * a.T);
    const int qx0 = (tile % a.TX) * kTile + ((wave & 1) << 3);
    const int qy0 = (tile / a.TX) * kTile + ((wave >> 1) << 3);
    const int px = qx0 + (lane & 7), py = qy0 + (lane >> 3);
    const bool inside = px < a.W && py < a.H;
    const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
    const float bx0 = (float)qx0 + 0.5f, by0 = (float)qy0 + 0.5f;
    const uint2 range = a.ranges[item];
    const uint32_t L = range.y - range.x;
    // this segment [seg_lo, seg_lo + seg_len) of list positions: all of them
    // without checkpoints, else segment s of the list's segments (kSegment
    // entries each, or a multiple of that for lists of more than
    // kMaxSegments * kSegment entries)
    static_assert(kSegment == 64 && kMaxSegments <= 64, "six bits name a segment; a chunk is 64 entries");
    const uint32_t seg_len = a.seg_list ? seg_len_of(L) : L;
    const uint32_t seg_lo = a.seg_list ? s * seg_len : 0u;
    const bool last_seg = !a.seg_list || seg_lo + seg_len >= L;
    // A one-chunk middle segment's list values, records and end checkpoint
    // are requested before the pixel state, so that the gather overlaps those
    // loads (requests past what the walk needs are harmless: positions below
    // the list length, slots inside the buffer).
    // A middle segment whose end checkpoint lies past the buffer (sized for a
    // smaller capacity than the binning's) walks from the end of the list,
    // where t_final and the background give the state, and adds only its own
    // entries: the same gradients, slower.
    const uint64_t slot = (range.x + seg_lo + seg_len) / kSegment;
    const bool from_end = !last_seg && slot >= a.ckpt_slots;
    const bool middle = !last_seg && !from_end;
    const bool pre = middle && seg_len == kSegment;
    uint32_t g_pre = 0;
    float4 p0 = make_float4(0.f, 0.f, 0.f, 0.f), p1 = p0, p2 = p0;
    if (pre && seg_lo + lane < L) {
        g_pre = a.vals[range.x + seg_lo + lane];
        p0 = a.rec[3 * (size_t)g_pre];
        p1 = a.rec[3 * (size_t)g_pre + 1];
        p2 = a.rec[3 * (size_t)g_pre + 2];
    }
    const bool ck_ok = middle;
    float ck[kCkptVals] = {1.0f, a.bg0, a.bg1, a.bg2, 0.0f};
    if (ck_ok) {
#pragma unroll
        for (int v = 0; v < kCkptVals; ++v) ck[v] = a.ckpt[ckpt_index(slot, wave, v, lane)];
    }

    float T = 1.0f, Tfin = 1.0f;
    uint32_t last = 0;
    float dR = 0.f, dG = 0.f, dB = 0.f, dD = 0.f, dA = 0.f;
    if (inside) {
        const size_t pix = ((size_t)view * a.H + py) * a.W + px;
        Tfin = a.t_final[pix];
        T = Tfin;
        last = a.n_contrib[pix];
        if (a.d_rgb) {
            dR = a.d_rgb[3 * pix];
            dG = a.d_rgb[3 * pix + 1];
            dB = a.d_rgb[3 * pix + 2];
        }
        if (a.d_depth) dD = a.d_depth[pix];
        if (a.d_alpha) dA = a.d_alpha[pix];
    }
    uint32_t maxlast = last;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) maxlast = max(maxlast, (uint32_t)__shfl_xor((int)maxlast, off, 64));
    maxlast = min(maxlast, L);
    const uint32_t seg_end = (last_seg || from_end) ? maxlast : seg_lo + seg_len;  // state known here
    const uint32_t own_hi = from_end ? seg_lo + seg_len : seg_end;  // entries this walk adds
    const uint32_t seg_hi = seg_end < maxlast ? seg_end : maxlast;
    if (seg_lo >= seg_hi) continue;
    // the suffix colour and depth behind the current entry over its
    // transmittance (the background at the end of the walk, else the
    // checkpoint at seg_end): the walk needs the colour only through its
    // product S with the pixel's adjoint of the colour; the depth Z, many
    // times the colours' size, on its own, so that its rounding stays its own
    float Sr = a.bg0, Sg = a.bg1, Sb = a.bg2, Z = 0.0f;
    if (seg_end < maxlast && ck_ok) {
        T = ck[0];
        Sr = ck[1];
        Sg = ck[2];
        Sb = ck[3];
        Z = ck[4];
    }
    float S = dR * Sr + dG * Sg + dB * Sb;
    const float dAT = dA * Tfin;
    const float amax = __builtin_canonicalizef(a.alpha_max);  // keeps the clamp's operand out of the loop
    // the image adjoints as feature columns; a pixel whose adjoint is not
    // finite would reach every entry of the product, so its column entry is
    // zero and its share is added apart (below)
    const bool odd_px = !(isfinite(dR) && isfinite(dG) && isfinite(dB) && isfinite(dD));
    const uint64_t odd_any = __ballot(odd_px);
    {
        float *st = &gw[0][0] + slot_px;
        lds_wave_sync();
        st[0] = odd_px ? 0.0f : dR;
        st[kGwStride] = odd_px ? 0.0f : dG;
        st[2 * kGwStride] = odd_px ? 0.0f : dB;
        st[3 * kGwStride] = odd_px ? 0.0f : dD;
        lds_wave_sync();
        if (d_col) {
            const f32x4 *src = reinterpret_cast<const f32x4 *>(&gw[0][0] + w_at);
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const f32x4 f = src[m];
#pragma unroll
                for (int c = 0; c < 4; ++c) feat_d[4 * m + c] = f[c];
            }
        }
        lds_wave_sync();
    }

    // chunks [lo, hi) of list positions, from the back (this wave's entries
    // end at seg_hi); while one is walked the next chunk's records and the
    // list values of the one after are in flight (every load unconditional:
    // a lane past the chunk or the list's front reads an entry of the list)
    float4 q0 = p0, q1 = p1, q2 = p2;
    uint32_t g = g_pre, g_next = 0u;
    const int32_t seg_a = (int32_t)seg_lo, jl = (int32_t)L - 1;
    auto position = [&](int32_t hi) {  // this lane's position in the chunk that ends at hi
        return range.x + (uint32_t)min(max(hi - 64, seg_a) + lane, jl);
    };
    if (!pre) {
        g = a.vals[position((int32_t)seg_hi)];
        g_next = a.vals[position((int32_t)seg_hi - 64)];
        q0 = a.rec[3 * (size_t)g];
        q1 = a.rec[3 * (size_t)g + 1];
        q2 = a.rec[3 * (size_t)g + 2];
    }
    // a middle segment's records, requested up front, are those of its whole
    // chunk: positions from its first entry on
    for (int32_t hi = (int32_t)seg_hi; hi > seg_a; hi -= 64) {
        const int32_t lo = max(hi - 64, seg_a);
        const uint32_t id = g;
        const float cu = q0.x, cv = q0.y, cA = q1.x, cB = q1.y, cC = q1.z, co = q1.w;
        uint4 grp = make_uint4(0u, 0u, 0u, 0u);
        const bool hit = lo + lane < hi && entry_reaches_box(cu, cv, cA, cB, cC, co, a.alpha_min, bx0, by0,
                                                             bx0 + 7.0f, by0 + 7.0f);
        const uint64_t bal = __ballot(hit);
        const int n = __popcll(bal);
        if (hit) {  // staged back to front
            const int pos = __popcll(bal & gt_mask);
            const Entry e = make_entry(q0, q1, q2);
            e0s[pos] = make_float4(e.u, e.v, e.a, e.b);
            e1s[pos] = make_float4(e.c, e.o, e.z, e.r);
            e2s[pos] = make_float2(e.g, e.bl);
            s_pos[pos] = (uint32_t)lane;
            grp = a.slots[id >> 6];  // (in flight while the chunk is walked)
        }
        if (hi - 64 > seg_a) {
            g = g_next;
            q0 = a.rec[3 * (size_t)g];
            q1 = a.rec[3 * (size_t)g + 1];
            q2 = a.rec[3 * (size_t)g + 2];
            g_next = a.vals[position(hi - 128)];
        }
        // pad to a multiple of 4 with entries of no position (never taken)
        if (lane < ((4 - (n & 3)) & 3)) {
            e0s[n + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            e1s[n + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            e2s[n + lane] = make_float2(0.0f, 0.0f);
            s_pos[n + lane] = ~0u;
        }
        lds_wave_sync();
        const uint32_t last_in = last > (uint32_t)lo ? last - (uint32_t)lo : 0u;  // positions below it contribute
        for (int q = 0; q < n; q += kBatch) {
            const int nb = min(n - q, kBatch);  // entries of this batch
            // four entries per step: their LDS reads and alphas together,
            // then the chain through T and S
            for (int e = 0; e < nb; e += 4) {
                const uint4 p4 = *reinterpret_cast<const uint4 *>(&s_pos[q + e]);
                const uint32_t pos[4] = {p4.x, p4.y, p4.z, p4.w};
                float G[4], oG[4], at[4], r[4], c[4], z[4];
                bool take[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float4 e0 = e0s[q + e + u], e1 = e1s[q + e + u];
                    const float2 e2 = e2s[q + e + u];
                    const float dx = fx - e0.x, dy = fy - e0.y;
                    G[u] = fast_exp2(entry_power2(e0.z, e0.w, e1.x, dx, dy));
                    oG[u] = e1.y * G[u];
                    const float al = fminf(amax, oG[u]);
                    take[u] = pos[u] < last_in && !(al < a.alpha_min);
                    at[u] = take[u] ? al : 0.0f;
                    r[u] = __builtin_amdgcn_rcpf(1.0f - at[u]);  // 1 ulp reciprocal (1 where skipped)
                    c[u] = fmaf(dR, e1.w, fmaf(dG, e2.x, dB * e2.y));
                    z[u] = e1.z;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    T = T * r[u];  // transmittance in front of this entry
                    // d . (c - S): what the entry's colour and depth change
                    const float dc = take[u] ? c[u] - S : 0.0f, dz = z[u] - Z;
                    const float dal = fmaf(T, fmaf(dD, dz, dc), dAT * r[u]);
                    S = fmaf(at[u], dc, S);
                    Z = fmaf(at[u], dz, Z);
                    gw[e + u][slot_px] = take[u] && !(oG[u] > a.alpha_max) ? dal * G[u] : 0.0f;
                    gw[kBatch + e + u][slot_px] = at[u] * T;
                }
            }
            lds_wave_sync();
            {
                const f32x4 *wr = reinterpret_cast<const f32x4 *>(&gw[kBatch][0] + w_at);
                const f32x4 wv[2] = {wr[0], wr[1]};
                f32x4 sw[4] = {};
#pragma unroll
                for (int st = 0; st < 8; ++st)
                    sw[st & 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[st >> 2][st & 3], feat_d[st], sw[st & 3], 0, 0, 0);
                if (d_col && (mi >> 3) == (mk >> 1)) {  // entries 4 (mk % 2) + r, over their own half
                    const int e4 = 4 * (mk & 1);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (e4 + r < nb) s_w[mi >> 3][mi & 7][q + e4 + r] = (sw[0][r] + sw[1][r]) + (sw[2][r] + sw[3][r]);
                }
            }
            {
                const int p = min(q + (lane >> 3), n - 1);  // this lane's entry (past the batch: not stored)
                const float2 uv = *reinterpret_cast<const float2 *>(&e0s[p]);
                const f32x4 *gr = reinterpret_cast<const f32x4 *>(&gw[0][0] + g_at);
                const f32x4 gv[2] = {gr[0], gr[1]};
                const float y0 = col == 0 ? 1.0f : by0 - uv.y, u0 = uv.x - (bx0 + (float)(4 * half));
                f32x4 U = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int y = 0; y < 8; ++y) {
                    const float dy = fmaf(b1, (float)y, y0);  // 1 in column 0
                    U = __builtin_amdgcn_mfma_f32_4x4x1f32(gv[y >> 2][y & 3], dy * fmaf(b2, dy, b3), U, 0, 0, 0);
                }
                float dx[4], t[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    dx[x] = (float)x - u0;
                    t[x] = dx[x] * U[x];
                }
                lds_wave_sync();  // every lane has its entry's centre: the sums take its place
                if ((lane >> 3) < nb && col < 3) {
                    float *o = sums + 4 * p;
                    o[at0] = (U[0] + U[1]) + (U[2] + U[3]);
                    if (col < 2) o[at1] = (t[0] + t[1]) + (t[2] + t[3]);
                    if (col == 0)
                        o[at0 + kSxx] = fmaf(dx[1], t[1], dx[0] * t[0]) + fmaf(dx[3], t[3], dx[2] * t[2]);
                }
            }
            if (odd_any) {  // uniform; rare
                lds_wave_sync();
                const float dv[4] = {dR, dG, dB, dD};
                for (int e = 0; e < nb; ++e) {
                    const float w = gw[kBatch + e][slot_px];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float sum = wave_sum_to_last(odd_px && w != 0.0f ? w * dv[k] : 0.0f);
                        if (lane == 63) s_w[0][k][q + e] += sum;
                    }
                }
            }
            lds_wave_sync();
        }
        // the survivors' adjoints from their sums, each by the lane that holds
        // its record (a walk from the list's end passes others' entries): with
        // dL/dP = o g,
        //   u, v: o (A sx + B sy), o (B sx + C sy)   with sx = sum g dx, sy = sum g dy
        //   conic: -o/2 sum g dx^2, -o sum g dx dy, -o/2 sum g dy^2;  opacity: sum g
        const int pos = __popcll(bal & gt_mask);
        double sum[kSums];
#pragma unroll
        for (int c = 0; c < kSums; ++c)
            sum[c] = hit ? (double)sums[sum_at(0, c, pos)] + (double)sums[sum_at(1, c, pos)] : 0.0;
        lds_wave_sync();  // the adjoints take the sums' place
        if (hit) {
            double *o = out + pos * kG2D;
            if ((uint32_t)(lo + lane) < own_hi) {
                o[kGU] = (double)co * ((double)cA * sum[kSx] + (double)cB * sum[kSy]);
                o[kGV] = (double)co * ((double)cB * sum[kSx] + (double)cC * sum[kSy]);
                o[kGA] = -0.5 * (double)co * sum[kSxx];
                o[kGB] = -(double)co * sum[kSxy];
                o[kGC] = -0.5 * (double)co * sum[kSyy];
                o[kGO] = sum[kS0];
#pragma unroll
                for (int j = 0; j < 4; ++j) o[kGR + j] = (double)s_w[0][j][pos] + (double)s_w[1][j][pos];
            } else {
#pragma unroll
                for (int j = 0; j < kG2D; ++j) o[j] = 0.0;
            }
            s_pos[pos] = slot_of(grp, id);
        }
        lds_wave_sync();
        for (int i = lane; i < n * kG2D; i += 64) {
            const double v = out[i];
            if (v != 0.0) atomicAdd(a.g2d + (size_t)s_pos[i / kG2D] * kG2D + (i % kG2D), v);
        }
        lds_wave_sync();
    }
    }  // work loop
    // the dense gradient planes, cleared by each workgroup once its walks
    // are done (their stores drain while later workgroups still walk)
    for (int z = 0; z < a.n_zero; ++z) zero_span_grid(a.zero_ptr[z], a.zero_n[z]);
}

// The backward's work list, built by one workgroup of NT threads: for every
// (view, tile) list of L > 0 entries its ceil(L / seg_len_of(L)) <=
// kMaxSegments segments, as (item << 6 | segment) in item order, after their
// count; at most `cap`.
// lists up to which the accumulator clear's first workgroup (256 threads)
// builds the segment list; more get a 1024-thread launch of their own
constexpr int64_t kListInClear = 2048;
template <int NT>
__device__ __forceinline__ void build_segment_list(const uint2 *ranges, int64_t n_items, uint32_t *list,
                                                   uint64_t cap) {
    __shared__ uint32_t s_w[NT / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t per = (n_items + NT - 1) / NT;
    const int64_t t0 = (int64_t)tid * per, t1 = (t0 + per < n_items) ? t0 + per : n_items;
    auto n_seg = [](uint2 r) -> uint32_t {
        const uint32_t L = r.y - r.x;
        return (L + seg_len_of(L) - 1u) / seg_len_of(L);
    };
    uint32_t cnt = 0u;
    for (int64_t t = t0; t < t1; ++t) cnt += n_seg(ranges[t]);
    uint32_t incl = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    uint64_t pos = incl - cnt, total = 0u;
    for (int k = 0; k < NT / 64; ++k) {
        if (k < wave) pos += s_w[k];
        total += s_w[k];
    }
    for (int64_t t = t0; t < t1; ++t) {
        const uint32_t c = n_seg(ranges[t]);
        for (uint32_t q = 0; q < c; ++q, ++pos)
            if (pos < cap) list[1 + pos] = ((uint32_t)t << 6) | q;
    }
    if (tid == 0) list[0] = (uint32_t)(total < cap ? total : cap);
}

// the segment list of a launch with many lists: one 1024-thread workgroup
__global__ void __launch_bounds__(1024) segment_list_kernel(const uint2 *ranges, int64_t n_items, uint32_t *list,
                                                            uint64_t cap) {
    build_segment_list<1024>(ranges, n_items, list, cap);
}

// waves of the segment walk's persistent grid: what the CUs hold at once (12, 16
// and 24 per CU measured within 8 % on 1300 segments)
constexpr int kSegWavesPerCu = 16;
hipError_t launch_backward_tiles(BackwardTileArgs a, int n_cu, hipStream_t s) {
    if (a.n_items == 0) return hipSuccess;
    if (!a.seg_list) {  // one workgroup per quadrant of a list
        const int64_t groups = 4 * kOrderQueues * order_stride(a.n_items);
        a.n_groups = (uint32_t)(groups < (1ll << 30) ? groups : (1ll << 30));
        return launch_kernel(backward_tile_kernel, dim3(a.n_groups), dim3(64), s, a);
    }
    // the work list: built by the accumulator clear for up to kListInClear
    // lists, else here
    if (a.n_items > kListInClear) {
        const hipError_t e = launch_kernel(segment_list_kernel, dim3(1), dim3(1024), s, a.ranges, a.n_items,
                                           a.seg_list, (uint64_t)(a.ckpt_slots * kListPerSlot));
        if (e != hipSuccess) return e;
    }
    a.n_groups = (uint32_t)(kSegWavesPerCu * n_cu);  // persistent
    return launch_kernel(backward_tile_kernel, dim3(a.n_groups), dim3(64), s, a);
}

// ---------------------------------------------------------------------------
// B2: screen-space adjoints -> 3D parameters
// ---------------------------------------------------------------------------
// zeros for floats [w * i0, w * i1) of a plane of w floats per Gaussian,
// by the workgroup: 16-byte stores on the 16-byte aligned stretch, single
// floats at the ends
__device__ __forceinline__ void zero_plane(float *p, int w, int64_t i0, int64_t i1) {
    if (!p) return;
    const int64_t f0 = (int64_t)w * i0, f1 = (int64_t)w * i1;
    const uint64_t base = (uint64_t)(uintptr_t)p;  // 4-byte aligned (floats)
    int64_t v0 = f0, v1 = f1;
    while (((base + 4u * (uint64_t)v0) & 15u) && v0 < f1) ++v0;
    while (((base + 4u * (uint64_t)v1) & 15u) && v1 > v0) --v1;
    if (v0 >= v1) {
        for (int64_t f = f0 + threadIdx.x; f < f1; f += blockDim.x) p[f] = 0.0f;
        return;
    }
    for (int64_t f = f0 + threadIdx.x; f < v0; f += blockDim.x) p[f] = 0.0f;
    for (int64_t f = v1 + threadIdx.x; f < f1; f += blockDim.x) p[f] = 0.0f;
    float4 *q = reinterpret_cast<float4 *>(p + v0);
    for (int64_t k = threadIdx.x; k < (v1 - v0) / 4; k += blockDim.x) q[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

// B2a: with the first chunk of views, zeros for every gradient the chain
// writes, each workgroup's stretch of every plane written with 16-byte stores
// (the drawn Gaussians are overwritten by B2b; later chunks add to what the
// first wrote); the drawn Gaussians appended to a.list, positions inside the
// workgroup from ballots and one atomic per workgroup (order of arrival: each
// Gaussian is handled on its own).  A workgroup takes kListSpan Gaussians, so
// that few atomics meet on the one counter (they serialise there).
__device__ __forceinline__ bool drawn_in(const BackwardProjectArgs &a, int vi, int64_t i) {
    const uint64_t inst = (uint64_t)(a.base[vi] + i);
    return reinterpret_cast<const uint32_t *>(a.slots + (inst >> 6))[(inst >> 5) & 1u] >> (inst & 31u) & 1u;
}
__device__ __forceinline__ const double *row_of(const BackwardProjectArgs &a, int vi, int64_t i) {
    const uint64_t inst = (uint64_t)(a.base[vi] + i);
    return a.g2d + (size_t)slot_of(a.slots[inst >> 6], (uint32_t)inst) * kG2D;
}
constexpr int kListChunks = 4, kListSpan = 1024 * kListChunks;
__global__ void __launch_bounds__(1024) zero_and_list_kernel(const BackwardProjectArgs a, int sh_floats) {
    __shared__ uint32_t s_cnt[kListChunks][16], s_base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t g0 = (int64_t)blockIdx.x * kListSpan, g1 = g0 + kListSpan < a.seg.n ? g0 + kListSpan : a.seg.n;
    // bal[c]: the drawn ones of the wave's 64 Gaussians of chunk c.  Lane v
    // takes view v's (a launch has at most 64): its table words from the first
    // of the 64 on, all loads in one round; a Gaussian is listed if any has it.
    // (As a loop over the views in each lane, 33 + 16 us of a 16-view step; so,
    // 10 + 7 us.)
    uint64_t bal[kListChunks];
    {
        uint2 w0[kListChunks], w1[kListChunks];
        const uint64_t base = (uint64_t)a.base[lane < a.nv ? lane : 0];
#pragma unroll
        for (int c = 0; c < kListChunks; ++c) {
            const uint64_t i0 = (uint64_t)g0 + c * 1024 + 64 * wave, inst = base + i0;
            w0[c] = w1[c] = make_uint2(0u, 0u);
            if (lane < a.nv && i0 < (uint64_t)g1) w0[c] = *reinterpret_cast<const uint2 *>(a.slots + (inst >> 6));
            if (lane < a.nv && (inst >> 6) * 64 + 64 < base + (uint64_t)g1)
                w1[c] = *reinterpret_cast<const uint2 *>(a.slots + (inst >> 6) + 1);
        }
#pragma unroll
        for (int c = 0; c < kListChunks; ++c) {
            const int64_t i0 = g0 + c * 1024 + 64 * wave;
            const uint32_t sh = (uint32_t)(base + (uint64_t)i0) & 63u;
            const uint64_t lo = (uint64_t)w0[c].y << 32 | w0[c].x, hi = (uint64_t)w1[c].y << 32 | w1[c].x;
            uint64_t m = lo >> sh | (sh ? hi << (64u - sh) : 0ull);
            uint32_t x = (uint32_t)m, y = (uint32_t)(m >> 32);
#pragma unroll
            for (int off = 1; off < 64; off <<= 1)
                if (off < a.nv) {
                    x |= (uint32_t)__shfl_xor((int)x, off, 64);
                    y |= (uint32_t)__shfl_xor((int)y, off, 64);
                }
            x = (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
            y = (uint32_t)__builtin_amdgcn_readfirstlane((int)y);
            m = (uint64_t)y << 32 | x;
            const int64_t left = g1 - i0;  // (the words go on with other segments' instances)
            bal[c] = left <= 0 ? 0ull : left < 64 ? m & ((1ull << left) - 1ull) : m;
            if (lane == 0) s_cnt[c][wave] = (uint32_t)__popcll(bal[c]);
        }
    }
    if (a.first && !a.zeroed) {
        const gs_gaussians_grad &G = a.grad;
        zero_plane(G.means, 3, g0, g1);
        zero_plane(G.opacity, 1, g0, g1);
        zero_plane(G.sh, sh_floats, g0, g1);
        if (a.seg.cov6) {
            zero_plane(G.cov6, 6, g0, g1);
        } else {
            zero_plane(G.log_scales, 3, g0, g1);
            zero_plane(G.quats, 4, g0, g1);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0u;
        for (int c = 0; c < kListChunks; ++c)
            for (int w = 0; w < 16; ++w) {
                const uint32_t k = s_cnt[c][w];
                s_cnt[c][w] = total;
                total += k;
            }
        s_base = total ? atomicAdd(a.count, total) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kListChunks; ++c)
        if (bal[c] >> lane & 1ull)
            a.list[s_base + s_cnt[c][wave] + (uint32_t)__popcll(bal[c] & ((1ull << lane) - 1ull))] =
                (uint32_t)(g0 + c * 1024 + threadIdx.x);
}

// B2b: a workgroup of two waves per 64 listed Gaussians.  Wave 0 takes the
// geometry (the FP32 projection repeated for its clamp decisions, then the
// chain in FP64 to the mean and covariance, and the opacity), wave 1 the
// colour (SH coefficients, and the view direction's share of the mean's
// gradient, handed to wave 0 through LDS): two chains of half the length,
// each holding about half the registers.
// Bounded by the latency of the gathered accumulators and, with several views,
// by memory traffic: what counts is the waves in flight (several views: three
// per SIMD, so the rotation and the scales are computed again behind the views'
// loop rather than held over it) and the rounds of dependent loads (one view,
// ONE: no loop, and the accumulators requested with the parameters).  The SH
// gradients leave through LDS, consecutive lanes on consecutive 16-byte pieces
// of a row: stored by each lane for its own row they were 50 M of 64-byte write
// requests for a million Gaussians at degree 3, and bound the kernel.  Measured
// (the 16-view joint step, room of 1 M and 8 x 50 k avatar Gaussians; one view
// of 1280x720; one of 256x256): 490 + 190, 16.0 and 10.7 us before, 321 + 118,
// 13.6 and 7.6 us with all three.  SH rows read through LDS the same way cost
// 33 us (a further round in the chain); four waves per SIMD, with spills, 60.
template <int D, bool ONE>
__global__ void __launch_bounds__(128, ONE ? 2 : 3) backward_project_kernel(const BackwardProjectArgs a) {
    constexpr int K = (D + 1) * (D + 1);
    // SH gradients leave in pieces of 16 bytes (4-byte aligned) where a row is
    // whole pieces, else of 4; the rows' stride in LDS keeps consecutive lanes
    // on different banks
    constexpr int kPiece = 3 * K % 4 == 0 ? 4 : 1, kPieces = 3 * K / kPiece;
    constexpr int kRow = kPiece == 4 ? 4 * (kPieces | 1) : (3 * K) | 1;
    typedef float Piece __attribute__((ext_vector_type(kPiece), aligned(4)));
    __shared__ float s_cam[kProjViews * kCamStride];
    __shared__ double s_dmu[3][64];
    __shared__ float s_dsh[64 * kRow] __attribute__((aligned(16)));
    __shared__ uint32_t s_id[64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nv = ONE ? 1 : a.nv;
    // the count, the listed Gaussian and the cameras in one round of loads
    const int64_t li = (int64_t)blockIdx.x * 64 + lane;
    const uint32_t count = *a.count, listed = a.list[li < a.seg.n ? li : a.seg.n - 1];
    for (int k = threadIdx.x; k < nv * 16; k += 128) {
        const int vi = k >> 4, f = k & 15;
        s_cam[vi * kCamStride + f] = reinterpret_cast<const float *>(a.cams + a.view[vi])[f];
    }
    if ((int64_t)blockIdx.x * 64 >= (int64_t)count) return;  // uniform per workgroup
    __syncthreads();
    for (int vi = threadIdx.x; vi < nv; vi += 128) {
        float *c = s_cam + vi * kCamStride;
#pragma unroll
        for (int j = 0; j < 3; ++j) c[16 + j] = -(c[j] * c[9] + c[3 + j] * c[10] + c[6 + j] * c[11]);
    }
    __syncthreads();
    const bool valid = li < (int64_t)count;
    const int64_t i = valid ? (int64_t)listed : 0;
    const bool use_cov6 = a.seg.cov6 != nullptr;
    const gs_gaussians_grad &G = a.grad;
    const bool first = a.first != 0;
    auto put = [&](float *dst, float v) {
        if (first) *dst = v;
        else *dst += v;
    };
    // FP32 as in the forward where its decisions are repeated (projection,
    // clamps, colour clamp, SH); FP64 along the chain from the conic back to
    // the covariance and the mean, where an elongated Gaussian's adjoints
    // cancel strongly
    float mx = 0.f, my = 0.f, mz = 0.f;
    // the views that draw it, their counts requested together (a listed
    // Gaussian is drawn by one of the launch's views: with one view, by that
    // one); then the drawn views in ascending order
    uint64_t drawn = 0u;
    if (valid) {
        mx = a.seg.means[3 * i + 0];
        my = a.seg.means[3 * i + 1];
        mz = a.seg.means[3 * i + 2];
        drawn = 1u;
        if (!ONE) {
            drawn = 0u;
            for (int v0 = 0; v0 < a.nv; v0 += 16) {
                bool t[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) t[k] = v0 + k < a.nv && drawn_in(a, v0 + k, i);
#pragma unroll
                for (int k = 0; k < 16; ++k) drawn |= (uint64_t)t[k] << (v0 + k);
            }
        }
    }
    // the row of the first view that draws it; inside the loops the next one's
    // is looked up while one is worked on
    auto next_row = [&](uint64_t m) { return row_of(a, m ? __ffsll((unsigned long long)m) - 1 : 0, i); };
    const double *g = next_row(drawn);
    if (wave == 1) {
        // ---- colour -> SH coefficients and view direction
        float dsh[3 * K];
#pragma unroll
        for (int k = 0; k < 3 * K; ++k) dsh[k] = 0.f;
        double dmd[3] = {0.0, 0.0, 0.0};
        float sh[3 * K];
        float dc[3];
        if (ONE && valid) {
            dc[0] = (float)g[kGR];
            dc[1] = (float)g[kGG];
            dc[2] = (float)g[kGBl];
        }
        s_id[lane] = (uint32_t)i;
        const float *src = a.seg.sh + (size_t)(3 * K) * i;
#pragma unroll
        for (int k = 0; k < 3 * K; ++k) sh[k] = src[k];
        for (uint64_t m = drawn; m; m = ONE ? 0u : m & (m - 1u)) {
            const int vi = ONE ? 0 : __ffsll((unsigned long long)m) - 1;
            if (!ONE) {
                dc[0] = (float)g[kGR];
                dc[1] = (float)g[kGG];
                dc[2] = (float)g[kGBl];
                g = next_row(m & (m - 1u));
            }
            const float *cam = s_cam + vi * kCamStride;
            float dx0 = mx - cam[16], dy0 = my - cam[17], dz0 = mz - cam[18];
            const float inv_dist = 1.0f / sqrtf(dx0 * dx0 + dy0 * dy0 + dz0 * dz0);
            const float x = dx0 * inv_dist, y = dy0 * inv_dist, z = dz0 * inv_dist;
            float Y[K];
            float3 dY[K];
            sh_basis<D>(x, y, z, Y);
            sh_basis_grad<D>(x, y, z, dY);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                float acc = 0.0f;  // same accumulation order as the forward
#pragma unroll
                for (int k = 0; k < K; ++k) acc += Y[k] * sh[3 * k + ch];
                if (!(acc + 0.5f > 0.0f)) dc[ch] = 0.0f;
            }
            float ddx = 0.f, ddy = 0.f, ddz = 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float cdot = dc[0] * sh[3 * k] + dc[1] * sh[3 * k + 1] + dc[2] * sh[3 * k + 2];
                ddx += cdot * dY[k].x;
                ddy += cdot * dY[k].y;
                ddz += cdot * dY[k].z;
#pragma unroll
                for (int ch = 0; ch < 3; ++ch) dsh[3 * k + ch] += dc[ch] * Y[k];
            }
            const float dd = x * ddx + y * ddy + z * ddz;
            dmd[0] += (double)((ddx - x * dd) * inv_dist);
            dmd[1] += (double)((ddy - y * dd) * inv_dist);
            dmd[2] += (double)((ddz - z * dd) * inv_dist);
        }
        const int pieces = kPieces * (int)(count - blockIdx.x * 64u < 64u ? count - blockIdx.x * 64u : 64u);
#pragma unroll
        for (int k = 0; k < 3 * K; ++k) s_dsh[lane * kRow + k] = dsh[k];
        lds_wave_sync();
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
            const int e = q * 64 + lane;
            if (e < pieces) {
                const int r = e / kPieces, c = kPiece * (e % kPieces);
                Piece v;
#pragma unroll
                for (int k = 0; k < kPiece; ++k) v[k] = s_dsh[r * kRow + c + k];
                Piece *dst = reinterpret_cast<Piece *>(G.sh + (size_t)(3 * K) * s_id[r] + c);
                if (!first) v += *dst;
                *dst = v;
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) s_dmu[k][lane] = dmd[k];
    }
    double dmu[3] = {0.0, 0.0, 0.0};
    double dS[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // symmetric adjoint of Sigma (xx, xy, xz, yy, yz, zz)
    float dop = 0.f;
    double scd[3] = {0.0, 0.0, 0.0};
    RotT<double> rotd;
    if (wave == 0 && valid) {
        double gl[kG2D];
        if (ONE) {
#pragma unroll
            for (int k = 0; k < kG2D; ++k) gl[k] = g[k];
        }
        float S[6];
        double Sd[6];
        if (use_cov6) {
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                S[k] = a.seg.cov6[6 * i + k];
                Sd[k] = (double)S[k];
            }
        } else {
            const float4 q = reinterpret_cast<const float4 *>(a.seg.quats)[i];
            const Rot rot = quat_rot(q.x, q.y, q.z, q.w);
            float sc[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float ls = a.seg.log_scales[3 * i + k];
                sc[k] = expf(ls);
                scd[k] = exp((double)ls);
            }
            cov_from_rot_scale(rot.R, sc, S);
            rotd = quat_rot_t<double>((double)q.x, (double)q.y, (double)q.z, (double)q.w);
            cov_from_rot_scale(rotd.R, scd, Sd);
        }
        for (uint64_t m = drawn; m; m = ONE ? 0u : m & (m - 1u)) {
            const int vi = ONE ? 0 : __ffsll((unsigned long long)m) - 1;
            if (!ONE) {
#pragma unroll
                for (int k = 0; k < kG2D; ++k) gl[k] = g[k];
                g = next_row(m & (m - 1u));
            }
            const float *cam = s_cam + vi * kCamStride;
            ViewProj p;
            // the same FP32 projection as the forward; the instance is known to
            // be visible (tiles_touched > 0), so every field used below is
            // computed
            const int TX = (a.W + kTile - 1) / kTile, TY = (a.H + kTile - 1) / kTile;
            (void)ewa_project(cam, mx, my, mz, S, a.W, a.H, TX, TY, a.near_plane, a.lowpass, a.sigma_cut, a.fov_clamp,
                              p);
            dop += (float)gl[kGO];
            // ---- the projection in FP64, with the forward's clamp decisions
            double R[9];
    #pragma unroll
            for (int k = 0; k < 9; ++k) R[k] = (double)cam[k];
            const double fxc = (double)cam[12], fyc = (double)cam[13];
            const double tx = R[0] * mx + R[1] * my + R[2] * mz + (double)cam[9];
            const double ty = R[3] * mx + R[4] * my + R[5] * mz + (double)cam[10];
            const double tz = R[6] * mx + R[7] * my + R[8] * mz + (double)cam[11];
            const double iz = 1.0 / tz, iz2 = iz * iz;
            const double limx = (double)a.fov_clamp * (0.5 * (double)a.W / fxc);
            const double limy = (double)a.fov_clamp * (0.5 * (double)a.H / fyc);
            const double xr = p.clx ? (tx * iz < 0.0 ? -limx : limx) : tx * iz;
            const double yr = p.cly ? (ty * iz < 0.0 ? -limy : limy) : ty * iz;
            const double j00 = fxc * iz, j02 = -fxc * xr * iz, j11 = fyc * iz, j12 = -fyc * yr * iz;
            double T0[3], T1[3];
    #pragma unroll
            for (int k = 0; k < 3; ++k) {
                T0[k] = j00 * R[k] + j02 * R[6 + k];
                T1[k] = j11 * R[3 + k] + j12 * R[6 + k];
            }
            double TS0[3], TS1[3];  // T Sigma
            TS0[0] = T0[0] * Sd[0] + T0[1] * Sd[1] + T0[2] * Sd[2];
            TS0[1] = T0[0] * Sd[1] + T0[1] * Sd[3] + T0[2] * Sd[4];
            TS0[2] = T0[0] * Sd[2] + T0[1] * Sd[4] + T0[2] * Sd[5];
            TS1[0] = T1[0] * Sd[0] + T1[1] * Sd[1] + T1[2] * Sd[2];
            TS1[1] = T1[0] * Sd[1] + T1[1] * Sd[3] + T1[2] * Sd[4];
            TS1[2] = T1[0] * Sd[2] + T1[1] * Sd[4] + T1[2] * Sd[5];
            const double lp = (double)a.lowpass;
            const double ca = TS0[0] * T0[0] + TS0[1] * T0[1] + TS0[2] * T0[2] + lp;
            const double cb = TS0[0] * T1[0] + TS0[1] * T1[1] + TS0[2] * T1[2];
            const double cc = TS1[0] * T1[0] + TS1[1] * T1[1] + TS1[2] * T1[2] + lp;
            const double idet = 1.0 / (ca * cc - cb * cb);
            const double qa = cc * idet, qb = -cb * idet, qc = ca * idet;
            // ---- conic -> 2D covariance: dS2 = -Q Gm Q, Gm = [[gA, gB/2], [gB/2, gC]]
            const double ga = gl[kGA], gbh = 0.5 * gl[kGB], gc = gl[kGC];
            const double m00 = qa * ga + qb * gbh, m01 = qa * gbh + qb * gc;
            const double m10 = qb * ga + qc * gbh, m11 = qb * gbh + qc * gc;
            const double s00 = -(m00 * qa + m01 * qb);
            const double s01 = -(m00 * qb + m01 * qc);
            const double s11 = -(m10 * qb + m11 * qc);
            // ---- 2D covariance -> Sigma and T:  S2 = T Sigma T^T + lp I; dSigma += T^T dS2 T
            double U[3][2];
    #pragma unroll
            for (int r = 0; r < 3; ++r) {
                U[r][0] = T0[r] * s00 + T1[r] * s01;
                U[r][1] = T0[r] * s01 + T1[r] * s11;
            }
            dS[0] += U[0][0] * T0[0] + U[0][1] * T1[0];
            dS[1] += U[0][0] * T0[1] + U[0][1] * T1[1];
            dS[2] += U[0][0] * T0[2] + U[0][1] * T1[2];
            dS[3] += U[1][0] * T0[1] + U[1][1] * T1[1];
            dS[4] += U[1][0] * T0[2] + U[1][1] * T1[2];
            dS[5] += U[2][0] * T0[2] + U[2][1] * T1[2];
            // dT = 2 dS2 T Sigma
            double dT0[3], dT1[3];
    #pragma unroll
            for (int c = 0; c < 3; ++c) {
                dT0[c] = 2.0 * (s00 * TS0[c] + s01 * TS1[c]);
                dT1[c] = 2.0 * (s01 * TS0[c] + s11 * TS1[c]);
            }
            // T = J W: dJ = dT W^T;  J00 = fx/z, J02 = -fx xr/z, J11 = fy/z, J12 = -fy yr/z
            const double dJ00 = dT0[0] * R[0] + dT0[1] * R[1] + dT0[2] * R[2];
            const double dJ02 = dT0[0] * R[6] + dT0[1] * R[7] + dT0[2] * R[8];
            const double dJ11 = dT1[0] * R[3] + dT1[1] * R[4] + dT1[2] * R[5];
            const double dJ12 = dT1[0] * R[6] + dT1[1] * R[7] + dT1[2] * R[8];
            double dtx = 0.0, dty = 0.0, dtz = 0.0;
            dtz += -fxc * iz2 * dJ00 - fyc * iz2 * dJ11;
            dtz += dJ02 * fxc * xr * iz2 + dJ12 * fyc * yr * iz2;
            if (!p.clx) {
                dtx += dJ02 * (-fxc * iz) * iz;
                dtz += dJ02 * (-fxc * iz) * (-tx * iz2);
            }
            if (!p.cly) {
                dty += dJ12 * (-fyc * iz) * iz;
                dtz += dJ12 * (-fyc * iz) * (-ty * iz2);
            }
            // ---- projected mean and depth
            dtx += gl[kGU] * fxc * iz;
            dty += gl[kGV] * fyc * iz;
            dtz += -gl[kGU] * fxc * tx * iz2 - gl[kGV] * fyc * ty * iz2 + gl[kGZ];
            dmu[0] += R[0] * dtx + R[3] * dty + R[6] * dtz;
            dmu[1] += R[1] * dtx + R[4] * dty + R[7] * dtz;
            dmu[2] += R[2] * dtx + R[5] * dty + R[8] * dtz;
        }
    }
    __syncthreads();  // the colour wave's share of the mean's gradient is in LDS
    if (wave != 0 || !valid) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) put(&G.means[3 * i + k], (float)(dmu[k] + s_dmu[k][lane]));
    put(&G.opacity[i], dop);
    if (use_cov6) {
        if (G.cov6) {
            // an off-diagonal cov6 entry stands for both symmetric entries
            put(&G.cov6[6 * i + 0], (float)dS[0]);
            put(&G.cov6[6 * i + 1], (float)(2.0 * dS[1]));
            put(&G.cov6[6 * i + 2], (float)(2.0 * dS[2]));
            put(&G.cov6[6 * i + 3], (float)dS[3]);
            put(&G.cov6[6 * i + 4], (float)(2.0 * dS[4]));
            put(&G.cov6[6 * i + 5], (float)dS[5]);
        }
    } else {
        // adjoint of every entry of the full symmetric Sigma
        const double full[9] = {dS[0], dS[1], dS[2], dS[1], dS[3], dS[4], dS[2], dS[4], dS[5]};
        double dls[3], dq[4];
        if (!ONE) {  // not held over the loop of the views: the registers bound the waves in flight
            const float4 q = reinterpret_cast<const float4 *>(a.seg.quats)[i];
#pragma unroll
            for (int k = 0; k < 3; ++k) scd[k] = exp((double)a.seg.log_scales[3 * i + k]);
            rotd = quat_rot_t<double>((double)q.x, (double)q.y, (double)q.z, (double)q.w);
        }
        cov_backward(rotd, scd, full, dls, dq);
        if (G.log_scales) {
#pragma unroll
            for (int k = 0; k < 3; ++k) put(&G.log_scales[3 * i + k], (float)dls[k]);
        }
        if (G.quats) {
#pragma unroll
            for (int k = 0; k < 4; ++k) put(&G.quats[4 * i + k], (float)dq[k]);
        }
    }
}

// The rows of the drawn instances (slot_of), cleared: B1 adds only to those and
// B2 reads only those.  Rows close together: at the instance's own place, a
// fifth of 22 M instances drawn, 208 us; so, 93 us, and B2's gathers 321 + 118
// -> 300 + 112 us.  Workgroup 0 also zeroes the list counters and, with
// checkpoints and at most kListInClear lists, builds the tile pass's segment
// list.
__global__ void __launch_bounds__(256) clear_g2d_kernel(const uint32_t *tt, int64_t n, uint4 *slots, double *g2d,
                                                        uint32_t *counts, int n_counts, const uint2 *ranges,
                                                        int64_t n_items, uint32_t *seg_list, uint64_t seg_cap) {
    static_assert(kG2D % 2 == 0, "two accumulators per 16-B store");
    static_assert(kSlotChunk == 1024, "four groups of 64 instances for each of four waves");
    __shared__ uint32_t s_w[4];
    if (blockIdx.x == 0) {
        for (int k = threadIdx.x; k < n_counts; k += 256) counts[k] = 0u;
        if (seg_list && n_items <= kListInClear) build_segment_list<256>(ranges, n_items, seg_list, seg_cap);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t c0 = (int64_t)blockIdx.x * kSlotChunk; c0 < n; c0 += (int64_t)gridDim.x * kSlotChunk) {
        uint64_t drawn[4];
        uint32_t mine = 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = c0 + 256 * wave + 64 * k + lane;
            drawn[k] = __ballot(i < n && tt[i] != 0u);
            mine += (uint32_t)__popcll(drawn[k]);
        }
        if (lane == 0) s_w[wave] = mine;
        __syncthreads();
        uint32_t row = 0u, total = 0u;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            row += w < wave ? s_w[w] : 0u;
            total += s_w[w];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (lane == k)
                slots[c0 / 64 + 4 * wave + k] = make_uint4((uint32_t)drawn[k], (uint32_t)(drawn[k] >> 32),
                                                           (uint32_t)c0 + row, 0u);
            row += (uint32_t)__popcll(drawn[k]);
        }
        double2 *g = reinterpret_cast<double2 *>(g2d + (size_t)c0 * kG2D);
        for (uint32_t k = threadIdx.x; k < total * (kG2D / 2); k += 256) g[k] = make_double2(0.0, 0.0);
    }
}

hipError_t launch_clear_g2d(const uint32_t *tiles_touched, int64_t n_instances, uint4 *slots, double *g2d,
                            uint32_t *counts, int n_counts, const uint2 *ranges, int64_t n_items, uint32_t *seg_list,
                            uint64_t seg_cap, hipStream_t s) {
    int64_t grid = (n_instances + kSlotChunk - 1) / kSlotChunk;
    if (grid > 1 << 20) grid = 1 << 20;
    if (grid < 1) grid = 1;
    return launch_kernel(clear_g2d_kernel, dim3((unsigned)grid), dim3(256), s, tiles_touched, n_instances, slots, g2d,
                         counts, n_counts, ranges, n_items, seg_list, seg_cap);
}

template <int D>
static hipError_t launch_backward_chain(const BackwardProjectArgs &a, unsigned grid, hipStream_t s) {
    if (a.nv == 1) return launch_kernel(backward_project_kernel<D, true>, dim3(grid), dim3(128), s, a);
    return launch_kernel(backward_project_kernel<D, false>, dim3(grid), dim3(128), s, a);
}

hipError_t launch_backward_project(const BackwardProjectArgs &a, hipStream_t s) {
    if (a.seg.n == 0) return hipSuccess;
    const int K = (a.seg.sh_degree + 1) * (a.seg.sh_degree + 1);
    hipError_t e;
    if ((e = launch_kernel(zero_and_list_kernel, dim3((unsigned)((a.seg.n + kListSpan - 1) / kListSpan)), dim3(1024), s,
                           a, 3 * K)) != hipSuccess)
        return e;
    if (a.nv == 0) return hipSuccess;
    const unsigned grid = (unsigned)((a.seg.n + 63) / 64);  // 64 listed Gaussians per two-wave workgroup
    switch (a.seg.sh_degree) {
        case 0: return launch_backward_chain<0>(a, grid, s);
        case 1: return launch_backward_chain<1>(a, grid, s);
        case 2: return launch_backward_chain<2>(a, grid, s);
        default: return launch_backward_chain<3>(a, grid, s);
    }
}

}  // namespace gs
