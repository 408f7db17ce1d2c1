// Backward of the bf16 path: host orchestration and the memory-bound kernels around the MFMA
// kernels (lifting of the upstream gradients; chain rule through the packing back to the
// inputs).  The paper gives no backward; formulas follow from Eqs. 3-4 and z_ij = z1_i^T z2_j.
//
// Chain: forward pack -> forward attention (leaves O^ and the log-sum-exp in memory, and for a kept step
// of the AlphaFold2 head shape the outputs as well) -> lift the upstream gradients (dO^ = [d_o | R_i d_o_pts
// in the hi and lo columns | z1 (.) d_o_pair], D_i = dO^_i . O^_i) -> dQ^, dK^, dV^ (MFMA kernels) -> unpack.
#include "fipa_gfx950.h"

namespace fipa {

namespace {

// Lanes of a wave that owns a residue: NG of them hold four neighbouring pair columns each (of every 256 where the lifted width
// is larger), the 64 / NG groups take every (64 / NG)-th head.  NG = 64 where r c_z >= 256, else r c_z / 4 or more (at 64 the heads are the
// same for all lanes, and the rows' addresses scalar).
template <class F>
hipError_t with_column_lanes(int DZ, F &&f)  // f(std::integral_constant<int, NG>{})
{
    switch (DZ) {
        case 32: f(std::integral_constant<int, 8>{}); break;
        case 64: f(std::integral_constant<int, 16>{}); break;
        case 128: f(std::integral_constant<int, 32>{}); break;
        default: f(std::integral_constant<int, 64>{}); break;
    }
    return hipGetLastError();
}

__device__ __forceinline__ f32x4 bf16x4_to_f32(uint2 v)
{
    return (f32x4){__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xFFFF0000u)};
}
__device__ __forceinline__ unsigned bf16_pair(float lo, float hi) { return (unsigned)f2bf(lo) | ((unsigned)f2bf(hi) << 16); }

// WPR waves per (batch, residue < Lp; the batch over two grid dimensions, 32768 at most in the first): the lifted upstream gradient
// rows of its heads, D_i, -lse, and the part of the gradient of z1 that comes through o~ = z1^T U, sum_h d_o_pair (.) U: the lifted
// output passes by here once.  That sum, float32, lies in the residue's rows of the outputs d_z1 (upper halves) and d_z2 (lower
// halves) until the unpack kernel writes them.
// The waves of a residue take every WPR-th head (group of heads), NH of them at a time, whose loads are all independent of each
// other and in flight together; the heads' sums meet in LDS in a fixed order.  Bound by memory: 30 KB per residue at H = 12,
// r c_z = 256.
template <int NG, int WPR, int NH>
__global__ __launch_bounds__(256, 4) void fipa_bwd_pack_bf16_kernel(BwdPackParams p)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), sub = WPR == 4 ? wave : 0;
    const int b = blockIdx.y + 32768 * blockIdx.z, i = WPR == 4 ? blockIdx.x : 4 * blockIdx.x + wave;
    if (b >= p.B) return;
    if (i >= ((p.kvlen[b] + 31) & ~31)) return;  // (the gradient kernels stream whole blocks of 32 rows and no further)
    const int c = p.c, D = kDH + p.DZ, PH = (p.Pv + 1) / 2;
    constexpr int HG = 64 / NG;
    const int grp = lane % NG, hg = sub * HG + (HG == 1 ? 0 : lane / NG);
    const bool inside = i < user_len(p, b);
    const size_t urow = inside ? user_row(p, b, i) : 0;
    const bool valid = inside && (p.mask ? p.mask[urow] != 0 : true);
    const size_t row0 = (size_t)b * p.H * p.Lp + i;  // (row of head h: h Lp further)
    if (!valid) {  // zeros; nothing reads the sum of such a residue
        for (int h = hg; h < p.H; h += WPR * HG) {
            bf16_t *dst = p.dOhat + (row0 + (size_t)h * p.Lp) * D;
            for (int x = 4 * grp; x < D; x += 4 * NG) *reinterpret_cast<uint2 *>(dst + x) = (uint2){0u, 0u};
            if (grp == 0) {
                p.Dvec[row0 + (size_t)h * p.Lp] = 0.f;
                p.nlse[row0 + (size_t)h * p.Lp] = -INFINITY;
            }
        }
        return;
    }
    float R[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) R[a] = p.rot[urow * 9 + a];
    f32x4 s1[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    for (int h0 = hg; h0 < p.H; h0 += WPR * NH * HG) {
        float dsum[NH];
        bool on[NH];
        size_t row[NH], rec[NH];
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            const int h = h0 + u * WPR * HG;
            on[u] = h < p.H;
            row[u] = row0 + (size_t)(on[u] ? h : h0) * p.Lp;
            rec[u] = urow * p.H + (on[u] ? h : h0);
            dsum[u] = 0.f;
        }
        // ---- pair part: columns kDH + x .. + 3
#pragma unroll
        for (int set = 0; set < 2; ++set) {  // (r c_z <= 512)
            const int x = 4 * grp + 256 * set;
            if (x >= p.DZ) break;
            const f32x4 z = bf16x4_to_f32(*reinterpret_cast<const uint2 *>(p.z1 + urow * p.DZ + x));
            f32x4 g4[NH], o4[NH];
#pragma unroll
            for (int u = 0; u < NH; ++u) {
                g4[u] = *reinterpret_cast<const f32x4 *>(p.d_o_pair + rec[u] * p.cz + x % p.cz);  // (cz is a multiple of 8)
                o4[u] = *reinterpret_cast<const f32x4 *>(p.Ohat + row[u] * D + kDH + x);
            }
#pragma unroll
            for (int u = 0; u < NH; ++u) {
                bf16_t bv[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    bv[e] = f2bf(z[e] * g4[u][e]);
                    dsum[u] += bf2f(bv[e]) * o4[u][e];  // D uses the rounded gradient the MFMAs will see
                    s1[set][e] += on[u] ? g4[u][e] * o4[u][e] : 0.f;
                }
                if (on[u])
                    *reinterpret_cast<uint2 *>(p.dOhat + row[u] * D + kDH + x) =
                        (uint2){(unsigned)bv[0] | ((unsigned)bv[1] << 16), (unsigned)bv[2] | ((unsigned)bv[3] << 16)};
            }
        }
        // ---- head-specific part: columns grp, grp + NG, ..
        for (int col = grp; col < kDH; col += NG) {
            // inverse of v_pt_col: which (point, axis) lives in this column, if any
            const int cp = col - c, within = cp & 7;
            const int gh = within >> 2, u1 = 4 * (cp >> 3) + (within & 3);
            const int lo = u1 / (3 * PH), u2 = u1 - lo * 3 * PH;
            const int pt = gh * PH + u2 / 3, ax = u2 % 3;
            const bool scalar = col < c, point = !scalar && lo < 2 && pt < p.Pv;
            const float r0 = ax == 0 ? R[0] : (ax == 1 ? R[3] : R[6]), r1 = ax == 0 ? R[1] : (ax == 1 ? R[4] : R[7]),
                        r2 = ax == 0 ? R[2] : (ax == 1 ? R[5] : R[8]);
            float o[NH], g[NH][3];
#pragma unroll
            for (int u = 0; u < NH; ++u) {
                // (a scalar column takes its one number three times, a column without either the first of d_o)
                const float *src = point ? p.d_o_pts + (rec[u] * p.Pv + pt) * 3 : p.d_o + rec[u] * c + (scalar ? col : 0);
                const int st = point ? 1 : 0;
                o[u] = p.Ohat[row[u] * D + col];
#pragma unroll
                for (int a = 0; a < 3; ++a) g[u][a] = src[a * st];
            }
#pragma unroll
            for (int u = 0; u < NH; ++u) {
                const float val = scalar ? g[u][0] : (point ? r0 * g[u][0] + r1 * g[u][1] + r2 * g[u][2] : 0.f);  // dG = R_i d_o_pts
                const bf16_t bv = f2bf(val);
                if (on[u]) p.dOhat[row[u] * D + col] = bv;
                dsum[u] += bf2f(bv) * o[u];
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
            if (o < NG)
#pragma unroll
                for (int u = 0; u < NH; ++u) dsum[u] += __shfl_xor(dsum[u], o);
#pragma unroll
        for (int u = 0; u < NH; ++u)
            if (on[u] && grp == 0) {
                const float l2 = p.lse2[row[u]];
                p.Dvec[row[u]] = p.neg_d ? -dsum[u] : dsum[u];
                p.nlse[row[u]] = l2 > -INFINITY && l2 < INFINITY ? -l2 : -INFINITY;
            }
    }
#pragma unroll
    for (int set = 0; set < 2; ++set)
        for (int o = NG; o < 64; o <<= 1)  // (the head groups of a wave, added pairwise in a fixed order)
#pragma unroll
            for (int e = 0; e < 4; ++e) s1[set][e] += __shfl_xor(s1[set][e], o);
    auto leave = [&](int x, const f32x4 &sum) {
        if (lane >= NG || x >= p.DZ) return;
        unsigned w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = __float_as_uint(sum[e]);
        *reinterpret_cast<uint2 *>(p.d_z1 + urow * p.DZ + x) = (uint2){(w[0] >> 16) | (w[1] & 0xFFFF0000u), (w[2] >> 16) | (w[3] & 0xFFFF0000u)};
        *reinterpret_cast<uint2 *>(p.d_z2 + urow * p.DZ + x) = (uint2){(w[0] & 0xFFFFu) | (w[1] << 16), (w[2] & 0xFFFFu) | (w[3] << 16)};
    };
    if constexpr (WPR == 1) {
        leave(4 * lane, s1[0]);
        leave(4 * lane + 256, s1[1]);
    } else {
        __shared__ f32x4 part[4][2][64];
        part[wave][0][lane] = s1[0];
        part[wave][1][lane] = s1[1];
        __syncthreads();
        if (wave < 2) leave(4 * lane + 256 * wave, ((part[0][wave][lane] + part[1][wave][lane]) + part[2][wave][lane]) + part[3][wave][lane]);
    }
}

// Two waves per (batch, residue): chain rule from dQ^, dK^, dV^ back to the inputs.  Nothing is exchanged between the waves, so
// there is no workgroup barrier: sums over the lanes of a wave go through shuffles in a fixed order.
//   one takes the per-head tasks -- 2 Pq + Pv point gradients and the three scalar rows of each head --
//   dealt to the lanes kind by kind (few bytes, many small scattered accesses);
//   the other (`pair`) the pair factors (the bulk of the bytes): a lane owns four neighbouring lifted columns and
//   adds up the heads one after the other (16-byte loads of the four big arrays, all independent);
//   where the lifted width is below 256 the lanes form 64 / (DZ / 4) groups that take every
//   group-th head and are added at the end, above it a lane takes DZ / 256 sets of columns.
// A residue that does not count reads nothing and writes zeros.
// One workgroup per residue with the sums of its threads meeting in LDS behind workgroup barriers was slower (191 us against 139).
template <int NG>
__device__ __forceinline__ void unpack_residue(const BwdUnpackParams &p, unsigned residue, bool pair)
{
    const int lane = threadIdx.x & 63;
    if (residue >= (unsigned)p.B * p.L) return;
    const int rr = (int)residue, b = rr / p.L, i = rr - b * p.L;  // (b, i)
    const int c = p.c, Pq = p.Pq, Pv = p.Pv, nq = 3 * Pq, D = kDH + p.DZ;
    if (i >= user_len(p, b)) return;  // (packed batch: the grid covers the longest chain)
    const size_t urow = user_row(p, b, i);
    const bool valid = p.mask ? p.mask[urow] != 0 : true;
    if (!valid) {  // (nothing was formed for it)
        if (pair) return;
        const int nc = p.H * c / 8, nk = p.H * Pq * 3, nv = p.H * Pv * 3;
        for (int x = lane; x < nc; x += 64) {
            const uint4 zero = {0u, 0u, 0u, 0u};
            *reinterpret_cast<uint4 *>(p.d_q + urow * p.H * c + 8 * x) = zero;
            *reinterpret_cast<uint4 *>(p.d_k + urow * p.H * c + 8 * x) = zero;
            *reinterpret_cast<uint4 *>(p.d_v + urow * p.H * c + 8 * x) = zero;
        }
        for (int x = lane; x < nk; x += 64) p.d_q_pts[urow * nk + x] = p.d_k_pts[urow * nk + x] = 0;
        for (int x = lane; x < nv; x += 64) p.d_v_pts[urow * nv + x] = 0;
        for (int x = 4 * lane; x < p.DZ; x += 256) {
            *reinterpret_cast<uint2 *>(p.d_z1 + urow * p.DZ + x) = (uint2){0u, 0u};
            *reinterpret_cast<uint2 *>(p.d_z2 + urow * p.DZ + x) = (uint2){0u, 0u};
        }
        for (int h = lane; h < p.H; h += 64) p.gpart[((size_t)b * p.H + h) * p.Lp + i] = 0.f;
        if (p.d_rot) {
            if (lane < 3) p.d_trans[urow * 3 + lane] = 0.f;
            if (lane < 9) p.d_rot[urow * 9 + lane] = 0.f;
        }
        return;
    }

    if (pair) {  // ---- pair factors: sums over heads
        constexpr int HG = 64 / NG;
        const int grp = lane % NG, hg = HG == 1 ? 0 : lane / NG;
        for (int x0 = 4 * grp; x0 < p.DZ; x0 += 256) {
            const int d0 = x0 % p.cz;
            f32x4 s1 = {0.f, 0.f, 0.f, 0.f}, s2 = {0.f, 0.f, 0.f, 0.f};
            const float kscale = p.dVz ? kLn2 : 1.f, qscale = p.w_L * p.ds_inv;
            // through o~ = z1^T U (see the pack kernel)
            const uint2 up = *reinterpret_cast<const uint2 *>(p.d_z1 + urow * p.DZ + x0), low = *reinterpret_cast<const uint2 *>(p.d_z2 + urow * p.DZ + x0);
#pragma unroll 4
            for (int h = hg; h < p.H; h += HG) {
                const size_t bh = (size_t)b * p.H + h;
                const size_t row = (bh * p.Lp + i) * D + kDH + x0;
                const f32x4 dq = *reinterpret_cast<const f32x4 *>(p.dQhat + row);
                const size_t zrow = (bh * p.Lp + i) * p.z_pitch + x0;
                const f32x4 dk = *reinterpret_cast<const f32x4 *>(p.dKz + zrow);
                f32x4 dv = {0.f, 0.f, 0.f, 0.f};
                if (p.dVz) dv = *reinterpret_cast<const f32x4 *>(p.dVz + zrow);
                const f32x4 wb = *reinterpret_cast<const f32x4 *>(p.w_b + (size_t)h * p.cz + d0);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s1[e] += qscale * wb[e] * dq[e];   // z1: through the bias vector b^{h1} = w_L w_b z1
                    s2[e] += kscale * dk[e] + dv[e];   // z2: as key feature (the log2e sits on the query side) and as value feature
                }
            }
            for (int o = NG; o < 64; o <<= 1)  // (HG > 1: the head groups, added pairwise in a fixed order)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s1[e] += __shfl_xor(s1[e], o);
                    s2[e] += __shfl_xor(s2[e], o);
                }
            if (hg == 0) {
                s1[0] += __uint_as_float((up.x << 16) | (low.x & 0xFFFFu));
                s1[1] += __uint_as_float((up.x & 0xFFFF0000u) | (low.x >> 16));
                s1[2] += __uint_as_float((up.y << 16) | (low.y & 0xFFFFu));
                s1[3] += __uint_as_float((up.y & 0xFFFF0000u) | (low.y >> 16));
                *reinterpret_cast<uint2 *>(p.d_z1 + urow * p.DZ + x0) = (uint2){bf16_pair(s1[0], s1[1]), bf16_pair(s1[2], s1[3])};
                *reinterpret_cast<uint2 *>(p.d_z2 + urow * p.DZ + x0) = (uint2){bf16_pair(s2[0], s2[1]), bf16_pair(s2[2], s2[3])};
            }
        }
        return;
    }

    // ---- per-head tasks ----------------------------------------------------------------------------
    const float *R = p.rot + urow * 9;
    const float *t = p.trans + urow * 3;
    float Rm[9], tc[3];
    for (int a = 0; a < 9; ++a) Rm[a] = R[a];
    for (int a = 0; a < 3; ++a) tc[a] = t[a] - p.cen[4 * b + a];

    // frame gradients: every global-frame point gradient g of a point with local coordinates x
    // contributes g to d t_i and g x^T to d R_i (G = R_i x + t_i); the output points
    // o_pts = R_i^T (G - t_i) contribute -R_i d_o_pts and (G - t_i) d_o_pts^T
    float ft[3] = {0.f, 0.f, 0.f}, fr[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // Three kinds of task, each dealt to the lanes in passes of its own so that a pass runs one
    // piece of code: the 2 Pq query and key points of a head (whole heads per pass: their
    // contributions to d gamma are added across the head's lanes), the Pv value points, and the
    // scalar rows d_q, d_k, d_v in pieces of eight channels.
    {
        const int per = 2 * Pq, HP = 64 / per;
        for (int h0 = 0; h0 < p.H; h0 += HP) {
            float gpartial = 0.f;
            const int hl = lane / per;
            const bool active = hl < HP && h0 + hl < p.H;
            const int h = active ? h0 + hl : 0, tk = active ? lane - hl * per : 0;
            const size_t bh = (size_t)b * p.H + h;
            if (active) {
                const size_t rec = urow * p.H + h;
                const float pscale = p.gamma[h] * p.w_L * p.w_C;
                const bool isq = tk < Pq;
                const float sc = isq ? 1.f : kLog2e * pscale, inv_sc = sc != 0.f ? 1.f / sc : 0.f;
                const int pt = isq ? tk : tk - Pq;
                const float *dX = (isq ? p.dQhat + (bh * p.Lp + i) * D : p.dKh + (bh * p.Lp + i) * p.h_pitch) + c + 3 * pt;  // hi columns of this point
                const int lo_off = isq ? nq : 2 * nq;                                             // to its lo columns
                const float ws = p.ds_inv * (isq ? p.rowsum : p.colsum)[bh * p.Lp + i];
                const bf16_t *src = (isq ? p.q_pts : p.k_pts) + (rec * Pq + pt) * 3;
                const float lc[3] = {bf2f(src[0]), bf2f(src[1]), bf2f(src[2])};
                float grad[3];
                float gacc = 0.f;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float G0 = Rm[3 * a] * lc[0] + Rm[3 * a + 1] * lc[1] + Rm[3 * a + 2] * lc[2] + tc[a];
                    const float X = p.ds_inv * (dX[a] + dX[lo_off + a]);  // sum over the other side of dS times its hi and lo coordinates
                    // the effective (hi + lo) global coordinate the kernels used: the query's as it is, the
                    // key's scaled by log2e gamma w_L w_C before the split
                    const float Gs = sc * G0;
                    const bf16_t hi = f2bf(Gs), lo = f2bf(Gs - bf2f(hi));
                    const float eff = sc != 0.f ? (bf2f(hi) + bf2f(lo)) * inv_sc : G0;
                    // query: d s / dQ = gamma w_L w_C (K - Q) summed with dS, and sum_j dS K^ sits in the Khi and
                    // Klo columns (in log2 units); key: the same with the sides exchanged
                    grad[a] = isq ? kLn2 * X - pscale * ws * eff : pscale * (X - ws * eff);
                    gacc += isq ? ws * eff * eff : ws * eff * eff - 2.f * eff * X;
                }
                gpartial = gacc;
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    ft[x] += grad[x];
#pragma unroll
                    for (int y = 0; y < 3; ++y) fr[3 * x + y] += grad[x] * lc[y];
                }
                bf16_t *dst = (isq ? p.d_q_pts : p.d_k_pts) + (rec * Pq + pt) * 3;
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    const float val = Rm[x] * grad[0] + Rm[3 + x] * grad[1] + Rm[6 + x] * grad[2];  // R^T
                    dst[x] = f2bf(valid ? val : 0.f);
                }
            }
            // d gamma: this residue's contribution, summed over the query and key points of a head in
            // a fixed order (they sit in the 2 Pq lanes from the head's first on)
            float gsum = 0.f;
            for (int x = 0; x < per; ++x) gsum += __shfl(gpartial, (lane + x) & 63);
            if (active && tk == 0) p.gpart[bh * p.Lp + i] = valid ? gsum : 0.f;
        }
    }
    for (int t0 = 0; t0 < p.H * Pv; t0 += 64) {
        const int tsk = t0 + lane;
        if (tsk < p.H * Pv) {
            const int h = tsk / Pv, pt = tsk - h * Pv;
            const size_t bh = (size_t)b * p.H + h;
            const size_t rec = urow * p.H + h;
            const float *dV = p.dVh + (bh * p.Lp + i) * p.h_pitch;
            float grad[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) grad[a] = dV[v_pt_col(c, Pv, pt, a, 0)];
            if (p.d_rot) {
                const bf16_t *vl = p.v_pts + (rec * Pv + pt) * 3;
                const float *gp = p.d_o_pts + (rec * Pv + pt) * 3;
                const float *oh = p.Ohat + (bh * p.Lp + i) * D;
                const bf16_t *dgh = p.dOhat + (bh * p.Lp + i) * D;
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    // R_i d_o_pts, in the rounded form that the gradient kernels used: it then cancels
                    // against the value-point term exactly where the mathematics says so (shift invariance)
                    const float dGx = bf2f(dgh[v_pt_col(c, Pv, pt, x, 0)]);
                    const float Gm = oh[v_pt_col(c, Pv, pt, x, 0)] + oh[v_pt_col(c, Pv, pt, x, 1)] - tc[x];
                    ft[x] += grad[x] - dGx;
#pragma unroll
                    for (int y = 0; y < 3; ++y) fr[3 * x + y] += grad[x] * bf2f(vl[y]) + Gm * gp[y];
                }
            }
            bf16_t *dst = p.d_v_pts + (rec * Pv + pt) * 3;
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                const float val = Rm[x] * grad[0] + Rm[3 + x] * grad[1] + Rm[6 + x] * grad[2];
                dst[x] = f2bf(valid ? val : 0.f);
            }
        }
    }
    {
        const int nchunk = c / 8, per = 3 * nchunk;  // (c is a multiple of 8; every piece is 16-byte aligned on both sides)
        for (int t0 = 0; t0 < p.H * per; t0 += 64) {
            const int tsk = t0 + lane;
            if (tsk < p.H * per) {
                const int h = tsk / per, rem = tsk - h * per;
                const int which = rem / nchunk, x = 8 * (rem - which * nchunk);  // 0: d_q, 1: d_k, 2: d_v
                const size_t row = ((size_t)b * p.H + h) * p.Lp + i;
                const float *src = (which == 0 ? p.dQhat + row * D : (which == 1 ? p.dKh : p.dVh) + row * p.h_pitch) + x;
                const float scale = which == 0 ? kLn2 * p.ds_inv : (which == 1 ? p.w_L * p.qk_scale * p.ds_inv : 1.f);
                bf16_t *dst = (which == 0 ? p.d_q : (which == 1 ? p.d_k : p.d_v)) + (urow * p.H + h) * c + x;
                const f32x4 v0 = *reinterpret_cast<const f32x4 *>(src);
                const f32x4 v1 = *reinterpret_cast<const f32x4 *>(src + 4);
                uint4 o;
                o.x = (unsigned)f2bf(valid ? scale * v0[0] : 0.f) | ((unsigned)f2bf(valid ? scale * v0[1] : 0.f) << 16);
                o.y = (unsigned)f2bf(valid ? scale * v0[2] : 0.f) | ((unsigned)f2bf(valid ? scale * v0[3] : 0.f) << 16);
                o.z = (unsigned)f2bf(valid ? scale * v1[0] : 0.f) | ((unsigned)f2bf(valid ? scale * v1[1] : 0.f) << 16);
                o.w = (unsigned)f2bf(valid ? scale * v1[2] : 0.f) | ((unsigned)f2bf(valid ? scale * v1[3] : 0.f) << 16);
                *reinterpret_cast<uint4 *>(dst) = o;
            }
        }
    }

    // frame gradients of this residue: sum over the lanes in a fixed order
    if (p.d_rot) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
            for (int x = 0; x < 3; ++x) ft[x] += __shfl_xor(ft[x], o);
#pragma unroll
            for (int x = 0; x < 9; ++x) fr[x] += __shfl_xor(fr[x], o);
        }
        if (lane < 3) p.d_trans[urow * 3 + lane] = valid ? (lane == 0 ? ft[0] : (lane == 1 ? ft[1] : ft[2])) : 0.f;
        if (lane < 9) {
            float v = fr[0];
#pragma unroll
            for (int x = 1; x < 9; ++x) v = lane == x ? fr[x] : v;
            p.d_rot[urow * 9 + lane] = valid ? v : 0.f;
        }
    }
}

// d gamma^h = -(w_L w_C / 2) * sum over (batch, residue) of the partial sums, in a fixed order:
// one workgroup of 1024 threads per head, four independent chains of loads per thread.
// (cu: row offsets of a packed batch, whose chain b has cu[b+1] - cu[b] residues, or null.)
__device__ __forceinline__ void gamma_sum(const float *gpart, float *d_gamma, int B, int H, int L, int Lp, const int *cu, float coef)
{
    __shared__ float red[1024];
    const int h = blockIdx.x, tid = threadIdx.x;
    float s4[4] = {0.f, 0.f, 0.f, 0.f};
    if (B >= 16) {  // many chains: a wave each (one after the other they are a chain of B dependent loads: 16 us at B = 32)
        for (int b = tid >> 6; b < B; b += 16) {
            const int len = cu ? cu[b + 1] - cu[b] : L;
            const float *g = gpart + ((size_t)b * H + h) * Lp;
            for (int i0 = tid & 63; i0 < len; i0 += 256)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + 64 * u;
                    s4[u] += i < len ? g[i] : 0.f;
                }
        }
    } else for (int b = 0; b < B; ++b) {
        const int len = cu ? cu[b + 1] - cu[b] : L;
        const float *g = gpart + ((size_t)b * H + h) * Lp;
        for (int i0 = tid; i0 < len; i0 += 4096)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + 1024 * u;
                s4[u] += i < len ? g[i] : 0.f;
            }
    }
    red[tid] = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    __syncthreads();
    for (int st = 512; st > 0; st >>= 1) {
        if (tid < st) red[tid] += red[tid + st];
        __syncthreads();
    }
    if (tid == 0) d_gamma[h] = coef * red[0];
}

// d w_b[h, d] = w_L * sum over (batch, residue, rho) of z1[b,i,rho,d] * dQ^[b,h,i, 64 + rho*cz + d]
// (b^{h1} = w_L w_b (.) z1, Algorithm 1 step 2 with Eq. 3's w_L).  Two passes with a fixed
// summation order: per (head, chunk of 32 residues) partial sums per lifted column, then the
// sum over chunks and rho.
constexpr int kWbChunk = 32;

// One workgroup per (chunk, NH heads): a thread takes four neighbouring lifted columns (16 bytes of
// dQ^ per head, 8 of z1) of every NRG-th residue of the chunk, all loads independent; the NRG partial sums
// per column meet in LDS and are added in a fixed order.  r c_z <= 512 here, so NRG >= 2.  Bound by reading dQ^; in a launch of its own 32 packed
// chains of 64 to 512 residues, H = 12, r c_z = 256 22.9 us for 111 MB, four chains of 2.7k to 7.1k residues at r c_z = 512 121 for
// 484 MB (a workgroup per head, which finds every residue's place and reads z1 again: 30 and 138).
template <int NH>
__device__ __forceinline__ void wb_partial(const BwdUnpackParams &p, int chunk, int h0, int nchunk)
{
    __shared__ f32x4 red[NH][256];  // [head][residue group][DZ]: NRG * DZ = 1024 numbers per head
    const int D = kDH + p.DZ;
    const int nres = p.total_rows;  // rows of the caller's tensors: B L, or the packed batch's total
    const int NG = p.DZ / 4, NRG = 256 / NG;
    const int cg = threadIdx.x % NG, rg = threadIdx.x / NG, x0 = 4 * cg;
    f32x4 s[NH];
#pragma unroll
    for (int u = 0; u < NH; ++u) s[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
    int b0 = 0;  // packed batch: the chain that holds the chunk's first row, the last b with cu[b] <= it
    if (p.cu) {
        int hi = p.B - 1;
        while (b0 < hi) {
            const int mid = (b0 + hi + 1) >> 1;
            if (p.cu[mid] <= chunk * kWbChunk) b0 = mid; else hi = mid - 1;
        }
    }
#pragma unroll 4
    for (int t = rg; t < kWbChunk; t += NRG) {
        const int bi = min(chunk * kWbChunk + t, nres - 1);
        int b, i;
        if (p.cu) {
            b = b0;
            while (b + 1 < p.B && p.cu[b + 1] <= bi) ++b;
            i = bi - p.cu[b];
        } else {
            b = bi / p.L;
            i = bi - b * p.L;
        }
        const bool valid = chunk * kWbChunk + t < nres && (p.mask ? p.mask[bi] != 0 : true);
        // (a residue that does not count takes the first row of all, so that the loads need no branch and padding costs no traffic)
        const uint2 zr = *reinterpret_cast<const uint2 *>(p.z1 + (valid ? (size_t)bi * p.DZ : 0) + x0);
        const f32x4 z = bf16x4_to_f32(zr);
        f32x4 dq[NH];
#pragma unroll
        for (int u = 0; u < NH; ++u) {
            const int h = min(h0 + u, p.H - 1);
            dq[u] = *reinterpret_cast<const f32x4 *>(p.dQhat + (valid ? (((size_t)b * p.H + h) * p.Lp + i) * D : 0) + kDH + x0);
        }
        if (valid)
#pragma unroll
            for (int u = 0; u < NH; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[u][e] += z[e] * dq[u][e];
    }
#pragma unroll
    for (int u = 0; u < NH; ++u) red[u][threadIdx.x] = s[u];
    __syncthreads();
    for (int x = threadIdx.x; x < NH * NG; x += 256) {
        const int u = x / NG, col = x - u * NG;
        if (h0 + u >= p.H) break;
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
        for (int g = 0; g < NRG; ++g) t += red[u][g * NG + col];
        *reinterpret_cast<f32x4 *>(p.wpart + ((size_t)(h0 + u) * nchunk + chunk) * p.DZ + 4 * col) = t;
    }
}

// For every 32 residues 16 workgroups of four waves (two residues each), then the workgroups that form the partial sums of d_w_b over 32
// rows, which read the same dQ^ at about the same time.  With the sums kernel behind it, us (a wave per residue that took its heads
// first and then its pair factors, the partial sums and the two last sums in launches of their own | this): 32 packed chains of 64 to 512
// residues, r c_z = 256 136 | 121, B = 2, L = 4096 108 | 94, B = 2, L = 2048 60 | 60, four chains of 2.7k to 7.1k residues, r c_z = 512 455 | 374.
// Of the first one's 114 us the pair factors take 46 (5.0 TB/s), the heads 61 and the partial sums 14 where they run alone.
template <int NG, int NH>
__global__ __launch_bounds__(256) void fipa_bwd_unpack_bf16_kernel(BwdUnpackParams p, int nchunk)
{
    const unsigned group = blockIdx.y + 32768 * blockIdx.z, y = blockIdx.x;
    if (y < 16) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        unpack_residue<NG>(p, 32u * group + 2 * y + (wave >> 1), (wave & 1) != 0);
    } else if (group < (unsigned)nchunk) {
        wb_partial<NH>(p, group, (y - 16) * NH, nchunk);
    }
}


// One workgroup of 1024 threads per head and 32 (where c_z is no multiple of 32: 8) of its c_z columns, of every factor slice: the
// chunks are dealt to the groups of threads that hold those columns (four independent chains of loads each); groups and
// slices are added in a fixed order.  (One workgroup per head: 82 us for 12 heads of 1024 chunks of 512 columns -> 25 us.)
__host__ __device__ inline int wb_columns(int cz) { return cz % 32 == 0 ? 32 : 8; }

__device__ __forceinline__ void wb_reduce(const BwdUnpackParams &p, int block, int nchunk)
{
    __shared__ float part[1024];  // [chunk group][slice][column]
    const int h = blockIdx.x, CB = wb_columns(p.cz), d0 = block * CB;
    const int NCOL = CB * p.r, NCG = 1024 / NCOL;  // (r c_z <= 512 here)
    const int cidx = threadIdx.x % NCOL, grp = threadIdx.x / NCOL;
    if (grp < NCG) {
        const int x = cidx / CB * p.cz + d0 + cidx % CB;
        float s4[4] = {0.f, 0.f, 0.f, 0.f};
        for (int ch0 = grp; ch0 < nchunk; ch0 += 4 * NCG)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ch = ch0 + u * NCG;
                const float v = p.wpart[((size_t)h * nchunk + min(ch, nchunk - 1)) * p.DZ + x];
                s4[u] += ch < nchunk ? v : 0.f;
            }
        part[grp * NCOL + cidx] = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    }
    __syncthreads();
    if (threadIdx.x < CB) {
        float t = 0.f;
        for (int rho = 0; rho < p.r; ++rho)
            for (int g = 0; g < NCG; ++g) t += part[g * NCOL + rho * CB + threadIdx.x];
        p.d_w_b[(size_t)h * p.cz + d0 + threadIdx.x] = p.w_L * p.ds_inv * t;
    }
}

// The two of them in one launch (5 us each, most of it start-up): a head's d gamma first, then its column blocks of d_w_b.
__global__ __launch_bounds__(1024) void fipa_bwd_sums_kernel(BwdUnpackParams p, int nchunk)
{
    if (blockIdx.y == 0) gamma_sum(p.gpart, p.d_gamma, p.B, p.H, p.L, p.Lp, p.cu, -0.5f * p.w_L * p.w_C);
    else wb_reduce(p, blockIdx.y - 1, nchunk);
}

// The lifted widths whose gradients go through stored weights (fipa_bf16_bwd_keys.hip, fipa_bf16_bwd_stored.hip), at any length (width 128:
// where the workspace holds enough of them, see stored_pays).  Kept
// training step, forming the weights in every product / stored, us: r c_z = 128, H = 12: one chain of 300 residues 111 / 98, four
// of up to 1000 306 / 255, 32 packed ones of 64 to 512 805 / 650, B = 2, L = 4096 1643 / 1298; r c_z = 256: one chain
// of 64 residues 103 / 90, 131 120 / 109, 256 138 / 125, 512 174 / 159, 1024 258 / 210, 16 chains of 130 310 / 226; H = 4, one of 64 93 / 82;
// r c_z = 512, H = 12: one chain of 64 130 / 101, 131 163 / 130, 512 262 / 194, 1024 582 / 257.
bool bwd_stored(int DZ) { return bwd_keys_fused(DZ) || DZ == 512; }

// Width 128 with the weights of nq query rows in memory against forming them in every product (the width for which both are there).
// Every range starts its kernels anew, and its query side runs on BH nq / 256 workgroups.  Kept training step, us, H = 12, formed | stored
// by rows: B = 2, L = 4096 1595 | 256 3001, 512 2021, 1024 1581, 2048 1304, all 1243; one chain of 1000 188 | 256 285, 512 201, all 158; of 2048
// 306 | 512 433, 1024 311, all 251; of 8192 2820 | 1024 3443, 2048 2630, 4096 2269; 2 x 1000 208 | 512 220; 4 x 1000 378 | 256 459, 512 358;
// 8 x 1024 639 | 256 725, 512 580; 8 x 700, H = 8, 324 | 256 357, 512 311; 2 x 2048, H = 8, 330 | 512 451, 1024 328; one chain of 16384, H = 4,
// 3594 | 2048 4823, 4096 3584; with one head (in the workspace of the query) of 12000 1268 | 8192 1252, of 24000 2545 | 8192 2879, of 32768
// 3558 | 8192 4599.
bool stored_pays(int DZ, size_t BH, int Lp, int nq)
{
    if (DZ != 128 || nq >= Lp) return true;
    if (nq == 0) return false;
    const size_t ranges = (Lp + nq - 1) / nq, tiles = BH * ((nq + 255) / 256);
    return ranges * (nq < 2048 ? 32 : nq < 4096 ? 24 : 16) <= tiles;
}

// Bytes of stored weights (P and dS', 4 per query row, key and pair) that the workspace query asks for: of 4096 query rows --
// every range of rows but the first adds its key-side sums to memory: 2048 / 4096 / 8192 rows measured 14.4 / 13.8 / 13.6 ms per
// training step on four chains of up to 8192 residues (r c_z = 512), 2.24 / 2.15 / 2.15 ms at B = 2, L = 4096 (r c_z = 256) --
// and of fewer where a pair's weights would pass the 31-bit byte offsets of the kernels (262144 residues) or all of them
// kStoredBytes.  Where dS' alone is stored, of 8192 rows, and room for the sums of tiles that are cut in parts: as much again, no more than
// kPartBytes (256 parts of either side take 136 MB at r c_z = 256).  Grows with the length throughout: chains that run one after the other
// share a workspace of the longest one's size.
constexpr size_t kPairBytes = 0x7FFFFFFF;  // of either weight of a pair
constexpr size_t kPartBytes = 160ull << 20;
// The least: as much as key-side gradients of the full width (dK^_z and dV^_z apart) would take more than dZ, so that the
// calls run in any workspace that is large enough to form the weights again in every product.
size_t stored_weight_least(size_t BH, int Lp, int DZ) { return BH * Lp * DZ * 4; }
size_t stored_weight_bytes(size_t BH, int Lp, int Lk, int DZ)
{
    const bool both = !bwd_keys_fused(DZ);  // P and dS', else dS' alone
    const size_t most = both ? 4096 : 8192, rows = (size_t)Lp < most ? Lp : most, pair = rows * Lk * 2, least = stored_weight_least(BH, Lp, DZ);
    const size_t one = BH * (pair < kPairBytes ? pair : kPairBytes), more = both || one < kPartBytes ? one : kPartBytes;
    const size_t cap = least > kStoredBytes ? least : kStoredBytes;
    return one + more < cap ? one + more : cap;
}
// Query rows whose weights fit: all of them, or whole tiles of 256, at the least half a tile (which every workspace of the
// least size holds: its DZ Lp / Lk rows, or 2 DZ Lp / Lk where dS' alone is stored, are at least 128, as Lk < 2 Lp).
int stored_query_rows(size_t bytes, size_t BH, int Lp, int Lk, int DZ)
{
    const bool both = !bwd_keys_fused(DZ);  // P and dS', else dS' alone
    const size_t most = kPairBytes / ((size_t)Lk * 2), rows_max = both ? 4096 : 8192, cap = most < rows_max ? most : rows_max;
    const size_t fit = bytes / (BH * Lk * (both ? 4 : 2));
    const size_t rows = fit < cap ? fit : cap;
    return rows >= (size_t)Lp ? Lp : (int)(rows >= 256 ? rows / 256 * 256 : rows / 128 * 128);
}

struct BwdLayout {
    Bf16Layout f;
    size_t dOhat, Dvec, nlse, dQhat, dKhat, dVhat, rowsum, colsum, gpart, wpart, total;
    size_t dKh, dVh, dZ, Wp, Ws;  // stored weights (in the place of dKhat and dVhat)
    bool stored;          // the gradients go through them
    int Lk, nq;           // keys per group of weights; query rows of which the given workspace holds the weights
    size_t parts, parts_bytes;  // what dS' alone leaves of the room of the weights: sums of the parts of a tile (see split_tiles)
    size_t least;         // what the calls run in (total: what the query asks for)
};

// `bytes`: the workspace that is laid out.
BwdLayout bwd_layout(const fipa_desc &d, size_t bytes)
{
    BwdLayout w;
    w.f = bf16_layout(d, true, true);
    const size_t BHL = (size_t)d.B * d.H * w.f.Lp;
    const size_t D = kDH + w.f.DZ;
    size_t off = w.f.total;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    w.dOhat = take(BHL * D * 2);
    w.nlse = take(BHL * 4);
    w.Dvec = take(BHL * 4);
    w.dQhat = take(BHL * D * 4);
    w.dKhat = w.dVhat = w.dKh = w.dVh = w.dZ = w.Wp = w.Ws = 0;
    w.Lk = (int)align_up(w.f.Lp, 256);
    w.nq = 0;
    w.parts = w.parts_bytes = 0;
    w.stored = bwd_stored(w.f.DZ);
    const size_t key_side = off;
    auto sums = [&] {
        w.rowsum = take(BHL * 4);
        w.colsum = take(BHL * 4);
        w.gpart = take(BHL * 4);
        w.wpart = take((size_t)d.H * (((size_t)d.B * d.L + kWbChunk - 1) / kWbChunk) * w.f.DZ * 4);
    };
    auto formed = [&] {  // dK^ and dV^ of the full width
        off = key_side;
        w.dKhat = take(BHL * D * 4);
        w.dVhat = take(BHL * D * 4);
        sums();
    };
    if (w.stored) {
        w.dKh = take(BHL * kDH * 4);
        w.dVh = take(BHL * kDH * 4);
        w.dZ = take(BHL * w.f.DZ * 4);
        sums();
        // (last: as many rows as the workspace has left)
        const size_t BH = (size_t)d.B * d.H, want = stored_weight_bytes(BH, w.f.Lp, w.Lk, w.f.DZ);
        const size_t have = bytes < off ? 0 : (bytes - off < want ? bytes - off : want);
        w.nq = stored_query_rows(have, BH, w.f.Lp, w.Lk, w.f.DZ);
        w.Wp = off;
        w.Ws = bwd_keys_fused(w.f.DZ) ? off : off + BH * w.nq * w.Lk * 2;
        w.parts = align_up(w.Ws + BH * w.nq * w.Lk * 2, 256);
        w.parts_bytes = off + have > w.parts ? off + have - w.parts : 0;
        const size_t least = stored_weight_least(BH, w.f.Lp, w.f.DZ);
        w.least = align_up(off + (least < want ? least : want), 256);
        take(want);
        const size_t total = off;
        if (!stored_pays(w.f.DZ, BH, w.f.Lp, w.nq)) {  // (no more than the least: dZ and the weights there make up dK^_z and dV^_z)
            w.stored = false;
            w.nq = 0;
            w.parts_bytes = 0;
            formed();
        }
        off = total;
    } else {
        formed();
        w.least = off;
    }
    w.total = off;
    return w;
}

}  // namespace

namespace {

template <int NG, int WPR>
void launch_pack(const BwdPackParams &p, int heads, hipStream_t stream)  // heads: per group at a time
{
    const dim3 grid(p.Lp / 4 * WPR, p.B < 32768 ? p.B : 32768, (p.B + 32767) / 32768);
    if (heads == 1) hipLaunchKernelGGL((fipa_bwd_pack_bf16_kernel<NG, WPR, 1>), grid, dim3(256), 0, stream, p);
    else if (heads == 2) hipLaunchKernelGGL((fipa_bwd_pack_bf16_kernel<NG, WPR, 2>), grid, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((fipa_bwd_pack_bf16_kernel<NG, WPR, 3>), grid, dim3(256), 0, stream, p);
}

}  // namespace

// One wave per residue where it takes all heads at once (three per group), else four; no more groups and no more heads at a time than
// there are heads.  Whole backward, us, forward kept: a wave per head and residue (the sum for z1 left to the unpack kernel, which read
// the lifted output again) | four waves per residue, three heads at a time, throughout | this rule, 64 chains of 256 residues: r c_z = 32, H = 1
// 90 | 192 | 89, H = 4 141 | 218 | 124, H = 8 264 | 317 | 232, H = 24 788 | 731 | 683; r c_z = 64, H = 4 162 | 202 | 142; 128, H = 3 188 | 198 | 151,
// H = 8 445 | 348 | 303; 256, H = 1 125 | 161 | 121, H = 3 210 | 243 | 205, H = 4 265 | 267 | 231, H = 12 808 | 644 | 635; B = 2, L = 4096, H = 12
// 1440 | 1250 | 1250 (the kernel 71 | 65 | 65).  One wave per residue at every size: 621 and 1245 in the last two, but 412 against 401 at
// r c_z = 512, H = 4 and 61 against 57 for one chain of 100 residues, H = 8.
// Up to 1024 residues, where latency is all there is: a head per wave, as many lanes as there are columns.  Whole backward with it and
// without: one chain of 200 residues, H = 8, r c_z = 32 68.4 and 70.6 us, r c_z = 64 75 and 77.9, 256 98.0 and 99.7; 16 x 256 at r c_z = 32 108
// and 101 (64 chains of 256 as above).
hipError_t launch_bwd_pack_bf16(const BwdPackParams &p, hipStream_t stream)
{
    const bool small = (long long)p.B * p.Lp <= 1024;
    int NG = p.DZ < 256 && !small ? p.DZ / 4 : 64;
    while (NG < 64 && 32 / NG >= p.H) NG *= 2;
    const int HG = 64 / NG, WPR = p.H > (small ? 1 : 3 * HG) ? 4 : 1, heads = (p.H + WPR * HG - 1) / (WPR * HG);
    const auto launch = [&](auto N) {
        if (WPR == 1) launch_pack<decltype(N)::value, 1>(p, heads, stream);
        else launch_pack<decltype(N)::value, 4>(p, heads, stream);
    };
    return with_column_lanes(4 * NG, launch);
}

hipError_t launch_bwd_unpack_bf16(const BwdUnpackParams &p, hipStream_t stream)
{
    const int nchunk = (p.total_rows + kWbChunk - 1) / kWbChunk;
    // (four heads at a time from as many chunks on as fill the chip that way: 4096 residues, r c_z = 256, one 12.2 us, two 14.6, four 15.0;
    // 9080 residues 30, 23.1, 22.9; 32768 residues padded, 512 columns, 138, 133, 121; fewer heads than four: one)
    const int NH = nchunk < 256 || p.H < 4 ? 1 : 4, nw = p.d_w_b ? (p.H + NH - 1) / NH : 0;
    const int groups = (int)(((long long)p.B * p.L + 31) / 32);
    const dim3 grid(16 + nw, groups < 32768 ? groups : 32768, (groups + 32767) / 32768);
    const hipError_t e = with_column_lanes(p.DZ, [&](auto N) {
        const auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, p, nchunk); };
        if (NH == 1) run(fipa_bwd_unpack_bf16_kernel<decltype(N)::value, 1>);
        else run(fipa_bwd_unpack_bf16_kernel<decltype(N)::value, 4>);
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fipa_bwd_sums_kernel, dim3(p.H, p.d_w_b ? 1 + p.cz / wb_columns(p.cz) : 1), dim3(1024), 0, stream, p, nchunk);
    return hipGetLastError();
}

size_t bf16_backward_workspace(const fipa_desc &d) { return bwd_layout(d, SIZE_MAX).total; }
size_t bf16_backward_workspace_min(const fipa_desc &d) { return bwd_layout(d, SIZE_MAX).least; }

namespace {

PackParams bwd_pack_params(const fipa_desc &d, const FwdArgs &f, const BwdLayout &w, char *base)
{
    PackParams pk;
    pk.q = (const bf16_t *)f.q; pk.k = (const bf16_t *)f.k; pk.v = (const bf16_t *)f.v;
    pk.q_pts = (const bf16_t *)f.q_pts; pk.k_pts = (const bf16_t *)f.k_pts;
    pk.v_pts = (const bf16_t *)f.v_pts;
    pk.z1 = (const bf16_t *)f.z1; pk.z2 = (const bf16_t *)f.z2;
    pk.rot = f.rot; pk.trans = f.trans; pk.w_b = f.w_b; pk.gamma = f.gamma;
    pk.cen = reinterpret_cast<float *>(base + w.f.cen);
    pk.mask = f.mask; pk.cu = f.cu;
    pk.Qh = (bf16_t *)(base + w.f.Qh); pk.Qz = (bf16_t *)(base + w.f.Qz);
    pk.Kh = (bf16_t *)(base + w.f.Kh); pk.Vh = (bf16_t *)(base + w.f.Vh); pk.Z2 = (bf16_t *)(base + w.f.Z2);
    pk.kbias = (float *)(base + w.f.kbias); pk.qbias = (float *)(base + w.f.qbias);
    pk.B = d.B; pk.L = d.L; pk.Lp = w.f.Lp; pk.NT = w.f.NT; pk.H = d.H; pk.c = d.c; pk.Pq = d.Pq;
    pk.Pv = d.Pv; pk.cz = d.cz; pk.r = d.r; pk.DZ = w.f.DZ;
    pk.w_L = d.w_L; pk.w_C = d.w_C; pk.qk_scale = d.qk_scale;
    pk.skip_qz = false;
    // (with the AlphaFold2 head shape the pack kernel finds the per-batch reference point and key-loop bound itself)
    const bool prep_in_pack = d.c == 16 && d.Pq == 4 && d.Pv == 8;
    pk.cen_out = prep_in_pack ? reinterpret_cast<float *>(base + w.f.cen) : nullptr;
    pk.kvlen_out = prep_in_pack ? reinterpret_cast<int *>(base + w.f.kvlen) : nullptr;
    pk.counters = nullptr; pk.n_counters = 0;
    pk.kvlen = reinterpret_cast<const int *>(base + w.f.kvlen);
    return pk;
}

// Forward pack and forward attention: leaves the lifted tensors, O^ and the log-sum-exp in the workspace; when f.o
// is set the core's outputs (steps 8-9) as well, by the attention kernel itself or, where that has no epilogue for
// the shape, from O^.
hipError_t backward_forward_part(const fipa_desc &d, const FwdArgs &f, const BwdLayout &w, char *base, hipStream_t stream)
{
    float *cen = reinterpret_cast<float *>(base + w.f.cen);
    int *kvlen = reinterpret_cast<int *>(base + w.f.kvlen);
    const PackParams pk = bwd_pack_params(d, f, w, base);
    hipError_t e = hipSuccess;
    if (!pk.cen_out) {
        e = launch_prep(d, f.trans, f.mask, f.cu, cen, kvlen, nullptr, 0, stream);
        if (e != hipSuccess) return e;
    }
    e = launch_pack_bf16(pk, stream);
    if (e != hipSuccess) return e;

    AttnParams at;
    at.Qh = pk.Qh; at.Qz = pk.Qz; at.Kh = pk.Kh; at.Vh = pk.Vh; at.Z2 = pk.Z2;
    at.kbias = pk.kbias; at.qbias = pk.qbias; at.kvlen = kvlen;
    at.Ohat = (float *)(base + w.f.Ohat); at.lse2 = (float *)(base + w.f.lse2);
    at.rot = f.rot; at.trans = f.trans; at.cen = cen; at.z1 = pk.z1; at.mask = f.mask; at.cu = f.cu;
    at.o = nullptr; at.o_pts = nullptr; at.o_pair = nullptr; at.lse = nullptr;
    at.B = d.B; at.L = d.L; at.Lp = w.f.Lp; at.H = d.H; at.NT = w.f.NT;
    at.nQT = w.f.Lp / kTileQ; at.total_tiles = at.nQT * d.B * d.H; at.cz = d.cz; at.r = d.r; at.w_b = f.w_b; at.w_L = d.w_L;
    at.plan = w.f.plan; at.partial = nullptr; at.counters = nullptr;  // (O^ is left: never split)
    at.deal = f.mask != nullptr || f.cu != nullptr;
    // Where steps 8-9 run on the accumulator the attention kernel leaves the outputs beside O^ (kept steps, module).
    const bool one_pass = attn_fwd_576_pays(at, w.f.DZ);
    const bool fused = f.o && (one_pass ? bf16_wide_fused_epilogue(d) : bf16_fused_epilogue(d));
    if (fused) {
        at.o = f.o; at.o_pts = f.o_pts; at.o_pair = f.o_pair; at.lse = f.lse;
    }
    e = one_pass          ? launch_attn_fwd_576_bf16(at, fused, stream)
        : w.f.DZ > 256    ? launch_attn_fwd_wide_bf16(at, w.f.DZ, false, stream)
        : fused           ? launch_attn_fwd_keep_bf16(at, w.f.DZ, stream)
                          : launch_attn_fwd_bf16(at, w.f.DZ, false, stream);
    if (e != hipSuccess || !f.o || fused) return e;

    EpiParams ep;
    ep.Ohat = at.Ohat; ep.lse2 = at.lse2; ep.qbias = pk.qbias; ep.rot = f.rot; ep.trans = f.trans;
    ep.cen = cen; ep.z1 = pk.z1; ep.mask = f.mask; ep.cu = f.cu;
    ep.o = f.o; ep.o_pts = f.o_pts; ep.o_pair = f.o_pair; ep.lse = f.lse;
    ep.B = d.B; ep.L = d.L; ep.Lp = w.f.Lp; ep.H = d.H; ep.c = d.c; ep.Pv = d.Pv; ep.cz = d.cz;
    ep.r = d.r; ep.DZ = w.f.DZ;
    return launch_epilogue_bf16(ep, stream);
}

// Everything after the forward part: lifting of the upstream gradients, the three gradient
// kernels, and the way back to the inputs.
hipError_t backward_gradient_part(const fipa_desc &d, const BwdArgs &a, const BwdLayout &w, char *base, hipStream_t stream,
                                  StageTimer &timer)
{
    const int total_rows = a.f.cu ? a.f.total_rows : d.B * d.L;  // rows of the caller's tensors
    float *cen = reinterpret_cast<float *>(base + w.f.cen);
    int *kvlen = reinterpret_cast<int *>(base + w.f.kvlen);
    const PackParams pk = bwd_pack_params(d, a.f, w, base);
    float *Ohat = (float *)(base + w.f.Ohat);

    BwdPackParams bp;
    bp.d_o = a.d_o; bp.d_o_pts = a.d_o_pts; bp.d_o_pair = a.d_o_pair; bp.rot = a.f.rot;
    bp.Ohat = Ohat; bp.lse2 = (float *)(base + w.f.lse2); bp.z1 = pk.z1; bp.mask = a.f.mask; bp.cu = a.f.cu;
    bp.dOhat = (bf16_t *)(base + w.dOhat); bp.Dvec = (float *)(base + w.Dvec); bp.nlse = (float *)(base + w.nlse);
    bp.B = d.B; bp.L = d.L; bp.Lp = w.f.Lp; bp.H = d.H; bp.c = d.c; bp.Pv = d.Pv; bp.cz = d.cz; bp.r = d.r;
    bp.DZ = w.f.DZ; bp.d_z1 = (bf16_t *)a.d_z1; bp.d_z2 = (bf16_t *)a.d_z2;
    const bool stored = w.stored;
    bp.neg_d = stored; bp.kvlen = kvlen;
    hipError_t e = launch_bwd_pack_bf16(bp, stream);
    if (e != hipSuccess) return e;
    timer.end(0);

    // ---- dQ^, dK^, dV^ --------------------------------------------------------------------------------
    timer.begin(1);
    if (stored) {
        BwdStoredParams sp;
        sp.Qh = pk.Qh; sp.Qz = pk.Qz; sp.Kh = pk.Kh; sp.Vh = pk.Vh; sp.Z2 = pk.Z2; sp.dOhat = bp.dOhat;
        sp.kbias = pk.kbias; sp.nlse = bp.nlse; sp.d_minus_nlse = (int)((w.Dvec - w.nlse)); sp.kvlen = kvlen;
        sp.Wp = (bf16_t *)(base + w.Wp); sp.Ws = (bf16_t *)(base + w.Ws);
        sp.dQ = (float *)(base + w.dQhat); sp.dKh = (float *)(base + w.dKh); sp.dVh = (float *)(base + w.dVh);
        sp.dZ = (float *)(base + w.dZ); sp.rowsum = (float *)(base + w.rowsum); sp.colsum = (float *)(base + w.colsum);
        sp.B = d.B; sp.L = d.L; sp.Lp = w.f.Lp; sp.H = d.H; sp.deal = a.f.mask != nullptr || a.f.cu != nullptr;
        sp.Lk = w.Lk; sp.nq_alloc = w.nq; sp.i0 = 0; sp.nq = 0;
        sp.parts = sp.q_parts = (float *)(base + w.parts); sp.parts_bytes = w.parts_bytes;
        sp.k_full = sp.q_full = 0; sp.k_S = sp.q_S = 1; sp.units = sp.q_units = sp.nseg = sp.seg_blocks = 0;
        e = launch_bwd_stored_bf16(sp, w.f.DZ, stream);
        if (e != hipSuccess) return e;
    } else {
        BwdParams bw;
        bw.Qh = pk.Qh; bw.Qz = pk.Qz; bw.Kh = pk.Kh; bw.Vh = pk.Vh; bw.Z2 = pk.Z2; bw.dOhat = bp.dOhat;
        bw.kbias = pk.kbias; bw.nlse = bp.nlse; bw.Dvec = bp.Dvec; bw.kvlen = kvlen;
        bw.B = d.B; bw.L = d.L; bw.Lp = w.f.Lp; bw.H = d.H; bw.total_tiles = (w.f.Lp / kTileQ) * d.B * d.H;
        bw.deal = a.f.mask != nullptr || a.f.cu != nullptr;
        bw.out = (float *)(base + w.dQhat); bw.wsum = (float *)(base + w.rowsum);
        e = launch_bwd_bf16(bw, w.f.DZ, FIPA_BWD_DQ, stream);
        if (e != hipSuccess) return e;
        bw.out = (float *)(base + w.dKhat); bw.wsum = (float *)(base + w.colsum);
        e = launch_bwd_bf16(bw, w.f.DZ, FIPA_BWD_DK, stream);
        if (e != hipSuccess) return e;
        bw.out = (float *)(base + w.dVhat); bw.wsum = nullptr;
        e = launch_bwd_bf16(bw, w.f.DZ, FIPA_BWD_DV, stream);
        if (e != hipSuccess) return e;
    }
    timer.end(1);

    // ---- back to the inputs ----------------------------------------------------------------------------
    timer.begin(2);
    BwdUnpackParams up;
    up.q_pts = pk.q_pts; up.k_pts = pk.k_pts; up.v_pts = pk.v_pts; up.z1 = pk.z1;
    up.d_o_pts = a.d_o_pts; up.d_rot = a.d_rot; up.d_trans = a.d_trans; up.dOhat = bp.dOhat;
    up.rot = a.f.rot; up.trans = a.f.trans; up.cen = cen; up.gamma = a.f.gamma; up.w_b = a.f.w_b;
    up.d_o_pair = a.d_o_pair; up.mask = a.f.mask; up.cu = a.f.cu;
    up.total_rows = total_rows;
    up.dQhat = (const float *)(base + w.dQhat); up.Ohat = Ohat;
    const int D = kDH + w.f.DZ;
    up.dKh = (const float *)(base + (stored ? w.dKh : w.dKhat));
    up.dVh = (const float *)(base + (stored ? w.dVh : w.dVhat));
    up.dKz = stored ? (const float *)(base + w.dZ) : up.dKh + kDH;
    up.dVz = stored ? nullptr : up.dVh + kDH;
    up.h_pitch = stored ? kDH : D;
    up.z_pitch = stored ? w.f.DZ : D;
    up.ds_inv = stored ? kLog2e : 1.f;
    up.rowsum = (const float *)(base + w.rowsum); up.colsum = (const float *)(base + w.colsum);
    up.d_q = (bf16_t *)a.d_q; up.d_k = (bf16_t *)a.d_k; up.d_v = (bf16_t *)a.d_v;
    up.d_q_pts = (bf16_t *)a.d_q_pts; up.d_k_pts = (bf16_t *)a.d_k_pts; up.d_v_pts = (bf16_t *)a.d_v_pts;
    up.d_z1 = (bf16_t *)a.d_z1; up.d_z2 = (bf16_t *)a.d_z2;
    up.gpart = (float *)(base + w.gpart); up.d_gamma = a.d_gamma;
    up.d_w_b = a.d_w_b; up.wpart = (float *)(base + w.wpart);
    up.B = d.B; up.L = d.L; up.Lp = w.f.Lp; up.H = d.H; up.c = d.c; up.Pq = d.Pq; up.Pv = d.Pv; up.cz = d.cz;
    up.r = d.r; up.DZ = w.f.DZ;
    up.w_L = d.w_L; up.w_C = d.w_C; up.qk_scale = d.qk_scale;
    e = launch_bwd_unpack_bf16(up, stream);
    timer.end(2);
    return e;
}

}  // namespace

hipError_t bf16_backward(const fipa_desc &d, const BwdArgs &a, void *ws, size_t ws_bytes, hipStream_t stream)
{
    const BwdLayout w = bwd_layout(d, ws_bytes);
    if (ws_bytes < w.least) return hipErrorInvalidValue;
    char *base = static_cast<char *>(ws);
    StageTimer timer(stream);
    timer.begin(0);
    FwdArgs f = a.f;
    f.o = nullptr;  // (the core's outputs are not needed here)
    const hipError_t e = backward_forward_part(d, f, w, base, stream);
    if (e != hipSuccess) return e;
    return backward_gradient_part(d, a, w, base, stream, timer);
}

// The same in two calls on one workspace, for a caller that needs the core's outputs before it
// can form the upstream gradients (the module's backward): the first call also writes f.o,
// f.o_pts, f.o_pair; the workspace must not be touched in between.
hipError_t bf16_backward_begin(const fipa_desc &d, const FwdArgs &f, void *ws, size_t ws_bytes, hipStream_t stream)
{
    const BwdLayout w = bwd_layout(d, ws_bytes);
    if (!f.o || !f.o_pts || !f.o_pair || ws_bytes < w.least) return hipErrorInvalidValue;
    return backward_forward_part(d, f, w, static_cast<char *>(ws), stream);
}

hipError_t bf16_backward_finish(const fipa_desc &d, const BwdArgs &a, void *ws, size_t ws_bytes, hipStream_t stream)
{
    const BwdLayout w = bwd_layout(d, ws_bytes);
    if (ws_bytes < w.least) return hipErrorInvalidValue;
    StageTimer timer;  // (not timed)
    return backward_gradient_part(d, a, w, static_cast<char *>(ws), stream, timer);
}

}  // namespace fipa
