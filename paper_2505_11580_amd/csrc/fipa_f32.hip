// fp32 direct path: logits from explicit point differences (Eq. 3), online softmax over key
// tiles, fp32 accumulation of the lifted values (Algorithm 1 steps 6-7), and the split /
// inverse frame / z1 contraction (steps 8-9, Eq. 4) in the same kernel.  The dot products run on
// the fp32 matrix instructions (full fp32 operands and accumulation: this is the accuracy path,
// 1e-4); the squared distances stay explicit differences on the vector ALU, because the expanded
// form cancels at global coordinates.
#include "fipa_bf16_common.h"
#include "fipa_f32.h"

namespace fipa {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// A packed record of residue i and head h, HRW floats, [B, H, L, HRW]:
//   [ k (c, padded to 16) | Kg (3 N_query, padded to 4) | v, Vg (padded to 16) | Qg, generic shapes only ].
// A key in LDS: the record up to Vg -- generic shapes leave Kg out, which has no bound there, and read it
// and Qg from memory -- and then the key's z2 row (DZ, padded to 16).
struct F32Geom {
    int c16, nq4, nh16, HRW, DZ16;
    int voff, zoff;  // v and z2 in an LDS record
    int S;    // LDS record stride in floats: an odd multiple of 4, so that 8 rows read 16 bytes each from 8 distinct bank groups
    int nch;  // 16-feature chunks of the contraction: k and z2
    int nt;   // 16-column tiles of the values: v, Vg and z2
};

__host__ __device__ constexpr F32Geom f32_geom(int c, int Pq, int Pv, int DZ, bool exact)
{
    F32Geom g{};
    g.c16 = (c + 15) / 16 * 16;
    g.nq4 = (3 * Pq + 3) / 4 * 4;
    g.nh16 = (c + 3 * Pv + 15) / 16 * 16;
    g.HRW = g.c16 + g.nq4 + g.nh16 + (exact ? 0 : g.nq4);
    g.DZ16 = (DZ + 15) / 16 * 16;
    g.voff = g.c16 + (exact ? g.nq4 : 0);
    g.zoff = g.voff + g.nh16;
    g.S = g.zoff + g.DZ16;
    if ((g.S / 4) % 2 == 0) g.S += 4;
    g.nch = (g.c16 + g.DZ16) / 16;
    g.nt = (g.nh16 + g.DZ16) / 16;
    return g;
}

// AlphaFold2's head shape, with rows that can be read as 16-byte pieces, at the widths that f32_forward has an EXACT kernel
// for (16, 32, .. 512).  The record, the workspace and the choice of the kernel all follow this one predicate: every other
// width (rank 3, say) takes the generic kernel, whose record also holds Qg.
bool f32_exact(const fipa_desc &d)
{
    const int DZ = d.r * d.cz;
    return d.c == 16 && d.Pq == 4 && d.Pv == 8 && d.cz % 4 == 0 && DZ >= 16 && (DZ & (DZ - 1)) == 0;
}

struct F32Params {
    const float *q, *k, *v, *q_pts, *k_pts, *v_pts, *z1, *z2, *rot, *trans, *gamma, *w_b;
    const uint8_t *mask;
    const int *cu;  // always null here (user_row and batch_reference want the member)
    float *HR, *cen;
    int *kvlen;
    float *o, *o_pts, *o_pair, *lse;
    int B, L, H, c, Pq, Pv, cz, r, DZ;
    F32Geom g;
    int n_units, n_rt;  // row tiles in all, and per (b, h)
    bool vec;           // c, cz and DZ are multiples of 4: rows can be read as 16-byte pieces
    float w_L, w_C, qk_scale;
};

// Key records (Algorithm 1 steps 4-6: K = T o k_pts, V = T o v_pts relative to the batch's reference
// point), zero for masked residues: one thread per 16 bytes of a record.  Every workgroup finds the
// reference point itself; the one that starts a batch element publishes it with the key-loop bound.
__global__ __launch_bounds__(256) void fipa_pack_f32_kernel(F32Params p)
{
    const int b = blockIdx.y, X4 = p.g.HRW / 4;
    float cen[3];
    int kv;
    batch_reference(p, b, cen, kv);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        for (int a = 0; a < 3; ++a) p.cen[4 * b + a] = cen[a];
        p.cen[4 * b + 3] = 0.f;
        p.kvlen[b] = kv;
    }
    // (whole workgroups per head: the pieces of all heads pass 32 bits at 64 GiB of records)
    const unsigned pieces = (unsigned)p.L * X4, per_head = (pieces + 255u) / 256u;
    const int h = blockIdx.x / per_head;
    const unsigned idx = (blockIdx.x - h * per_head) * 256u + threadIdx.x;
    if (idx >= pieces) return;
    const int i = idx / X4, x0 = 4 * (int)(idx - i * X4);
    const size_t urow = (size_t)b * p.L + i, row = urow * p.H + h;
    const bool ok = p.mask ? p.mask[urow] != 0 : true;
    const int nv = 3 * p.Pv;
    f32x4 out = {0.f, 0.f, 0.f, 0.f};
    if (ok) {
        const float *R = p.rot + urow * 9, *t = p.trans + urow * 3;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int x = x0 + e, pt = -1;
            const float *src = nullptr;
            float val = 0.f;
            if (x < p.g.c16) {
                if (x < p.c) val = p.k[row * p.c + x];
            } else if (x < p.g.c16 + p.g.nq4) {
                x -= p.g.c16;
                if (x < 3 * p.Pq) { pt = x; src = p.k_pts + row * 3 * p.Pq; }
            } else if (x < p.g.c16 + p.g.nq4 + p.g.nh16) {
                x -= p.g.c16 + p.g.nq4;
                if (x < p.c) val = p.v[row * p.c + x];
                else if (x < p.c + nv) { pt = x - p.c; src = p.v_pts + row * nv; }
            } else {
                x -= p.g.c16 + p.g.nq4 + p.g.nh16;
                if (x < 3 * p.Pq) { pt = x; src = p.q_pts + row * 3 * p.Pq; }
            }
            if (pt >= 0) {
                const int pp = pt / 3, a = pt - 3 * pp;
                const float *l = src + 3 * pp;
                val = R[3 * a] * l[0] + R[3 * a + 1] * l[1] + R[3 * a + 2] * l[2] + (t[a] - cen[a]);
            }
            out[e] = val;
        }
    }
    *reinterpret_cast<f32x4 *>(p.HR + (((size_t)b * p.H + h) * p.L + i) * p.g.HRW + x0) = out;
}

__device__ __forceinline__ float group_max(float x)  // over the four 16-lane groups of a wave
{
    x = fmaxf(x, __shfl_xor(x, 16));
    return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float group_sum(float x)
{
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// One workgroup = RG groups of 16 query rows; its four waves are RG row groups x KS = 4 / RG shares
// of the key tiles (16 keys each), merged through LDS at the end.  Both products are formed
// transposed with the 16x16x4 fp32 MFMA (S^T = K Q^T, O^T += V^T P^T): a lane then owns one query
// (lane % 16) and the four keys 4 (lane / 16) + e of a tile, its S^T registers are the B operand of
// the second product as they stand (step e takes key 4 g + e from lane group g), and the softmax
// statistics are per-lane scalars.  The contraction index is permuted the same way on both sides
// (feature 16 ch + 4 g + e in step e of lane group g), so the operands are read 16 bytes at a time.
// NCH, NT: chunk and tile counts, compile-time exact when EXACT (AlphaFold2's head shape with 12 query
// coordinates kept in registers), otherwise upper bounds.
// Bound: fp32 matrix pipe, 256 flop per clock and CU; one 16x16x4 takes 32 clocks, in which a wave
// needs one 4-byte LDS operand per lane, so LDS and the vector ALU have room to spare.  With KS key
// shares per workgroup the units are small (16 or 32 rows) and every CU gets several.
// B = 2, L = 1024, H = 12, r c_z = 256: 0.44 ms, 43 % of the 157 TFLOP/s of the fp32 matrix pipe (the
// vector-ALU form, one wave per four rows, 5.32 ms); L = 64, H = 4, r c_z = 32: 8 us (40 us).  Longer chains of
// AlphaFold2's head shape at r c_z = 32 to 256 run on split operands (fipa_f32_split.hip).
// PACK (EXACT, RG = 1): short chains, no records in memory: a workgroup forms those of the keys that it loads, and the batch's reference
// point, itself, and the call is one launch (see f32_one_launch).  One chain of 64 residues, H = 4, r c_z = 32: 13.2 -> 10.2 us.
template <int NCH, int NT, bool EXACT, int RG, bool PACK>
__global__ __launch_bounds__(256, EXACT && (NCH + NT) * 4 + 60 <= 256 ? 2 : 1) void fipa_attn_f32_kernel(F32Params p)
{
    constexpr int KS = 4 / RG;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const F32Geom G = EXACT ? f32_geom(16, 4, 8, 16 * (NCH - 1), true) : p.g;  // (the first is folded to constants)
    const int S = G.S;
    float *const tiles = smem;                       // [KS][16][S]; at the end partial sums and output rows
    float *const kb = smem + KS * 16 * S;            // [KS * 16] 0 or -inf
    float *const ml = kb + KS * 16;                  // [4][16][2] maximum and sum of a wave's share

    const int per = (p.n_units + 7) / 8;             // an XCD gets neighbouring units: it shares their keys in its L2
    const int unit = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if ((int)(blockIdx.x / 8) >= per || unit >= p.n_units) return;
    const int bh = unit / p.n_rt, b = bh / p.H, h = bh - b * p.H;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int rg = wave % RG, ks = wave / RG;
    const int i_wg = (unit - bh * p.n_rt) * (16 * RG);
    const int L = p.L, H = p.H, DZ = p.DZ, nq = 3 * p.Pq, nv = 3 * p.Pv;
    // (The reference point is read where it is wanted up to r c_z = 256: kept to the end it took up to 1 % of one chain of 257 to 383
    // residues.  At 512 it is the other way round.)
    constexpr bool kKeepReference = PACK || NCH == 33;
    [[maybe_unused]] float cen[3];
    int kvlen;
    if constexpr (PACK) {
        batch_reference(p, b, cen, kvlen);
    } else {
        kvlen = p.kvlen[b];
        if constexpr (kKeepReference)
            for (int a = 0; a < 3; ++a) cen[a] = p.cen[4 * b + a];
    }
    const auto reference = [&](int a) {
        if constexpr (kKeepReference) return cen[a];
        else return p.cen[4 * b + a];
    };
    const int nch = G.nch, nt = G.nt;
    const int zoff = G.zoff, voff = G.voff, cch = G.c16 / 16;
    const float coef = kLog2e * 0.5f * p.gamma[h] * p.w_L * p.w_C;

    // query side: scaled scalars and factor bias vector b^{h1} (log2 units), global points
    const int iq = min(i_wg + 16 * rg + n, L - 1);
    const size_t urow = (size_t)b * L + iq, row = urow * H + h;
    f32x4 qf[NCH];
    {
        const float sc = kLog2e * p.w_L * p.qk_scale, bz = kLog2e * p.w_L;
        const float *q = p.q + row * p.c, *z1 = p.z1 + urow * DZ, *wb = p.w_b + (size_t)h * p.cz;
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            qf[ch] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (EXACT) {
                const int x = 16 * (ch - cch) + 4 * g;
                if (ch < cch)
                    qf[ch] = sc * *reinterpret_cast<const f32x4 *>(q + x + 16);
                else
                    qf[ch] = bz * *reinterpret_cast<const f32x4 *>(wb + x % p.cz) * *reinterpret_cast<const f32x4 *>(z1 + x);
            } else if (ch < nch) {
                const int x = 16 * ch + 4 * g, xz = x - 16 * cch;
                for (int e = 0; e < 4; ++e) {
                    float val = 0.f;
                    if (ch < cch) {
                        if (x + e < p.c) val = sc * q[x + e];
                    } else if (xz + e < DZ) {
                        val = bz * wb[(xz + e) % p.cz] * z1[xz + e];
                    }
                    qf[ch][e] = val;
                }
            }
        }
    }
    const float *const hr = p.HR + (size_t)bh * L * G.HRW;
    float qg[12];
    const float *qg_mem = hr + (size_t)iq * G.HRW + G.c16 + G.nq4 + G.nh16;
    if (EXACT) {
        const float *R = p.rot + urow * 9, *t = p.trans + urow * 3, *src = p.q_pts + row * nq;
#pragma unroll
        for (int x = 0; x < 12; ++x) {
            const int pp = x / 3, a = x % 3;
            qg[x] = R[3 * a] * src[3 * pp] + R[3 * a + 1] * src[3 * pp + 1] + R[3 * a + 2] * src[3 * pp + 2] + (t[a] - reference(a));
        }
    }

    float m = -INFINITY, l = 0.f;
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const float *z2 = p.z2 + (size_t)b * L * DZ;
    const int nhr = G.zoff / 4, nz = G.DZ16 / 4;
    const float *tile = tiles + ks * 16 * S;
    for (int j0 = 0; j0 < kvlen; j0 += 16 * KS) {
        __syncthreads();
        const int nj = min(16 * KS, kvlen - j0);  // rows past it are zero and masked
        if constexpr (PACK) {
            // the record of every key: a thread per point, then one per 16 bytes of scalars or padding
            constexpr int kPts = 12, kRest = 10;
#pragma unroll
            for (int it = 0; it < 16 * KS * kPts / 256; ++it) {
                const int idx = threadIdx.x + 256 * it, jj = idx / kPts, pt = idx - kPts * jj;
                const size_t ukey = (size_t)b * L + min(j0 + jj, L - 1);
                const bool ok = jj < nj && (p.mask ? p.mask[ukey] != 0 : true);
                const float *src = pt < 4 ? p.k_pts + (ukey * H + h) * 12 + 3 * pt : p.v_pts + (ukey * H + h) * 24 + 3 * (pt - 4);
                const float *R = p.rot + ukey * 9, *t = p.trans + ukey * 3;
                float *dst = tiles + jj * S + (pt < 4 ? 16 + 3 * pt : 44 + 3 * (pt - 4));
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float val = R[3 * a] * src[0] + R[3 * a + 1] * src[1] + R[3 * a + 2] * src[2] + (t[a] - cen[a]);
                    dst[a] = ok ? val : 0.f;
                }
            }
#pragma unroll
            for (int it = 0; it < (16 * KS * kRest + 255) / 256; ++it) {
                const int idx = threadIdx.x + 256 * it, jj = idx / kRest, x = idx - kRest * jj;
                if (jj >= 16 * KS) break;
                const size_t ukey = (size_t)b * L + min(j0 + jj, L - 1);
                const bool ok = jj < nj && (p.mask ? p.mask[ukey] != 0 : true);
                const f32x4 val = *reinterpret_cast<const f32x4 *>((x < 4 ? p.k : p.v) + (ukey * H + h) * 16 + 4 * (x & 3));
                *reinterpret_cast<f32x4 *>(tiles + jj * S + (x < 4 ? 4 * x : x < 8 ? 28 + 4 * (x - 4) : 68 + 4 * (x - 8))) =
                    ok && x < 8 ? val : (f32x4){0.f, 0.f, 0.f, 0.f};
            }
        } else
#pragma unroll 4
        for (int idx = threadIdx.x; idx < 16 * KS * nhr; idx += 256) {
            const int jj = idx / nhr, x = 4 * (idx - jj * nhr);
            f32x4 val = {0.f, 0.f, 0.f, 0.f};
            if (jj < nj)
                val = *reinterpret_cast<const f32x4 *>(hr + (size_t)(j0 + jj) * G.HRW + x + (EXACT || x < G.c16 ? 0 : G.nq4));
            *reinterpret_cast<f32x4 *>(tiles + jj * S + x) = val;
        }
#pragma unroll 4
        for (int idx = threadIdx.x; idx < 16 * KS * nz; idx += 256) {
            const int jj = idx / nz, x = 4 * (idx - jj * nz);
            f32x4 val = {0.f, 0.f, 0.f, 0.f};
            if (jj < nj) {
                const float *src = z2 + (size_t)(j0 + jj) * DZ + x;
                if (EXACT || (p.vec && x < DZ)) {
                    val = *reinterpret_cast<const f32x4 *>(src);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (x + e < DZ) val[e] = src[e];
                }
            }
            *reinterpret_cast<f32x4 *>(tiles + jj * S + zoff + x) = val;
        }
        if (threadIdx.x < 16 * KS) {
            const int j = j0 + threadIdx.x;
            kb[threadIdx.x] = j < kvlen && (p.mask ? p.mask[(size_t)b * L + j] != 0 : true) ? 0.f : -INFINITY;
        }
        __syncthreads();
        if (j0 + 16 * ks >= kvlen) continue;  // (wave uniform; the barriers above are reached by every wave)

        // S^T of this wave's 16 keys: two accumulation chains
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            // (generic shapes: the surplus chunks read something finite against zero query features)
            const int off = ch < cch || (!EXACT && ch >= nch) ? (EXACT || ch < cch ? 16 * ch : 0) : zoff + 16 * (ch - cch);
            const f32x4 a = *reinterpret_cast<const f32x4 *>(tile + n * S + off + 4 * g);
            f32x4 &s = ch & 1 ? s1 : s0;
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], qf[ch][e], s, 0, 0, 0);
        }
        // explicit squared distances of the four keys 4 g + e
        f32x4 dist = {0.f, 0.f, 0.f, 0.f};
        if (EXACT) {
            const float *kg = tile + 4 * g * S + G.c16;
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int x = 0; x < 12; x += 4) {
                    const f32x4 kv4 = *reinterpret_cast<const f32x4 *>(kg + e * S + x);
#pragma unroll
                    for (int y = 0; y < 4; ++y) {
                        const float df = qg[x + y] - kv4[y];
                        dist[e] += df * df;
                    }
                }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float *kg = hr + (size_t)min(j0 + 16 * ks + 4 * g + e, L - 1) * G.HRW + G.c16;
                for (int x = 0; x < G.nq4; x += 4) {
                    const f32x4 df = *reinterpret_cast<const f32x4 *>(qg_mem + x) - *reinterpret_cast<const f32x4 *>(kg + x);
                    dist[e] += (df[0] * df[0] + df[1] * df[1]) + (df[2] * df[2] + df[3] * df[3]);
                }
            }
        }
        const f32x4 mb = *reinterpret_cast<const f32x4 *>(kb + 16 * ks + 4 * g);
        f32x4 s;
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = mb[e] == 0.f ? (s0[e] + s1[e]) - coef * dist[e] : -INFINITY;
        // online softmax (running maximum and sum; the accumulator is rescaled when a maximum moved)
        const float mt = group_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
        if (__any(mt > m)) {
            const float m_new = fmaxf(m, mt);
            const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - m_new);
            l *= alpha;
            m = m_new;
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] *= alpha;
        }
        const float m_use = m == -INFINITY ? 0.f : m;
        f32x4 pw;
#pragma unroll
        for (int e = 0; e < 4; ++e) pw[e] = __builtin_amdgcn_exp2f(s[e] - m_use);
        l += (pw[0] + pw[1]) + (pw[2] + pw[3]);
        // O^T += V^T P^T
        const float *vt = tile + 4 * g * S + voff + n;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                // (generic shapes: the surplus tiles accumulate column block 0 again, unused)
                const int off = EXACT || t < nt ? 16 * t : 0;
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vt[e * S + off], pw[e], acc[t], 0, 0, 0);
            }
    }
    l = group_sum(l);

    // merge the key shares: every wave but those of share 0 leaves its sums in LDS
    const int RS = 16 * nt + 4;  // row stride of the partial sums; 16 rows fit a key tile's space
    __syncthreads();
    if (g == 0) {
        ml[(wave * 16 + n) * 2] = m;
        ml[(wave * 16 + n) * 2 + 1] = l;
    }
    if (ks > 0) {
        float *dst = tiles + (wave - RG) * 16 * S + n * RS + 4 * g;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (EXACT || t < nt) *reinterpret_cast<f32x4 *>(dst + 16 * t) = acc[t];
    }
    __syncthreads();
    if (ks == 0) {
        float m_all = m;
        for (int x = 1; x < KS; ++x) m_all = fmaxf(m_all, ml[((x * RG + rg) * 16 + n) * 2]);
        const float m_use = m_all == -INFINITY ? 0.f : m_all;
        float w = __builtin_amdgcn_exp2f(m - m_use);
        float l_all = l * w;
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] *= w;
        for (int x = 1; x < KS; ++x) {
            const float *s_ml = ml + ((x * RG + rg) * 16 + n) * 2;
            w = __builtin_amdgcn_exp2f(s_ml[0] - m_use);
            l_all += s_ml[1] * w;
            const float *src = tiles + ((x - 1) * RG + rg) * 16 * S + n * RS + 4 * g;
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (EXACT || t < nt) acc[t] += w * *reinterpret_cast<const f32x4 *>(src + 16 * t);
        }
        // (only this wave has read the space that its output rows now take)
        const float inv = l_all > 0.f ? 1.f / l_all : 0.f;
        float *dst = tiles + rg * 16 * S + n * RS + 4 * g;
#pragma unroll
        for (int t = 0; t < NT; ++t)
            if (EXACT || t < nt) *reinterpret_cast<f32x4 *>(dst + 16 * t) = inv * acc[t];
        if (g == 0) {
            ml[(wave * 16 + n) * 2] = m_all;
            ml[(wave * 16 + n) * 2 + 1] = l_all;
        }
    }
    __syncthreads();

    // split, inverse frame, z1 contraction (Algorithm 1 steps 8-9, Eq. 4): 16 threads per row and group
    for (int rr = 0; rr < RG; ++rr) {
        const int rl = threadIdx.x >> 4, x0 = threadIdx.x & 15;
        const int i = i_wg + 16 * rr + rl;
        if (i >= L) continue;
        const size_t ui = (size_t)b * L + i, ro = ui * H + h;
        const float *rb = tiles + rr * 16 * S + rl * RS;
        const float m_row = ml[(rr * 16 + rl) * 2], l_row = ml[(rr * 16 + rl) * 2 + 1];
        const bool valid = (p.mask ? p.mask[ui] != 0 : true) && l_row > 0.f;
        for (int d = x0; d < p.c; d += 16) p.o[ro * p.c + d] = valid ? rb[d] : 0.f;
        const float *R = p.rot + ui * 9, *t = p.trans + ui * 3;
        for (int idx = x0; idx < nv; idx += 16) {
            const int pp = idx / 3, x = idx - 3 * pp;
            float val = 0.f;
            for (int y = 0; y < 3; ++y) val += R[3 * y + x] * (rb[p.c + 3 * pp + y] - (t[y] - reference(y)));
            p.o_pts[ro * nv + idx] = valid ? val : 0.f;
        }
        const float *z1 = p.z1 + ui * DZ;
        if (p.vec) {
            for (int d = 4 * x0; d < p.cz; d += 64) {
                f32x4 val = {0.f, 0.f, 0.f, 0.f};
                for (int rho = 0; rho < p.r; ++rho)
                    val += *reinterpret_cast<const f32x4 *>(z1 + rho * p.cz + d) *
                           *reinterpret_cast<const f32x4 *>(rb + G.nh16 + rho * p.cz + d);
                if (!valid) val = (f32x4){0.f, 0.f, 0.f, 0.f};
                *reinterpret_cast<f32x4 *>(p.o_pair + ro * p.cz + d) = val;
            }
        } else {
            for (int d = x0; d < p.cz; d += 16) {
                float val = 0.f;
                for (int rho = 0; rho < p.r; ++rho) val += z1[rho * p.cz + d] * rb[G.nh16 + rho * p.cz + d];
                p.o_pair[ro * p.cz + d] = valid ? val : 0.f;
            }
        }
        if (p.lse && x0 == 0) p.lse[((size_t)b * H + h) * L + i] = valid ? kLn2 * (m_row + __log2f(l_row)) : 0.f;
    }
}

struct F32Layout {
    size_t cen, kvlen, HR, total;
};

F32Layout f32_layout(const fipa_desc &d)
{
    F32Layout w;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    w.cen = take((size_t)d.B * 4 * sizeof(float));
    w.kvlen = take((size_t)d.B * sizeof(int));
    w.HR = take((size_t)d.B * d.H * d.L * f32_geom(d.c, d.Pq, d.Pv, d.r * d.cz, f32_exact(d)).HRW * sizeof(float));
    w.total = off;
    return w;
}

// Chains short enough that every workgroup forms the records of all keys itself (fipa_attn_f32_kernel<.., PACK>) in less than a launch takes.
// Two launches | one, us per call: r c_z = 32, H = 4, L = 64 14.0 | 11.1, 256 21.7 | 17.2; B = 2, H = 12, L = 256 24.8 | 20.0, 384 34.4 | 46.5;
// r c_z = 128, B = 2, H = 12, L = 64 16.8 | 12.3, 256 37.4 | 32.0, 384 76.0 | 74.5; r c_z = 256, H = 12, L = 64 20.8 | 18.1, 128 27.3 | 26.6,
// two chains of 117, H = 4 25.4 | 26.1, 192 34.2 | 35.1; r c_z = 512, H = 12, L = 64 30.8 | 29.1, 128 43.2 | 43.9.
// The workgroups that repeat this work should all be resident: up to three per compute unit at r c_z = 16, two at 32 and 64, one from 256
// on (of 128 it pays at any number).  B H = 48, L = 256, 768 workgroups: r c_z = 16 1 : 0.82 (1024 1.11), 32 34.1 | 42.7, 64 1 : 1.24, 128 1 : 0.91;
// B H = 128, L = 64, 512: 32 1 : 0.65, 64 1 : 0.67; r c_z = 512, B H = 64, L = 64, 256 1 : 0.97, B H = 192, L = 33, 576 72 | 78.
bool f32_one_launch(int L, int DZ, long long workgroups)
{
    const int resident = DZ == 16 ? 3 : DZ <= 64 ? 2 : DZ == 128 ? 4 : 1;
    return L <= (DZ <= 128 ? 256 : 64) && workgroups <= 256 * resident;
}

size_t f32_lds_bytes(const F32Geom &g, int KS) { return ((size_t)KS * 16 * g.S + KS * 16 + 128) * sizeof(float); }

template <int NCH, int NT, bool EXACT, int RG, bool PACK = false>
hipError_t launch_attn(const F32Params &p, hipStream_t stream)
{
    const int KS = 4 / RG;
    const size_t lds = f32_lds_bytes(p.g, KS);
    static LdsLimit lim;
    const hipError_t e = raise_lds_limit(lim, (const void *)fipa_attn_f32_kernel<NCH, NT, EXACT, RG, PACK>, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fipa_attn_f32_kernel<NCH, NT, EXACT, RG, PACK>), dim3((p.n_units + 7) / 8 * 8), dim3(256), lds, stream, p);
    return hipGetLastError();
}

}  // namespace

size_t f32_forward_workspace_min(const fipa_desc &d) { return f32_layout(d).total; }

size_t f32_forward_workspace(const fipa_desc &d)
{
    const size_t least = f32_forward_workspace_min(d), split = f32_split_workspace(d);
    return split > least ? split : least;
}

hipError_t f32_forward(const fipa_desc &d, const FwdArgs &a, void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (f32_split_applies(d, a.mask != nullptr) && ws_bytes >= f32_split_workspace_min(d)) return f32_split_forward(d, a, ws, ws_bytes, stream);
    const F32Layout w = f32_layout(d);
    char *base = static_cast<char *>(ws);
    F32Params p;
    p.q = (const float *)a.q; p.k = (const float *)a.k; p.v = (const float *)a.v;
    p.q_pts = (const float *)a.q_pts; p.k_pts = (const float *)a.k_pts; p.v_pts = (const float *)a.v_pts;
    p.z1 = (const float *)a.z1; p.z2 = (const float *)a.z2;
    p.rot = a.rot; p.trans = a.trans; p.gamma = a.gamma; p.w_b = a.w_b; p.mask = a.mask; p.cu = nullptr;
    p.HR = reinterpret_cast<float *>(base + w.HR);
    p.cen = reinterpret_cast<float *>(base + w.cen);
    p.kvlen = reinterpret_cast<int *>(base + w.kvlen);
    p.o = a.o; p.o_pts = a.o_pts; p.o_pair = a.o_pair; p.lse = a.lse;
    p.B = d.B; p.L = d.L; p.H = d.H; p.c = d.c; p.Pq = d.Pq; p.Pv = d.Pv; p.cz = d.cz; p.r = d.r;
    p.DZ = d.r * d.cz;
    const bool exact = f32_exact(d);
    p.g = f32_geom(d.c, d.Pq, d.Pv, p.DZ, exact);
    p.vec = d.c % 4 == 0 && d.cz % 4 == 0;
    p.w_L = d.w_L; p.w_C = d.w_C; p.qk_scale = d.qk_scale;

    StageTimer timer(stream);
    timer.begin(0);
    const long long bh = (long long)d.B * d.H;
    // 16-row workgroups where 32-row ones would not give every CU two (the widest records fit LDS only as 32-key tiles)
    const bool small = bh * ((d.L + 31) / 32) < 512 && f32_lds_bytes(p.g, 4) <= 160 * 1024;
    const bool one_launch = exact && small && f32_one_launch(d.L, p.DZ, bh * ((d.L + 15) / 16));
    if (!one_launch) {
        const unsigned per_head = ((unsigned)d.L * (p.g.HRW / 4) + 255u) / 256u;
        hipLaunchKernelGGL(fipa_pack_f32_kernel, dim3(d.H * per_head, d.B), dim3(256), 0, stream, p);
    }
    timer.end(0);

    timer.begin(1);  // the fp32 kernel contains the epilogue; stage 2 stays empty
    p.n_rt = small ? (d.L + 15) / 16 : (d.L + 31) / 32;
    p.n_units = (int)(bh * p.n_rt);
    hipError_t e;
#define FIPA_F32_RUN(NCH, NT, EXACT) \
    e = one_launch ? launch_attn<NCH, NT, EXACT, 1, EXACT>(p, stream) \
        : small    ? launch_attn<NCH, NT, EXACT, 1>(p, stream) : launch_attn<NCH, NT, EXACT, 2>(p, stream)
    if (exact && p.g.nch == 2) FIPA_F32_RUN(2, 4, true);
    else if (exact && p.g.nch == 3) FIPA_F32_RUN(3, 5, true);
    else if (exact && p.g.nch == 5) FIPA_F32_RUN(5, 7, true);
    else if (exact && p.g.nch == 9) FIPA_F32_RUN(9, 11, true);
    else if (exact && p.g.nch == 17) FIPA_F32_RUN(17, 19, true);
    else if (exact && p.g.nch == 33) FIPA_F32_RUN(33, 35, true);
    else if (p.g.nt <= 8) FIPA_F32_RUN(8, 8, false);
    else if (p.g.nt <= 20) FIPA_F32_RUN(20, 20, false);
    else FIPA_F32_RUN(37, 37, false);
#undef FIPA_F32_RUN
    timer.end(1);
    return e;
}

}  // namespace fipa
