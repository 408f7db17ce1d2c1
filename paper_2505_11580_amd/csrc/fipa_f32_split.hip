// fp32 forward of AlphaFold2's head shape on the bf16 matrix instructions.  Every operand of the two products is the exact
// sum of three bf16 numbers (8 + 8 + 8 bits of a float's 24), and a product of two such sums is taken as its six largest
// products of parts (Henry, Tang, Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision
// Computations", 2019).  The three left out are at most 2^-24 of |a| |b| together, about the rounding of an fp32 product.
// The squared distances stay explicit fp32 differences on the vector ALU, the softmax is fp32 throughout.
//
// Bound: bf16 matrix pipe, six instructions for one of the fp32 pipe's at 16 times its rate.  A wave owns 32 queries, whose
// split features (51 fragments at r c_z = 256) stay in registers beside the 32 x (64 + r c_z) accumulator, one wave per SIMD;
// an operand read from LDS feeds one to three instructions, so that LDS is half busy.  Key blocks of 32 residues come by
// direct loads into two stages, in the order and swizzle in which the pack kernel left them.  Where the tiles of 128 queries
// fill half of the compute units or less, the keys are cut into ranges whose sums a small kernel adds.
// B = 2, L = 1024, H = 12, r c_z = 256: 448 us on the fp32 matrix instructions (fipa_f32.hip) -> 171; 4.9 us per key block, of
// which the 222 matrix instructions take 3.8 at the clock that they leave (17.3 ns each), 32 us before and behind the loop.
// Distance from float64 (2-norm, o | o_pts | o_pair | lse): 4.50e-7 | 2.40e-6 | 4.49e-7 | 3.78e-7 -> 4.40e-7 | 2.39e-6 | 4.43e-7 |
// 3.73e-7; no larger at any of the sizes compared (450 to 2048 residues, r c_z = 32 to 256).
#include "fipa_gfx950.h"
#include "fipa_f32.h"

#include <algorithm>

namespace fipa {

namespace {

// A key block of 32 residues as it lies in memory and in LDS (bytes): three planes of z2 [32][DZ], then per head three planes
// of k [32][16] and of v | Vg | 0 [32][64], Kg [32][12] in fp32, and 0 or -inf per key.  16-byte slots of the planes with rows
// of 128 bytes and more are swizzled (swz_z, swz_h).
template <int DZ>
struct Fs {
    static constexpr int KSZ = DZ / 16, KS = KSZ + 1, NB = DZ / 32, NA = NB + 2;
    static constexpr int ZROW = 2 * DZ, ZP = 32 * ZROW, ZBLK = 3 * ZP;
    static constexpr int K = 0, KP = 1024, V = 3 * KP, VP = 4096, G = V + 3 * VP, M = G + 1536, HBLK = 17408;  // (M + 128, to whole KiB)
    static constexpr int STAGE = ZBLK + HBLK;
    static constexpr int kDma = (ZBLK + 4095) / 4096 + HBLK / 4096 + 1;  // 1 KiB pieces that a wave requests of a block
    static constexpr bool apart(int cb) { return cb >= NB || DZ == 32; }  // column blocks that are summed apart for 16 keys
    static constexpr int RS = DZ + 44;  // floats of a row of results: pair part, v | Vg (40), reference and sum
    static constexpr int kLds = 2 * STAGE > 128 * RS * 4 ? 2 * STAGE : 128 * RS * 4;
};
constexpr int kHeadBlock = 17408;

struct SplitParams {
    const float *q, *k, *v, *q_pts, *k_pts, *v_pts, *z1, *z2, *rot, *trans, *gamma, *w_b;
    const uint8_t *mask;
    const int *cu;  // always null here (user_row and batch_reference want the member)
    char *zb, *hb;  // key blocks: [B][n_kb][ZBLK], [B * H][n_kb][HBLK]
    float *cen, *part;
    int *kvlen;
    float *o, *o_pts, *o_pair, *lse;
    int B, L, H, cz, r, DZ;
    int n_kb, n_rt, n_parts, n_units;
    float w_L, w_C, qk_scale;
};

// x = hi + mid + lo, each a bf16 to the nearest: |mid| is at most 2^-8 of |x|, |lo| 2^-17.  (The largest floats would round up to
// infinity: the first part stops at the largest bf16.)
__device__ __forceinline__ void split3(float x, unsigned &hi, unsigned &mid, unsigned &lo)
{
    constexpr float kMax = 3.3895313892515355e38f;
    const float a = fabsf(x) <= 3.4028234663852886e38f ? fminf(fmaxf(x, -kMax), kMax) : x;
    const __bf16 h = (__bf16)a;
    const float r1 = x - (float)h;
    const __bf16 m = (__bf16)r1;
    const __bf16 l = (__bf16)(r1 - (float)m);
    hi = __builtin_bit_cast(unsigned short, h);
    mid = __builtin_bit_cast(unsigned short, m);
    lo = __builtin_bit_cast(unsigned short, l);
}

// Swizzle of the 16-byte slots of row `row` of a z2 plane: rows of 256 bytes and more, of 128 and of 64 bytes.
__device__ __forceinline__ int swz_row(int DZ, int row) { return DZ >= 128 ? swz_z(row) : DZ == 64 ? swz_h(row) : (row >> 2) & 3; }

// Eight floats -> one 16-byte slot of each plane.
__device__ __forceinline__ void split_slot(const float (&x)[8], u32x4 (&out)[3])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        unsigned a[3], b[3];
        split3(x[2 * e], a[0], a[1], a[2]);
        split3(x[2 * e + 1], b[0], b[1], b[2]);
#pragma unroll
        for (int s = 0; s < 3; ++s) out[s][e] = a[s] | (b[s] << 16);
    }
}

// Key blocks: workgroups 0 .. H n_kb - 1 of a batch element take a head's block each, the others 256 slots of the z2 planes.
// Masked residues and those past the chain's end are zero.
__global__ __launch_bounds__(256) void fipa_pack_split_kernel(SplitParams p)
{
    const int b = blockIdx.y;
    int unit = blockIdx.x;
    if (unit >= p.H * p.n_kb) {  // z2
        unit -= p.H * p.n_kb;
        const int per_row = p.DZ / 8, idx = unit * 256 + threadIdx.x;
        const int j = idx / per_row, slot = idx - j * per_row;
        if (j >= 32 * p.n_kb) return;
        const size_t u = (size_t)b * p.L + j;
        float x[8] = {};
        if (j < p.L && (p.mask ? p.mask[u] != 0 : true)) {
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(p.z2 + u * p.DZ + 8 * slot);
            const f32x4 hi = *reinterpret_cast<const f32x4 *>(p.z2 + u * p.DZ + 8 * slot + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[e] = lo[e];
                x[4 + e] = hi[e];
            }
        }
        u32x4 out[3];
        split_slot(x, out);
        const int row = j & 31, at = slot ^ swz_row(p.DZ, row);
        const int plane = 64 * p.DZ;
        char *dst = p.zb + ((size_t)b * p.n_kb + j / 32) * (3 * plane) + row * (2 * p.DZ) + 16 * at;
#pragma unroll
        for (int s = 0; s < 3; ++s) *reinterpret_cast<u32x4 *>(dst + s * plane) = out[s];
        return;
    }
    using F = Fs<64>;  // (the head's part of a block is the same for all widths)
    float cen[3];
    int kv;
    batch_reference(p, b, cen, kv);
    if (unit == 0 && threadIdx.x == 0) {
        for (int a = 0; a < 3; ++a) p.cen[4 * b + a] = cen[a];
        p.cen[4 * b + 3] = 0.f;
        p.kvlen[b] = kv;
    }
    const int h = unit / p.n_kb, kb = unit - h * p.n_kb;
    char *blk = p.hb + (((size_t)b * p.H + h) * p.n_kb + kb) * kHeadBlock;
    // pieces of a key: 0-1 k, 2-3 v, 4-6 Vg, 7-9 zero columns, 10-12 Kg, 13 the mask
#pragma unroll 2
    for (int idx = threadIdx.x; idx < 32 * 14; idx += 256) {
        const int row = idx / 14, x0 = idx - 14 * row, j = 32 * kb + row;
        const size_t u = (size_t)b * p.L + min(j, p.L - 1), hrow = u * p.H + h;
        const bool ok = j < p.L && (p.mask ? p.mask[u] != 0 : true);
        if (x0 == 13) {
            *reinterpret_cast<float *>(blk + F::M + 4 * row) = ok ? 0.f : -INFINITY;
            continue;
        }
        float x[8] = {};
        if (ok && x0 < 4) {
            const float *src = (x0 < 2 ? p.k : p.v) + hrow * 16 + 8 * (x0 & 1);
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = src[e];
        } else if (ok && (x0 < 7 || x0 >= 10)) {
            const float *R = p.rot + u * 9, *t = p.trans + u * 3;
            const float *src = x0 < 7 ? p.v_pts + hrow * 24 : p.k_pts + hrow * 12;
            const int y0 = x0 < 7 ? 8 * (x0 - 4) : 4 * (x0 - 10);
#pragma unroll
            for (int e = 0; e < 8; ++e) {  // (of Kg the last four are not used)
                const int y = x0 < 7 ? y0 + e : y0 + (e & 3), pp = y / 3, a = y - 3 * pp;
                const float *l = src + 3 * pp;
                x[e] = R[3 * a] * l[0] + R[3 * a + 1] * l[1] + R[3 * a + 2] * l[2] + (t[a] - cen[a]);
            }
        }
        if (x0 >= 10) {
            *reinterpret_cast<f32x4 *>(blk + F::G + 48 * row + 16 * (x0 - 10)) = (f32x4){x[0], x[1], x[2], x[3]};
            continue;
        }
        u32x4 out[3];
        split_slot(x, out);
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            char *dst = x0 < 2 ? blk + F::K + s * F::KP + 32 * row + 16 * x0 : blk + F::V + s * F::VP + 128 * row + 16 * ((x0 - 2) ^ swz_h(row));
            *reinterpret_cast<u32x4 *>(dst) = out[s];
        }
    }
}

__device__ __forceinline__ f32x16 mfma(const bf16x8 &a, const bf16x8 &b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The value of the lane 32 away.
__device__ __forceinline__ float other_half(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}

// Two weights -> their three parts, packed.
__device__ __forceinline__ void split_pair(float a, float b, unsigned (&out)[3])
{
    const bf16x2 h = __builtin_convertvector((f32x2){a, b}, bf16x2);
    const unsigned hu = __builtin_bit_cast(unsigned, h);
    const float a1 = a - __uint_as_float(hu << 16), b1 = b - __uint_as_float(hu & 0xFFFF0000u);
    const bf16x2 m = __builtin_convertvector((f32x2){a1, b1}, bf16x2);
    const unsigned mu = __builtin_bit_cast(unsigned, m);
    const float a2 = a1 - __uint_as_float(mu << 16), b2 = b1 - __uint_as_float(mu & 0xFFFF0000u);
    out[0] = hu;
    out[1] = mu;
    out[2] = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a2, b2}, bf16x2));
}

// Floats of a row of partial results: o (16), the points (24), o_pair (cz), reference and sum of the weights, to 16 bytes.
__host__ __device__ __forceinline__ int part_row(int cz) { return 44 + cz; }

// What a row's head part (v and the global points' sums, `head(x)`) gives: 16 threads, x0 = 0 .. 15.
template <class F>
__device__ __forceinline__ void finish_row(const SplitParams &p, int b, int h, int i, int x0, const float *cen, float m, float l, F &&head)
{
    const size_t ui = (size_t)b * p.L + min(i, p.L - 1), ro = ui * p.H + h;
    const bool valid = (p.mask ? p.mask[ui] != 0 : true) && l > 0.f;
    const float *R = p.rot + ui * 9, *t = p.trans + ui * 3;
    float val[2] = {0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int idx = u == 0 ? x0 : 16 + (x0 & 7), pp = idx / 3, x = idx - 3 * pp;
#pragma unroll
        for (int y = 0; y < 3; ++y) val[u] += R[3 * y + x] * (head(16 + 3 * pp + y) - (t[y] - cen[y]));
    }
    const float o = head(x0);
    if (i >= p.L) return;
    p.o[ro * 16 + x0] = valid ? o : 0.f;
    p.o_pts[ro * 24 + x0] = valid ? val[0] : 0.f;
    if (x0 < 8) p.o_pts[ro * 24 + 16 + x0] = valid ? val[1] : 0.f;
    if (p.lse && x0 == 0) p.lse[((size_t)b * p.H + h) * p.L + i] = valid ? kLn2 * (m + __log2f(l)) : 0.f;
}

// A wave's rows `again` against the keys j0 .. j1 - 1 from the inputs, in fp32 on the vector ALU: a lane takes its row and every second key,
// and leaves what the tile left of the row in LDS (`out`, also the room for the row's features).  For rows with an infinite operand, which
// six products of parts do not carry (an infinity has no second part, and a product far beyond the largest float leaves parts of
// either sign): an infinite logit or value then gives what fp32 arithmetic gives.  B = 2, L = 1024, H = 12, r c_z = 256, one infinite value:
// 5.8 ms (one row after the other, a lane per key: 50; without it 0.17).
template <int DZ>
__device__ __forceinline__ void direct_rows(const SplitParams &p, int b, int h, int i, unsigned again, int j0, int j1, const float *cen, bool whole,
                                            float *out)
{
    constexpr int NC = (DZ + 40) / 4;
    const int hf = (threadIdx.x >> 5) & 1;
    const bool mine = (again >> (threadIdx.x & 31) & 1u) != 0u;
    const size_t row0 = (size_t)b * p.L, ui = row0 + i;
    const float sc = kLog2e * p.w_L * p.qk_scale, bz = kLog2e * p.w_L, coef = kLog2e * 0.5f * p.gamma[h] * p.w_L * p.w_C;
    if (mine && hf == 0) {
        const float *q = p.q + (ui * p.H + h) * 16, *z1 = p.z1 + ui * DZ, *wb = p.w_b + (size_t)h * p.cz;
#pragma unroll 4
        for (int x = 0; x < DZ + 16; ++x) out[x] = x < 16 ? sc * q[x] : bz * wb[(x - 16) & (p.cz - 1)] * z1[x - 16];
    }
    asm volatile("" ::: "memory");  // (the LDS accesses of a wave execute in order)
    auto point = [&](size_t u, const float *pts, int x) {  // global coordinate x of a residue's points
        const float *R = p.rot + u * 9 + 3 * (x % 3), *l = pts + x / 3 * 3;
        return R[0] * l[0] + R[1] * l[1] + R[2] * l[2] + (p.trans[u * 3 + x % 3] - cen[x % 3]);
    };
    float qg[12];
#pragma unroll
    for (int x = 0; x < 12; ++x) qg[x] = point(ui, p.q_pts + (ui * p.H + h) * 12, x);
    float m = -INFINITY, l = 0.f;
    f32x4 acc[NC];
#pragma unroll
    for (int x = 0; x < NC; ++x) acc[x] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int t = j0; t < j1; t += 2) {
        const int j = t + hf;
        const size_t u = row0 + min(j, p.L - 1), hrow = u * p.H + h;
        if (j >= j1 || (p.mask ? p.mask[u] == 0 : false)) continue;
        const float *k = p.k + hrow * 16, *z2 = p.z2 + u * DZ, *v = p.v + hrow * 16;
        float s = 0.f, dist = 0.f;
#pragma unroll
        for (int x = 0; x < 16; x += 4) {
            const f32x4 f = *reinterpret_cast<const f32x4 *>(out + x), y = *reinterpret_cast<const f32x4 *>(k + x);
            for (int e = 0; e < 4; ++e) s += f[e] * y[e];
        }
#pragma unroll 8
        for (int x = 0; x < DZ; x += 4) {
            const f32x4 f = *reinterpret_cast<const f32x4 *>(out + 16 + x), y = *reinterpret_cast<const f32x4 *>(z2 + x);
            for (int e = 0; e < 4; ++e) s += f[e] * y[e];
        }
#pragma unroll
        for (int x = 0; x < 12; ++x) {
            const float df = qg[x] - point(u, p.k_pts + hrow * 12, x);
            dist += df * df;
        }
        s -= coef * dist;
        if (s > m) {
            const float alpha = __builtin_amdgcn_exp2f(m - s);
            l *= alpha;
            m = s;
#pragma unroll
            for (int x = 0; x < NC; ++x) acc[x] *= alpha;
        }
        const float w = __builtin_amdgcn_exp2f(s - (m == -INFINITY ? 0.f : m));
        l += w;
#pragma unroll
        for (int x = 0; x < DZ / 4; ++x) acc[x] += w * *reinterpret_cast<const f32x4 *>(z2 + 4 * x);
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[DZ / 4 + x] += w * *reinterpret_cast<const f32x4 *>(v + 4 * x);
#pragma unroll
        for (int x = 0; x < 24; ++x) acc[DZ / 4 + 4 + x / 4][x % 4] += w * point(u, p.v_pts + hrow * 24, x);
    }
    const float m_all = fmaxf(m, other_half(m)), wm = __builtin_amdgcn_exp2f(m - (m_all == -INFINITY ? 0.f : m_all));
    l *= wm;
    l += other_half(l);
    const float scale = !whole ? 1.f : l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int x = 0; x < NC; ++x) {
        f32x4 a = acc[x] * wm;
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = scale * (a[e] + other_half(a[e]));
        if (mine && hf == 0) *reinterpret_cast<f32x4 *>(out + 4 * x) = a;
    }
    if (mine && hf == 0) *reinterpret_cast<f32x2 *>(out + DZ + 40) = (f32x2){m_all, l};
}

constexpr float kRaise = 1.f;  // log2 units: an exponent of up to 1 is rounded no worse than one below 0 (30: lse 4.17e-7 from float64, 1: 3.73e-7)

template <int DZ>
__global__ __launch_bounds__(256, DZ == 32 ? 2 : 1) void fipa_attn_f32_split_kernel(SplitParams p)
{
    using F = Fs<DZ>;
    extern __shared__ __attribute__((aligned(256))) char smem[];

    const int per = (p.n_units + 7) / 8;  // an XCD gets neighbouring units: it shares their keys in its L2
    const int unit = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if ((int)(blockIdx.x / 8) >= per || unit >= p.n_units) return;
    const int part = unit % p.n_parts, tile = unit / p.n_parts;
    const int bh = tile / p.n_rt, b = bh / p.H, h = bh - b * p.H;
    const int i_wg = (tile - bh * p.n_rt) * 128;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, n = lane & 31, hf = lane >> 5;
    const int L = p.L, H = p.H;
    const int kvlen = __builtin_amdgcn_readfirstlane(p.kvlen[b]);
    float cen[3];
    for (int a = 0; a < 3; ++a) cen[a] = p.cen[4 * b + a];

    // this part's key blocks lo .. lo + len - 1, from the one nearest the tile's residues away from them
    const int nkb = i_wg < kvlen ? (kvlen + 31) / 32 : 0;  // (a tile past the last valid residue has no work)
    const int lo = (int)((long long)nkb * part / p.n_parts), len = (int)((long long)nkb * (part + 1) / p.n_parts) - lo;
    const int diag = i_wg / 32, dir = diag >= lo + len ? -1 : 1;
    int blk = max(lo, min(diag, lo + len - 1));

    const char *zsrc = p.zb + (size_t)b * p.n_kb * F::ZBLK, *hsrc = p.hb + (size_t)bh * p.n_kb * F::HBLK;
    const unsigned lds0 = lds_address(smem);
    struct Source {
        u32x4 z, h;
    };
    auto source = [&](int kb) { return Source{buffer_desc(zsrc + (size_t)kb * F::ZBLK), buffer_desc(hsrc + (size_t)kb * F::HBLK)}; };
    auto request = [&](const Source &s, int stage, auto c_) {
        constexpr int c = decltype(c_)::value, nz = (F::ZBLK + 4095) / 4096, nh = F::HBLK / 4096;
        const unsigned dst = lds0 + stage * F::STAGE;
        int voff;  // 16 * lane, formed again each time: a register kept for it would be spilled
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0\n\tv_lshlrev_b32 %0, 4, %0" : "=v"(voff));
        if constexpr (c < nz) {
            const int piece = min(4 * c + wave, F::ZBLK / 1024 - 1);  // (surplus waves: the last piece again)
            dma16b(s.z, voff, piece * 1024, dst + piece * 1024);
        }
        else if constexpr (c < nz + nh)
            dma16b(s.h, voff, (4 * (c - nz) + wave) * 1024, dst + F::ZBLK + (4 * (c - nz) + wave) * 1024);
        else  // (every wave: the same bytes to the same place)
            dma16b(s.h, voff, 4 * nh * 1024, dst + F::ZBLK + 4 * nh * 1024);
    };
    static_assert(F::ZBLK % 1024 == 0 && F::HBLK % 4096 == 1024);
    if (len > 0) {
        const Source src = source(blk);
        static_for<F::kDma>([&](auto c) { request(src, 0, c); });
    }

    // query side: scaled scalars and factor bias vector b^{h1} (log2 units) in three parts, global points
    const int iq = min(i_wg + 32 * wave + n, L - 1);
    const size_t urow = (size_t)b * L + iq, row = urow * H + h;
    bf16x8 qf[F::KS][3];
    {
        // (all rows of z1 in flight at once; the scale vector through the space of the other stage)
        float *const wl = reinterpret_cast<float *>(smem + F::STAGE);
        const float sc = kLog2e * p.w_L * p.qk_scale, bz = kLog2e * p.w_L;
        const float *q = p.q + row * 16 + 8 * hf, *z1 = p.z1 + urow * DZ + 8 * hf;
        f32x4 zr[F::KS][2];
#pragma unroll
        for (int ks = 0; ks < F::KS; ++ks)
#pragma unroll
            for (int e = 0; e < 2; ++e) zr[ks][e] = *reinterpret_cast<const f32x4 *>(ks == 0 ? q + 4 * e : z1 + 16 * (ks - 1) + 4 * e);
        if ((int)threadIdx.x < p.cz) wl[threadIdx.x] = bz * p.w_b[(size_t)h * p.cz + threadIdx.x];
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wg_barrier();
#pragma unroll
        for (int ks = 0; ks < F::KS; ++ks) {
            unsigned s[4][3];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                f32x4 val;
                if (ks == 0)
                    val = sc * zr[ks][e];
                else
                    val = *reinterpret_cast<const f32x4 *>(wl + ((16 * (ks - 1) + 4 * e + 8 * hf) & (p.cz - 1))) * zr[ks][e];
                split_pair(val[0], val[1], s[2 * e]);
                split_pair(val[2], val[3], s[2 * e + 1]);
            }
#pragma unroll
            for (int t = 0; t < 3; ++t) qf[ks][t] = __builtin_bit_cast(bf16x8, (u32x4){s[0][t], s[1][t], s[2][t], s[3][t]});
        }
    }
    float qg[12];
    {
        const float *R = p.rot + urow * 9, *t = p.trans + urow * 3, *src = p.q_pts + row * 12;
#pragma unroll
        for (int x = 0; x < 12; ++x) {
            const int pp = x / 3, a = x % 3;
            qg[x] = R[3 * a] * src[3 * pp] + R[3 * a + 1] * src[3 * pp + 1] + R[3 * a + 2] * src[3 * pp + 2] + (t[a] - cen[a]);
        }
    }
    const float coef = kLog2e * 0.5f * p.gamma[h] * p.w_L * p.w_C;
    if constexpr (DZ >= 128) {
#pragma unroll
        for (int ks = 0; ks < F::KS; ++ks)
#pragma unroll
            for (int t = 0; t < 3; ++t) asm volatile("" : "+a"(qf[ks][t]));
    }

    float m = -INFINITY, l = 0.f;
    f32x16 acc[F::NA];
#pragma unroll
    for (int t = 0; t < F::NA; ++t)
#pragma unroll
        for (int x = 0; x < 16; ++x) acc[t][x] = 0.f;

    // lane addresses within a stage
    constexpr bool kWide = DZ >= 128;
    const int at_z = n * F::ZROW + 16 * (hf ^ swz_row(DZ, n));  // rows of the z2 planes, ^ 32 ks
    const int at_k = F::ZBLK + F::K + 32 * n + 16 * hf;
    const int j4 = (lane >> 2) & 3, gq = (lane >> 4) & 1;  // transposing reads: row 4 hf + j4, 16 columns 16 gq
    int at_vz[2], at_vh[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int r0 = 8 * x + 4 * hf + j4, c0 = 2 * gq + ((lane >> 1) & 1), in = 8 * (lane & 1);
        at_vz[x] = r0 * F::ZROW + 16 * (c0 ^ swz_row(DZ, r0)) + in;
        at_vh[x] = F::ZBLK + F::V + r0 * 128 + 16 * (c0 ^ swz_h(r0)) + in;
    }
    const int at_g = F::ZBLK + F::G + 4 * hf * 48, at_m = F::ZBLK + F::M + 16 * hf;

    for (int it = 0; it < len; ++it) {
        wait_and_barrier<0>();  // this block has landed, and everyone has left the other stage
        const char *st = smem + (it & 1) * F::STAGE;
        if (it + 1 < len) {  // (a block more is requested after the last one, the last one again: no branches in the steps)
            blk += dir;
            if (blk == lo + len) blk = lo;
        }
        const Source next = source(blk);
        // (addresses of this stage; opaque, or their swizzled forms would be kept in registers across the blocks)
        int zk = at_z + (it & 1) * F::STAGE, zv[2], hv[2];
        asm volatile("" : "+v"(zk));
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            zv[x] = at_vz[x] + (it & 1) * F::STAGE;
            hv[x] = at_vh[x] + (it & 1) * F::STAGE;
            asm volatile("" : "+v"(zv[x]), "+v"(hv[x]));
        }
        auto load_k = [&](int ks, bf16x8 (&a)[3]) {
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const char *src = ks == 0 ? st + at_k + t * F::KP
                                          : smem + (zk ^ (32 * ((ks - 1) & (DZ >= 128 ? 7 : DZ / 16 - 1)))) + t * F::ZP + (kWide ? 256 * ((ks - 1) / 8) : 0);
                a[t] = *reinterpret_cast<const bf16x8 *>(src);
            }
        };
        auto load_v = [&](int kk, int cb, bf16x8 (&a)[3]) {
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const char *src[2];
#pragma unroll
                for (int x = 0; x < 2; ++x)
                    src[x] = cb < F::NB ? smem + (zv[x] ^ (64 * (cb & (DZ >= 128 ? 3 : DZ / 32 - 1)))) + t * F::ZP + 16 * kk * F::ZROW + (kWide ? 256 * (cb / 4) : 0)
                                        : smem + (hv[x] ^ (64 * (cb - F::NB))) + t * F::VP + 16 * kk * 128;
                a[t] = lds_read_tr(src[0], src[1]);
            }
        };

        // S^T of the block, small products apart; squared distances beside them, each key's coordinates read a step ahead
        f32x16 s0, s1;
#pragma unroll
        for (int x = 0; x < 16; x += 4) {  // (the small products start from the mask)
            const f32x4 mb = *reinterpret_cast<const f32x4 *>(st + at_m + 8 * x);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s0[x + e] = 0.f;
                s1[x + e] = mb[e];
            }
        }
        float dist[16];
        bf16x8 a[2][3];
        constexpr int kPer = (16 + F::KS - 1) / F::KS;  // keys per step
        f32x4 kg[kPer][3];
        auto load_g = [&](int ks) {
#pragma unroll
            for (int y = 0; y < kPer; ++y) {
                const int x = ks * kPer + y;
#pragma unroll
                for (int z = 0; z < 3; ++z)
                    if (x < 16) kg[y][z] = *reinterpret_cast<const f32x4 *>(st + at_g + (8 * (x >> 2) + (x & 3)) * 48 + 16 * z);
            }
        };
        load_k(0, a[0]);
        load_g(0);
        static_for<F::KS>([&](auto ks_) {
            constexpr int ks = decltype(ks_)::value;
            const bf16x8(&c)[3] = a[ks & 1];
            // One product per slot: the operands of the next step are read behind the first, the distances are spread over the last
            // four, and the coordinates they used are replaced by the next.
            float d[kPer] = {};
            auto slot = [&](auto n_) {
                constexpr int n = decltype(n_)::value;
                if constexpr (n == 0) s1 = mfma(c[2], qf[ks][0], s1);
                if constexpr (n == 1) s1 = mfma(c[1], qf[ks][1], s1);
                if constexpr (n == 2) s1 = mfma(c[0], qf[ks][2], s1);
                if constexpr (n == 3) s1 = mfma(c[1], qf[ks][0], s1);
                if constexpr (n == 4) s1 = mfma(c[0], qf[ks][1], s1);
                if constexpr (n == 5) s0 = mfma(c[0], qf[ks][0], s0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (n == 0 && ks + 1 < F::KS) load_k(ks + 1, a[(ks + 1) & 1]);
                if constexpr (n == 0 && ks + 1 == F::KS) load_v(0, 0, a[(ks + 1) & 1]);
                if constexpr (n == 1) {  // the next block's pieces, spread over the steps
                    constexpr int kStep = (F::kDma + F::KS - 1) / F::KS;
                    static_for<kStep>([&](auto c_) {
                        constexpr int piece = ks * kStep + decltype(c_)::value;
                        if constexpr (piece < F::kDma) request(next, (it + 1) & 1, std::integral_constant<int, piece>{});
                    });
                }
                if constexpr (n >= 2) {
#pragma unroll
                    for (int y = 0; y < kPer; ++y)
#pragma unroll
                        for (int z = 3 * (n - 2); z < 3 * (n - 1); ++z) {
                            const float df = qg[z] - kg[y][z / 4][z % 4];
                            d[y] += df * df;
                        }
                }
                if constexpr (n == 5) {
#pragma unroll
                    for (int y = 0; y < kPer; ++y)
                        if (ks * kPer + y < 16) dist[ks * kPer + y] = d[y];
                    if constexpr (ks + 1 < F::KS) load_g(ks + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            static_for<6>(slot);
        });

        float s[16];
        float mt = -INFINITY;
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            s[x] = (s0[x] + s1[x]) - coef * dist[x];
            mt = fmaxf(mt, s[x]);
        }
        mt = fmaxf(mt, other_half(mt));
        if (__any(mt > m + kRaise)) {
            const float m_new = mt > m + kRaise ? mt : m;
            const float alpha = m_new == m ? 1.f : __builtin_amdgcn_exp2f(m - m_new);
            l *= alpha;
            m = m_new;
#pragma unroll
            for (int t = 0; t < F::NA; ++t) acc[t] *= alpha;
        }
        const float m_use = m == -INFINITY ? 0.f : m;
        unsigned pw[2][3][4];  // weights of keys 16 kk ..: three parts, four pairs
        auto weights = [&](int kk, int e) {
            const float p0 = __builtin_amdgcn_exp2f(s[8 * kk + 2 * e] - m_use), p1 = __builtin_amdgcn_exp2f(s[8 * kk + 2 * e + 1] - m_use);
            l += p0 + p1;
            unsigned t[3];
            split_pair(p0, p1, t);
#pragma unroll
            for (int x = 0; x < 3; ++x) pw[kk][x][e] = t[x];
        };
#pragma unroll
        for (int e = 0; e < 4; ++e) weights(0, e);
        __builtin_amdgcn_sched_barrier(0);

        // O^T += V^T P^T; the head's columns (points, whose sums cancel against the frame's origin; at r c_z = 32 all) are summed apart for 16 keys
        // (o_pts 2.58e-6 from float64 where only their small products were, 2.39e-6 now)
        f32x16 small;
        static_for<2 * F::NA>([&](auto n_) {
            constexpr int nn = decltype(n_)::value, kk = nn / F::NA, cb = nn % F::NA;
            constexpr int at = (F::KS + nn) & 1;
            const bf16x8(&c)[3] = a[at];
            bf16x8 w[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) w[t] = __builtin_bit_cast(bf16x8, (u32x4){pw[kk][t][0], pw[kk][t][1], pw[kk][t][2], pw[kk][t][3]});
            constexpr int last = (nn + F::NA - 1) % F::NA;  // the column block of the step before
            f32x16 now;
            if constexpr (!F::apart(cb)) {
                now = acc[cb];
            } else {
#pragma unroll
                for (int x = 0; x < 16; ++x) now[x] = 0.f;
            }
            now = mfma(c[2], w[0], now);
            if constexpr (nn + 1 < 2 * F::NA) load_v((nn + 1) / F::NA, (nn + 1) % F::NA, a[at ^ 1]);
            now = mfma(c[1], w[1], now);
            now = mfma(c[0], w[2], now);
            now = mfma(c[1], w[0], now);
            now = mfma(c[0], w[1], now);
            if constexpr (nn > 0 && F::apart(last)) acc[last] += small;
            if constexpr (!F::apart(cb)) {
                acc[cb] = mfma(c[0], w[0], now);
            } else {
                small = mfma(c[0], w[0], now);
            }
            if constexpr (kk == 0) {  // (three column blocks at r c_z = 32)
                constexpr int per = (4 + F::NA - 1) / F::NA;
#pragma unroll
                for (int e = per * cb; e < per * (cb + 1) && e < 4; ++e) weights(1, e);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
            for (int x = 0; x < 5; ++x) {
                __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        acc[F::NA - 1] += small;
    }
    l += other_half(l);

    // Rows for direct_rows.  An infinite factor of a logit (with one of z2 as a value too) makes a row's sum of weights a NaN; an infinite
    // v or point the row's sum of that column, which a finite one of which twice is infinite can make an infinity.
    f32x4 odd = {l - l, 0.f, 0.f, 0.f};  // 0, or NaN
#pragma unroll
    for (int x = 0; x < 20; ++x) odd[x & 3] = fmaf(acc[F::NB + x / 16][x % 16], 0.f, odd[x & 3]);
    const float any_odd = (odd[0] + odd[1]) + (odd[2] + odd[3]);
    const int own = i_wg + 32 * wave + n;
    const unsigned again = (unsigned)__ballot(any_odd + other_half(any_odd) != 0.f && own < L && (p.mask ? p.mask[(size_t)b * L + own] != 0 : true));

    // the wave's rows through LDS: 16 lanes per row
    const bool whole = p.n_parts == 1;
    const float scale = !whole ? 1.f : l > 0.f ? 1.f / l : 0.f;
    float *const rows = reinterpret_cast<float *>(smem) + wave * (32 * F::RS);
    const int x0 = lane & 15, r4 = lane >> 4, prow = part_row(p.cz);
    float *const out_part = p.part + ((size_t)unit * 128 + 32 * wave) * prow;
    wait_vmem<0>();
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < F::NA; ++cb)
#pragma unroll
        for (int x = 0; x < (cb == F::NA - 1 ? 4 : 16); x += 4)  // (of the head's second block 8 columns are in use)
            *reinterpret_cast<f32x4 *>(rows + n * F::RS + 32 * cb + 2 * x + 4 * hf) =
                (f32x4){acc[cb][x], acc[cb][x + 1], acc[cb][x + 2], acc[cb][x + 3]} * scale;
    if (hf == 0) *reinterpret_cast<f32x2 *>(rows + n * F::RS + DZ + 40) = (f32x2){m, l};
    if (__builtin_expect(again != 0u, 0)) {
        // (the arguments by a pointer that is formed here: kept for this they would take scalar registers through the loop)
        uint64_t args = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        direct_rows<DZ>(*reinterpret_cast<const SplitParams *>(args), b, h, min(own, L - 1), again, 32 * lo, min(32 * (lo + len), L), cen, whole,
                        rows + n * F::RS);
    }
    __syncthreads();
#pragma unroll 2
    for (int it = 0; it < 8; ++it) {
        const int rl = 4 * it + r4, i = i_wg + 32 * wave + rl;
        const size_t ui = (size_t)b * L + min(i, L - 1);
        const float *u = rows + rl * F::RS, *hr = u + DZ, *z1 = p.z1 + ui * DZ;
        f32x4 zr[DZ / 64 > 0 ? DZ / 64 : 1];
#pragma unroll
        for (int x = 0; x < DZ / 64; ++x) zr[x] = *reinterpret_cast<const f32x4 *>(z1 + 4 * x0 + 64 * x);
        bool valid = p.mask ? p.mask[ui] != 0 : true;
        float *dst = whole ? p.o_pair + (ui * H + h) * p.cz : out_part + (size_t)rl * prow + 40;
        if (whole) {
            valid = valid && hr[41] > 0.f;
            finish_row(p, b, h, i, x0, cen, hr[40], hr[41], [&](int x) { return hr[x]; });
        } else if (i < L) {
            float *ph = out_part + (size_t)rl * prow;
            for (int x = x0; x < 40; x += 16) ph[x] = hr[x];
            if (x0 < 2) ph[40 + p.cz + x0] = hr[40 + x0];
        }
        if (DZ >= 64 && p.cz >= 64) {  // a lane's columns of all ranks
            f32x4 val[DZ / 64 > 0 ? DZ / 64 : 1];
#pragma unroll
            for (int x = 0; x < DZ / 64; ++x) val[x] = zr[x] * *reinterpret_cast<const f32x4 *>(u + 4 * x0 + 64 * x);
            const int nc = p.cz / 64;
#pragma unroll
            for (int x = 1; x < DZ / 64; ++x) {
                const int to = x & (nc - 1);
#pragma unroll
                for (int y = 0; y < x; ++y)
                    if (y == to) val[y] += x >= nc ? val[x] : (f32x4){0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int x = 0; x < DZ / 64; ++x)
                if (x < nc && i < L) *reinterpret_cast<f32x4 *>(dst + 4 * x0 + 64 * x) = valid ? val[x] : (f32x4){0.f, 0.f, 0.f, 0.f};
        } else if (4 * x0 < p.cz && i < L) {
            f32x4 val = {0.f, 0.f, 0.f, 0.f};
            for (int d = 4 * x0; d < DZ; d += p.cz) val += *reinterpret_cast<const f32x4 *>(z1 + d) * *reinterpret_cast<const f32x4 *>(u + d);
            *reinterpret_cast<f32x4 *>(dst + 4 * x0) = valid ? val : (f32x4){0.f, 0.f, 0.f, 0.f};
        }
    }
}

// Rows of calls whose key range is split: the parts' sums added in the order of their keys.  16 threads per row.
template <int N>
__global__ __launch_bounds__(256) void fipa_merge_split_kernel(SplitParams p)
{
    const int tile = blockIdx.x >> 3, bh = tile / p.n_rt, b = bh / p.H, h = bh - b * p.H;
    const int rl = (blockIdx.x & 7) * 16 + (threadIdx.x >> 4), x0 = threadIdx.x & 15;
    const int i = (tile - bh * p.n_rt) * 128 + rl;
    if (i >= p.L) return;
    const int prow = part_row(p.cz);
    const float *src = p.part + ((size_t)tile * p.n_parts * 128 + rl) * prow;
    const size_t step = (size_t)128 * prow;
    // (all loads in flight at once: parts past the last are the last one again, with weight 0)
    const float *at[N];
    float m = -INFINITY, l = 0.f, w[N], ls[N];
#pragma unroll
    for (int s = 0; s < N; ++s) {
        at[s] = src + min(s, p.n_parts - 1) * step;
        w[s] = at[s][40 + p.cz];
        ls[s] = at[s][41 + p.cz];
        m = fmaxf(m, w[s]);
    }
    const float m_use = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int s = 0; s < N; ++s) {
        w[s] = s < p.n_parts ? __builtin_amdgcn_exp2f(w[s] - m_use) : 0.f;
        l += w[s] * ls[s];
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const float cen[3] = {p.cen[4 * b], p.cen[4 * b + 1], p.cen[4 * b + 2]};
    finish_row(p, b, h, i, x0, cen, m, l, [&](int x) {
        float v = 0.f;
#pragma unroll
        for (int s = 0; s < N; ++s) v += w[s] * at[s][x];
        return v * inv;
    });
    const size_t ui = (size_t)b * p.L + i;
    const bool valid = (p.mask ? p.mask[ui] != 0 : true) && l > 0.f;
    for (int d = 4 * x0; d < p.cz; d += 64) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < N; ++s) v += w[s] * *reinterpret_cast<const f32x4 *>(at[s] + 40 + d);
        v *= inv;
        if (!valid) v = (f32x4){0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f32x4 *>(p.o_pair + (ui * p.H + h) * p.cz + d) = v;
    }
}

struct SplitLayout {
    size_t cen, kvlen, zb, hb, part;  // part: also the size without the space for the key ranges' sums
};

constexpr int kUnits = 256;  // one workgroup per compute unit: a call of at most half as many tiles splits its key range

SplitLayout split_layout(const fipa_desc &d)
{
    SplitLayout w;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    const size_t n_kb = (d.L + 31) / 32;
    w.cen = take((size_t)d.B * 4 * sizeof(float));
    w.kvlen = take((size_t)d.B * sizeof(int));
    w.zb = take((size_t)d.B * n_kb * 3 * 64 * d.r * d.cz);
    w.hb = take((size_t)d.B * d.H * n_kb * kHeadBlock);
    w.part = off;
    return w;
}

long long split_tiles(const fipa_desc &d) { return (long long)d.B * d.H * ((d.L + 127) / 128); }

size_t split_parts_bytes(const fipa_desc &d, int parts)
{
    return parts > 1 ? (size_t)split_tiles(d) * parts * 128 * part_row(d.cz) * sizeof(float) : 0;
}

// Key ranges of a call; in less space than they take, as many as fit.
int split_parts(const fipa_desc &d)
{
    const long long tiles = split_tiles(d);
    const int n_kb = (d.L + 31) / 32;
    if (tiles > kUnits / 2) return 1;
    return std::max(1, std::min({(int)(kUnits / tiles), 8, n_kb / 2}));
}

template <int DZ>
hipError_t run_split(const SplitParams &p, hipStream_t stream)
{
    static LdsLimit lim;
    const hipError_t e = raise_lds_limit(lim, (const void *)fipa_attn_f32_split_kernel<DZ>, Fs<DZ>::kLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fipa_attn_f32_split_kernel<DZ>), dim3((p.n_units + 7) / 8 * 8), dim3(256), Fs<DZ>::kLds, stream, p);
    return hipGetLastError();
}

}  // namespace

// The lengths from which on the kernel may be the faster one (f32_split_applies); they only grow with the batch's at r c_z = 256.
static bool split_reaches(const fipa_desc &d)
{
    const int DZ = d.r * d.cz;
    if (d.c != 16 || d.Pq != 4 || d.Pv != 8 || d.cz % 4 != 0) return false;
    if (DZ == 256) return d.L >= 384 || (long long)d.B * d.H * ((d.L + 15) / 16) > 256;
    return (DZ == 128 && d.L >= 384) || ((DZ == 64 || DZ == 32) && d.L >= 512);
}

// Against the fp32 matrix instructions, us per call (those | this): r c_z = 256, one chain of 256, H = 4 to 12 41 | 38 to 41, of 320
// 48 | 41 to 49, of 384 54 to 98 | 42 to 49, of 1024 and H = 12 342 | 103; two chains, H = 12, of 160 34 | 43, of 192 60 | 44 (there
// the other kernel's tiles of 16 queries pass one round of the chip); r c_z = 128, H = 12, of 320 36 | 41, of 384 45 | 43, of 1024
// 174 | 80; r c_z = 64, H = 12, of 384 34 | 34, of 512 45 | 40, of 1024 90 | 70; r c_z = 32, H = 12, of 384 29 | 29, of 512 37 | 34, of 1024 75 | 62.
// Short calls are bound by start-up, which is longer here.
// Batches of short chains, r c_z = 256, whose tiles of 128 queries stand partly empty: up to 64 residues only where the other kernel's
// tiles of 16 queries, which it takes below 512 tiles of 32, make more than two rounds and the tiles here make one (B H = 192, 64 residues
// 52 | 38, 160 of 48 1 : 1.12, 256 of 64 37 | 41, 384 of 32 48 | 51, 768 of 32 48 | 73); from 65 to 96 residues not where a second round
// would be less than half full (B H = 300, 65 residues 1 : 1.10, 96 1 : 1.02, 380 of 65 1 : 0.92, 513 1 : 1.02; 256 1 : 0.77).
// r c_z = 32, up to 704 residues: not where little more than half of the compute units get a tile (144 tiles of 641 residues 1 : 1.11, of 672
// 1 : 1.09, of 704 1 : 0.96; 160 of 641 1 : 0.97), nor at 512 where the key ranges of more than 10 heads leave compute units idle (B H = 10
// 1 : 0.95, 12 1 : 1.02, 16 1 : 0.94, 24 1 : 1.03, 32 1 : 0.94, 60 1 : 0.66; of 528 12 1 : 0.91, 24 1 : 0.92).  r c_z = 128, below 432 residues:
// B H = 6 1 : 0.95 at 384, 8 1 : 1.02 (0.98 at 432), 10 1 : 1.05 (416 0.95), 12 1 : 0.98, 16 1 : 1.04 and at 392 0.96, 24 1 : 0.64.
// Batches with a mask, whose chains are shorter than the batch (70, and 70 and 40 % of it valid below), of fewer than 20 (batch, head) pairs:
// r c_z = 32 700 residues 1 : 0.90 to 1.02 (512 to 600 1 : 0.98 to 1.14), 64 560 residues 1 : 0.92 to 0.98 (512 1.00 to 1.10; B H = 8 1.04, 700 0.99), 128 above 512
// 1 : 0.91 to 0.96 (449 1.04 to 1.21; B H = 16 480 1 : 0.93), 256 B H = 8 480 1 : 0.90 (384 to 449 1.02 to 1.07).
bool f32_split_applies(const fipa_desc &d, bool masked)
{
    if (!split_reaches(d)) return false;
    const int DZ = d.r * d.cz;
    const long long bh = (long long)d.B * d.H;
    if (masked && bh < 20 && d.L < (DZ == 32 ? 700 : DZ == 64 ? (bh > 6 && bh < 12 ? 640 : 560) : DZ == 128 ? (bh >= 16 ? 480 : 513) : bh > 6 && bh < 12 ? 480 : 0)) return false;
    if (DZ == 256 && d.L <= 64) return bh <= kUnits && bh * ((d.L + 31) / 32) < 512 && bh * ((d.L + 15) / 16) > 512;
    if (DZ == 256 && d.L <= 96) return bh <= kUnits || bh >= 384;
    if (DZ == 128 && d.L < 432) return bh <= 6 || bh >= 20 || (bh >= 12 && (d.L > 384 || bh < 16)) || (d.L >= 416 && bh >= 10);
    if (DZ == 32 && d.L <= 512 && bh > 10 && split_tiles(d) <= kUnits / 2) return split_tiles(d) * split_parts(d) == kUnits;
    if (DZ == 32 && d.L > 512 && d.L < 704) return split_tiles(d) <= kUnits / 2 || split_tiles(d) >= 160;
    return true;
}

size_t f32_split_workspace_min(const fipa_desc &d) { return split_layout(d).part; }

// The key blocks, and the most that the key ranges of a chain up to this length take: a workspace for the longest chain of a batch serves
// the shorter ones too, and grows evenly with the length.
size_t f32_split_workspace(const fipa_desc &d)
{
    if (!split_reaches(d)) return 0;
    size_t parts = 0;
    fipa_desc x = d;
    for (int rt = 1; rt <= (d.L + 127) / 128 && (long long)d.B * d.H * rt <= kUnits / 2; ++rt) {
        x.L = std::min(128 * rt, d.L);
        if (split_reaches(x)) parts = std::max(parts, split_parts_bytes(x, split_parts(x)));
    }
    return split_layout(d).part + parts;
}

hipError_t f32_split_forward(const fipa_desc &d, const FwdArgs &a, void *ws, size_t ws_bytes, hipStream_t stream)
{
    const SplitLayout w = split_layout(d);
    char *base = static_cast<char *>(ws);
    SplitParams p;
    p.q = (const float *)a.q; p.k = (const float *)a.k; p.v = (const float *)a.v;
    p.q_pts = (const float *)a.q_pts; p.k_pts = (const float *)a.k_pts; p.v_pts = (const float *)a.v_pts;
    p.z1 = (const float *)a.z1; p.z2 = (const float *)a.z2;
    p.rot = a.rot; p.trans = a.trans; p.gamma = a.gamma; p.w_b = a.w_b; p.mask = a.mask; p.cu = nullptr;
    p.zb = base + w.zb;
    p.hb = base + w.hb;
    p.cen = reinterpret_cast<float *>(base + w.cen);
    p.kvlen = reinterpret_cast<int *>(base + w.kvlen);
    p.part = reinterpret_cast<float *>(base + w.part);
    p.o = a.o; p.o_pts = a.o_pts; p.o_pair = a.o_pair; p.lse = a.lse;
    p.B = d.B; p.L = d.L; p.H = d.H; p.cz = d.cz; p.r = d.r;
    p.DZ = d.r * d.cz;
    p.n_kb = (d.L + 31) / 32;
    p.n_rt = (d.L + 127) / 128;
    p.n_parts = split_parts(d);
    while (p.n_parts > 1 && w.part + split_parts_bytes(d, p.n_parts) > ws_bytes) --p.n_parts;
    p.n_units = d.B * d.H * p.n_rt * p.n_parts;
    p.w_L = d.w_L; p.w_C = d.w_C; p.qk_scale = d.qk_scale;

    StageTimer timer(stream);
    timer.begin(0);
    const int z_units = (int)(((long long)32 * p.n_kb * (p.DZ / 8) + 255) / 256);
    hipLaunchKernelGGL(fipa_pack_split_kernel, dim3(p.H * p.n_kb + z_units, p.B), dim3(256), 0, stream, p);
    timer.end(0);
    timer.begin(1);
    hipError_t e = p.DZ == 32 ? run_split<32>(p, stream) : p.DZ == 64 ? run_split<64>(p, stream) : p.DZ == 128 ? run_split<128>(p, stream) : run_split<256>(p, stream);
    if (e == hipSuccess && p.n_parts > 1) {
        const dim3 grid(p.n_units / p.n_parts * 8);
        if (p.n_parts == 2) hipLaunchKernelGGL(fipa_merge_split_kernel<2>, grid, dim3(256), 0, stream, p);
        else if (p.n_parts <= 4) hipLaunchKernelGGL(fipa_merge_split_kernel<4>, grid, dim3(256), 0, stream, p);
        else hipLaunchKernelGGL(fipa_merge_split_kernel<8>, grid, dim3(256), 0, stream, p);
        e = hipGetLastError();
    }
    timer.end(1);
    return e;
}

}  // namespace fipa
