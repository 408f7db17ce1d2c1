// k-nearest-neighbour distogram features (Section 2.5 of the paper): for every residue the k
// nearest valid residues of its chain by the distance of the frame origins, their squared
// distances and distogram bins -- [L, k] instead of the [L, L] distogram.  The paper gives one
// paragraph and no formula; the readings are stated in include/fipa.h.
//
// One wave per query residue or four of them.  The wave keeps its 64 best candidates so far as a sorted list, one
// entry per lane (lane s holds the s-th nearest), scans the chain 64 residues at a time, and
// inserts the few candidates that beat the current k-th entry one by one (a shift by one lane
// from the insertion point on); the scan starts at the residue's own block, which is ranked as a whole, and moves outwards.
// Order is by (squared distance, index), a strict total order, so the result does not depend on
// the order of the scan.  Every decision is taken in float32 on
// ((dx*dx + dy*dy) + dz*dz) with one rounding per operation (no fused multiply-add).
#include "fipa_internal.h"

#include <climits>

// This file is compiled with -ffp-contract=off: the distance arithmetic is specified with one
// rounding per operation, and the compiler would otherwise contract a*b + c into a fused
// multiply-add (also through the __fmul_rn / __fadd_rn intrinsics, which are plain operators).

namespace fipa {

namespace {

__device__ __forceinline__ bool before(float ad, int aj, float bd, int bj) { return ad < bd || (ad == bd && aj < bj); }

// One wave per R residues of a batch element (R = 4 where there are enough residues for it: the candidates'
// coordinates are then loaded, and the loop run, once per four residues).
// Four chains of up to 8192 residues, k = 20: 220 us with one residue per wave, every candidate of its own block inserted by
// itself and validity and self tested per candidate (28 instructions per residue and block of candidates) -> 175 us.
template <int R>
__global__ __launch_bounds__(256) void fipa_knn_distogram_kernel(const float *__restrict__ trans,
                                                                 const uint8_t *__restrict__ mask, int B, int L, int k,
                                                                 int n_bins, float d_min, float w,
                                                                 int *__restrict__ nbr_idx, float *__restrict__ nbr_d2,
                                                                 int *__restrict__ nbr_bin)
{
    const int lane = threadIdx.x & 63;
    // Workgroup g of every element side by side, the elements in a rotating order: chains of different lengths (a masked batch)
    // then leave every compute unit about the same number of residues.
    const int g = blockIdx.x / B, b = (blockIdx.x % B + (g >> 6)) % B;
    const int i0 = (4 * g + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * R;  // uniform over the wave
    if (i0 >= L) return;
    const float *t = trans + (size_t)b * L * 3;
    const uint8_t *m = mask ? mask + (size_t)b * L : nullptr;

    float best_d[R];  // lane s: the s-th nearest so far
    int best_j[R];
    float xi[R], yi[R], zi[R], thr_d[R];  // thr: entry k - 1 of the list
    int thr_j[R];
    bool any = false;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        best_d[q] = INFINITY;
        best_j[q] = INT_MAX;
        const int i = min(i0 + q, L - 1);
        const bool on = i0 + q < L && (!m || m[i] != 0);
        any |= on;
        xi[q] = t[3 * i]; yi[q] = t[3 * i + 1]; zi[q] = t[3 * i + 2];
        thr_d[q] = on ? INFINITY : -1.f;  // (a residue that wants no neighbours: nothing passes)
        thr_j[q] = INT_MAX;
    }
    if (any) {
        // The blocks of 64 candidates are visited outwards from the residues' own: in a chain the
        // neighbours along the sequence are near in space, so the list fills with near residues at
        // once and few later candidates beat its k-th entry (in index order every residue before i
        // arrives nearer than the one before it and is inserted, one at a time).
        const int nblk = (L + 63) / 64, own = i0 / 64;
        struct Cand {
            float x, y, z;  // x: not a number where there is no candidate, so that no comparison holds
        };
        auto load = [&](int j0) {
            const int j = j0 + lane, jc = min(j, L - 1);
            const bool ok = j < L && (!m || m[jc] != 0);
            Cand c = {t[3 * jc], t[3 * jc + 1], t[3 * jc + 2]};
            c.x = ok ? c.x : __builtin_nanf("");
            return c;
        };
        auto dist = [&](const Cand &c, int q) {
            const float dx = __fsub_rn(c.x, xi[q]), dy = __fsub_rn(c.y, yi[q]), dz = __fsub_rn(c.z, zi[q]);
            return __fadd_rn(__fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy)), __fmul_rn(dz, dz));
        };
        // The residues' own block fills the empty lists: every candidate counts those before it and goes to that place.
        // (i0 .. i0 + R - 1 lie in one block: R divides 64.)
        {
            const Cand c = load(64 * own);
            const int j = 64 * own + lane;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const float d2 = dist(c, q);
                const bool cand = d2 <= thr_d[q] && j != i0 + q;
                const unsigned long long cands = __ballot(cand), below = (1ull << lane) - 1ull;
                int rank = cand ? 0 : __popcll(cands) + __popcll(~cands & below);
                for (unsigned long long rest = cands; rest; rest &= rest - 1) {
                    const int l = __ffsll((long long)rest) - 1;
                    const float dl = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, d2), l));
                    rank += cand && (dl < d2 || (dl == d2 && l < lane)) ? 1 : 0;
                }
                best_d[q] = __builtin_bit_cast(float, __builtin_amdgcn_ds_permute(4 * rank, __builtin_bit_cast(int, cand ? d2 : INFINITY)));
                best_j[q] = __builtin_amdgcn_ds_permute(4 * rank, cand ? j : INT_MAX);
                if (thr_d[q] >= 0.f) {
                    thr_d[q] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, best_d[q]), k - 1));
                    thr_j[q] = __builtin_amdgcn_readlane(best_j[q], k - 1);
                }
            }
        }
        int up = own + 1, down = own - 1;
        auto next = [&](int step) {  // alternately above and below while both sides have blocks left
            const bool take_up = up < nblk && (down < 0 || (step & 1) == 0);
            return 64 * (take_up ? up++ : down--);
        };
        int j0 = nblk > 1 ? next(0) : 0;
        Cand c = load(j0);
        for (int step = 1; step < nblk; ++step) {
            const Cand now = c;
            const int jnow = j0 + lane;
            if (step + 1 < nblk) {
                j0 = next(step);
                c = load(j0);
            }
            float d2[R];
            unsigned long long todo[R], some = 0ull;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                d2[q] = dist(now, q);
                todo[q] = __ballot(d2[q] <= thr_d[q]);  // (candidates at the threshold itself are decided by their index)
                some |= todo[q];
            }
            if (some == 0ull) continue;
#pragma unroll
            for (int q = 0; q < R; ++q)
                while (todo[q]) {
                    const int l = __ffsll((long long)todo[q]) - 1;
                    todo[q] &= todo[q] - 1;
                    const float nd = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, d2[q]), l));
                    const int nj = __builtin_amdgcn_readlane(jnow, l);
                    if (!before(nd, nj, thr_d[q], thr_j[q])) continue;  // (also: the threshold has moved since the ballot)
                    // insert: the entries behind the new one move one lane up
                    const int behind = before(nd, nj, best_d[q], best_j[q]) ? 1 : 0;
                    const float prev_d = __shfl_up(best_d[q], 1);
                    const int prev_j = __shfl_up(best_j[q], 1);
                    const int up_behind = __shfl_up(behind, 1);  // (every lane takes part in the exchange)
                    const int prev_behind = lane > 0 ? up_behind : 0;
                    if (behind) {
                        best_d[q] = prev_behind ? prev_d : nd;
                        best_j[q] = prev_behind ? prev_j : nj;
                    }
                    thr_d[q] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, best_d[q]), k - 1));
                    thr_j[q] = __builtin_amdgcn_readlane(best_j[q], k - 1);
                }
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (i0 + q >= L || lane >= k) continue;
        const bool have = best_j[q] != INT_MAX;
        int bin = -1;
        if (have) {
            bin = 0;
            for (int e = 0; e < n_bins - 1; ++e) {
                const float edge = __fadd_rn(d_min, __fmul_rn((float)e, w));
                bin += __fmul_rn(edge, edge) <= best_d[q] ? 1 : 0;
            }
        }
        const size_t at = ((size_t)b * L + i0 + q) * k + lane;
        nbr_idx[at] = have ? best_j[q] : -1;
        nbr_d2[at] = have ? best_d[q] : INFINITY;
        nbr_bin[at] = bin;
    }
}

}  // namespace

}  // namespace fipa

extern "C" int fipa_knn_distogram(int32_t B, int32_t L, int32_t k, int32_t n_bins, float d_min, float d_max,
                                  const float *trans, const uint8_t *mask, int32_t *nbr_idx, float *nbr_d2,
                                  int32_t *nbr_bin, void *hip_stream)
{
    if (B <= 0 || L <= 0 || k <= 0 || n_bins < 2 || !(d_min >= 0.f) || !(d_max > d_min)) return FIPA_ERR_INVALID_ARG;
    if (!trans || !nbr_idx || !nbr_d2 || !nbr_bin) return FIPA_ERR_INVALID_ARG;
    if (k > 64 || n_bins > 4096 || (long long)B * L * k >= (1LL << 31)) return FIPA_ERR_UNSUPPORTED;
    const void *al[] = {trans, nbr_idx, nbr_d2, nbr_bin};
    for (const void *ptr : al)
        if ((reinterpret_cast<uintptr_t>(ptr) & 3u) != 0) return FIPA_ERR_ALIGNMENT;
    const float w = (d_max - d_min) / (float)(n_bins - 1);
    // four residues per wave once that leaves four waves per SIMD
    const int R = (long long)B * ((L + 3) / 4) >= 4096 ? 4 : 1;
    const dim3 grid((unsigned)(B * ((L + 4 * R - 1) / (4 * R))));
    hipLaunchKernelGGL(R == 4 ? fipa::fipa_knn_distogram_kernel<4> : fipa::fipa_knn_distogram_kernel<1>, grid, dim3(256), 0,
                       static_cast<hipStream_t>(hip_stream), trans, mask, B, L, k, n_bins, d_min, w, nbr_idx, nbr_d2, nbr_bin);
    return hipGetLastError() == hipSuccess ? FIPA_OK : FIPA_ERR_LAUNCH;
}
