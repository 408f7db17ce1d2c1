// Pair pseudo-factors from k-nearest-neighbour features (Section 2.4 of the paper: each pair
// feature is represented by two [L, r, c_z] tensors obtained by linear projections; Section 2.5:
// the features are the distogram bins of the k nearest neighbours plus a positional encoding of
// the neighbours' indices).  The paper gives no formula; the readings are stated in include/fipa.h.
//
// A linear projection of concatenated one-hot vectors is a sum of table rows, so nothing is
// multiplied: z_i = bias + sum over the neighbour slots s of (e_bin[s][bin_is] + e_pos[s][code_is]).
// One thread per (residue, 8 output columns): the threads of a residue read the same k indices
// (one broadcast load each) and consecutive 16-byte pieces of the selected rows; the tables (a
// few MB at most) stay in L2, so the kernel is bound by L2 reads of 2 k n_out bf16 per residue,
// not by HBM (the algorithmic HBM traffic is the n_out bf16 written and 8 k index bytes read).
// Sums are float32 in slot order (bias, then per slot the bin row, then the position row), rounded
// to bf16 once at the end.
#include "fipa_gfx950.h"
#include "fipa_internal.h"

#include <climits>

namespace fipa {

namespace {

__device__ __forceinline__ void add_row(float (&acc)[8], const bf16_t *row, bool on)
{
    const uint4 v = *reinterpret_cast<const uint4 *>(row);
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        acc[2 * q] += on ? __uint_as_float(w[q] << 16) : 0.f;
        acc[2 * q + 1] += on ? __uint_as_float(w[q] & 0xffff0000u) : 0.f;
    }
}

template <bool HAS_POS>
__global__ __launch_bounds__(256) void fipa_factor_project_kernel(const int *__restrict__ nbr_idx, const int *__restrict__ nbr_bin,
                                                                  const bf16_t *__restrict__ e_bin, const bf16_t *__restrict__ e_pos,
                                                                  const float *__restrict__ bias, bf16_t *__restrict__ z,
                                                                  long long rows, int L, int k, int n_bins, int n_pos,
                                                                  int pos_mode, int nchunk)
{
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= rows * nchunk) return;
    const long long row = t / nchunk;
    const int ch = (int)(t - row * nchunk), i = (int)(row % L);
    const size_t n_out = (size_t)nchunk * 8;
    float acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = bias ? bias[ch * 8 + q] : 0.f;
    const int *ji = nbr_idx + row * k, *bi = nbr_bin + row * k;
    const int half = (n_pos - 1) >> 1;
#pragma unroll 4
    for (int s = 0; s < k; ++s) {
        const int j = ji[s];
        const bool filled = j >= 0 && j < L;
        // an empty slot reads row 0 and adds nothing (no divergent branch around the loads); a bin
        // outside the table is clamped into it, so every address is inside the tables
        const bool on = filled;
        const int bn = filled ? min(max(bi[s], 0), n_bins - 1) : 0;
        add_row(acc, e_bin + ((size_t)s * n_bins + bn) * n_out + ch * 8, on);
        if constexpr (HAS_POS) {
            int code = pos_mode == 0 ? min(j, n_pos - 1) : min(max(j - i, -half), half) + half;
            code = filled ? code : 0;
            add_row(acc, e_pos + ((size_t)s * n_pos + code) * n_out + ch * 8, on);
        }
    }
    uint4 o;
    o.x = (unsigned)f2bf(acc[0]) | ((unsigned)f2bf(acc[1]) << 16);
    o.y = (unsigned)f2bf(acc[2]) | ((unsigned)f2bf(acc[3]) << 16);
    o.z = (unsigned)f2bf(acc[4]) | ((unsigned)f2bf(acc[5]) << 16);
    o.w = (unsigned)f2bf(acc[6]) | ((unsigned)f2bf(acc[7]) << 16);
    *reinterpret_cast<uint4 *>(z + row * n_out + ch * 8) = o;
}

// The same with the tables of 32 columns (64 bytes per row) in LDS, where a workgroup then adds up many residues: the rows of
// a residue come out of LDS instead of L2.  1024 threads, four per residue; a wave takes groups of 16 residues that lie gridDim.y * 16 groups
// apart, so that the masked ends of a padded batch (no slot filled: nothing to add) are spread over all workgroups, and needs no other wave
// behind the loading of the table: it looks up the table rows of its own residues.  An empty slot takes a row of zeros.  Same sums in the same
// order.  (One instruction per value and slot, a product of the slot's two rows with ones, is 2 to 6 us faster at the size below, but it does
// not round to nearest: of random sums with one row in five was off by a last place.)
// 32768 residues (60 % of them valid), 20 slots, 81 rows per slot, 512 columns: 99 us from L2; from LDS 60 us with contiguous ranges of
// residues per workgroup, a barrier per 256 of them and indices that were loaded where they were looked at, 38 us so (all valid: 62, 53).
// What is left is the LDS reads of rows that meet in the banks (64 bytes each, any of four places) and the loading of the table (about 5 us).
// Used where every workgroup has enough residues to add for the table that it loads (factor_rows) and the table fits: one chain of 4096
// residues, 512 columns, 16.8 us from L2, 12.0 so; 2048 11.5 and 9.9; 8192 residues of 128 columns, 16 slots 10.1 and 9.2.
constexpr int kFpThreads = 1024, kFpPass = kFpThreads / 4;
constexpr int kFpAhead = 8;  // slots of a thread whose indices and bins wait in registers: 32 of a residue
// Residues per workgroup from which the table is worth loading.  From L2 | so, 512 columns, 33 + 16 rows per slot, us or ratio: 16 slots, 128 residues
// 10.1 | 9.2, 30 slots 15.8 | 12.0; just above 128 residues, where the kernel that reads from L2 needs a round of workgroups more, 10 slots 1 : 0.88 (at
// 128 1.01 to 1.08), 6 1 : 0.95 to 0.98 (1.12 to 1.17), 4 1 : 1.01 to 1.07; just above 192, where it is another, 4 slots 1 : 0.91 to 0.97, 2 1 : 0.88.
inline int factor_rows(int k) { return k >= 16 ? 128 : k >= 6 ? 136 : 200; }
inline size_t factor_lds_bytes(int k, int n_bins, int n_pos)
{
    return 64 * ((size_t)k * (n_bins + n_pos) + 1) + (size_t)kFpPass * k * 4;
}

__global__ __launch_bounds__(kFpThreads) void fipa_factor_project_lds_kernel(const int *__restrict__ nbr_idx, const int *__restrict__ nbr_bin,
                                                                             const bf16_t *__restrict__ e_bin, const bf16_t *__restrict__ e_pos,
                                                                             const float *__restrict__ bias, bf16_t *__restrict__ z, int rows,
                                                                             int L, int k, int n_bins, int n_pos, int pos_mode, int n_out)
{
    extern __shared__ __attribute__((aligned(16))) char fp_smem[];  // table rows [k][n_bins + n_pos], the row of zeros | row numbers [k][residue of the pass]
    const int tid = threadIdx.x, per = n_bins + n_pos, nrow = k * per, half = (n_pos - 1) >> 1;
    const int col0 = blockIdx.x * 32;
    unsigned *const codes = reinterpret_cast<unsigned *>(fp_smem + 64 * ((size_t)nrow + 1));
    const int part = tid & 3, col = col0 + 8 * part;
    // A wave takes every 16 gridDim.y-th group of 16 residues, four lanes each, and looks up the rows (bin, position) of their slots itself, a lane
    // every fourth slot: codes[slot][residue].  The indices and bins of the first kFpAhead of those slots are requested (ask) before the
    // group before is added up, and looked at (look_up) behind it.
    const int rr = tid >> 2, stride = kFpPass * gridDim.y, turn = stride % L;
    const int first = 16 * (blockIdx.y + gridDim.y * (tid >> 6)) + (rr & 15);  // this lane's residues: first, first + stride, ..
    int i_next = first % L;  // place in the chain of the one that is looked up next
    int nbr[kFpAhead], bins[kFpAhead];
    auto ask = [&](int res) {
        const size_t at = (size_t)min(res, rows - 1) * k;
#pragma unroll
        for (int u = 0; u < kFpAhead; ++u) {
            if (4 * u >= k) break;
            const int s = min(part + 4 * u, k - 1);
            nbr[u] = nbr_idx[at + s];
            bins[u] = nbr_bin[at + s];
        }
    };
    auto look_up = [&](int res) {
        const size_t at = (size_t)min(res, rows - 1) * k;
        const int i = i_next;
        bool any = false;
        auto one = [&](int s, int j, int bn) {
            unsigned bin_row = nrow, pos_row = nrow;  // zeros
            if (j >= 0 && j < L) {
                any = true;
                bin_row = s * per + min(max(bn, 0), n_bins - 1);
                if (n_pos > 0) pos_row = s * per + n_bins + (pos_mode == 0 ? min(j, n_pos - 1) : min(max(j - i, -half), half) + half);
            }
            codes[s * kFpPass + rr] = bin_row | (pos_row << 16);
        };
#pragma unroll
        for (int u = 0; u < kFpAhead; ++u) {
            if (4 * u >= k) break;
            if (part + 4 * u < k) one(part + 4 * u, nbr[u], bins[u]);
        }
        for (int s = part + 4 * kFpAhead; s < k; s += 4) one(s, nbr_idx[at + s], nbr_bin[at + s]);
        i_next += turn;
        if (i_next >= L) i_next -= L;
        return __any(any) != 0;
    };
    ask(first);
    for (int x0 = tid; x0 < 4 * (nrow + 1); x0 += 8 * kFpThreads) {  // (eight loads in flight)
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int x = x0 + u * kFpThreads, row = min(x >> 2, nrow - 1), c = col0 + 8 * (x & 3);
            const int s = row / per, m = row - s * per;
            const bf16_t *src = m < n_bins ? e_bin + ((size_t)s * n_bins + m) * n_out : e_pos + ((size_t)s * n_pos + m - n_bins) * n_out;
            v[u] = *reinterpret_cast<const uint4 *>(src + min(c, n_out - 8));
            if (x >= 4 * nrow || c >= n_out) v[u] = (uint4){0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int x = x0 + u * kFpThreads;
            if (x < 4 * (nrow + 1)) *reinterpret_cast<uint4 *>(fp_smem + 16 * (size_t)x) = v[u];
        }
    }
    float b8[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) b8[q] = bias && col < n_out ? bias[col + q] : 0.f;
    auto add = [](float (&acc)[8], const char *row) {
        const uint4 v = *reinterpret_cast<const uint4 *>(row);
        const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc[2 * q] += __uint_as_float(w[q] << 16);
            acc[2 * q + 1] += __uint_as_float(w[q] & 0xffff0000u);
        }
    };
    __syncthreads();  // the table is there
    const int whole = 16 * (blockIdx.y + gridDim.y * (tid >> 6));  // (the wave's first residue)
    for (int r0 = whole, res = first; r0 < rows; r0 += stride, res += stride) {
        const bool some = look_up(res);
        ask(res + stride);
        asm volatile("" ::: "memory");  // (the LDS accesses of a wave execute in order)
        if (res < rows && col < n_out) {
            float acc[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] = b8[q];
            const int slots = some ? k : 0;
#pragma unroll 4
            for (int s = 0; s < slots; ++s) {
                const unsigned c = codes[s * kFpPass + rr];
                add(acc, fp_smem + 64 * (c & 0xFFFFu) + 16 * part);
                add(acc, fp_smem + 64 * (c >> 16) + 16 * part);
            }
            uint4 o;
            o.x = (unsigned)f2bf(acc[0]) | ((unsigned)f2bf(acc[1]) << 16);
            o.y = (unsigned)f2bf(acc[2]) | ((unsigned)f2bf(acc[3]) << 16);
            o.z = (unsigned)f2bf(acc[4]) | ((unsigned)f2bf(acc[5]) << 16);
            o.w = (unsigned)f2bf(acc[6]) | ((unsigned)f2bf(acc[7]) << 16);
            *reinterpret_cast<uint4 *>(z + (size_t)res * n_out + col) = o;
        }
        asm volatile("" ::: "memory");
    }
}

// Gradient with respect to the tables: d e_bin[s, m, :] is the sum of d_z[b, i, :] over the residues
// whose slot s is filled and holds bin m, likewise d e_pos by position code, d bias the sum over
// all residues.  A scatter of rows -- but a scatter into shared sums either serialises on LDS
// round trips (per-wave table copies updated row by row: 2.1 ms at 32768 residues, 512 columns; with
// LDS float atomics 8.6 ms) or loses the fixed summation order.  Here it is the contraction it
// also is, over the residue axis: dE_s [rows, 64 columns] = X_s^T [rows, residues] . dZ [residues, 64],
// with X_s the one-hot features of slot s -- exact in bf16 -- on the matrix pipe with float32
// accumulation in a fixed order (the same bits on every run).
//
// One workgroup per (slot, 64 output columns), eight waves, each of which takes every eighth tile of 32
// residues with all rows of the tables: nothing is shared between waves until their sums are added at the
// end, so there is no barrier in the loop, and two waves per SIMD cover each other.  A tile without a residue that counts is left out.
// A tile's d_z rows arrive by direct loads two tiles ahead, its indices, bins and mask one tile earlier; d_z is read with the transposing LDS
// read.  The one-hot operand is a tile of the wave in LDS, [table row][residue], read as it stands: a tile's residues set their
// ones and take them back behind it.  The operands of a tile are read while the tile before is multiplied, each into the registers
// of the one that has just been used (two sets of registers: spilled).
// 32768 residues (60 % of them valid), 20 slots, 82 rows, 512 columns: 555 us with four waves that shared each tile and its one-hot tile
// (one barrier per tile, the mask on the way of every load) -> 131 us with the operand formed by comparing 16-bit codes in
// registers (16 vector instructions per operand) -> 103 us with the tile of ones -> 60 us without the masked tiles and with fewer instructions
// around the products.  Without a mask 110 -> 99 -> 86 us (operands read ahead), of which 41 are matrix instructions; loads of the indices
// and bins from neighbouring addresses would save 4.  A bit per residue and row, set with LDS or, and a table of
// the 256 possible operands: 165 us (many residues share a row, and the or's on one address run one after the other).
// rows = n_bins + n_pos + 1 (the last one collects the bias gradient, in slot 0's workgroups).
constexpr int kFbWaves = 8, kFbMaxRowBlocks = 5;
constexpr int kFbZ = 32 * 128;                          // a tile's d_z: 32 rows of 64 columns, the 64-byte halves of a row exchanged in every other pair of rows
constexpr int kFbCodes = 256 + 256;                     // 32 indices, 32 bins | 64 mask values
template <int RB>
struct FbCfg {
    static constexpr int kStages = RB <= 3 ? 3 : 2, kCodeStages = 4;
    static constexpr int kOnes = kStages * kFbZ + kCodeStages * kFbCodes;  // one-hot tile: 64 bytes per table row, its 16-byte slots c at c ^ (row / 4 mod 4)
    static constexpr int kWaveBytes = kOnes + 32 * RB * 64;
    static constexpr int kSum = RB * 2 * 16 * 64 * 4;   // bytes of a wave's sums
    static constexpr int kBytes = kFbWaves * kWaveBytes > kSum * (kFbWaves / 2) ? kFbWaves * kWaveBytes : kSum * (kFbWaves / 2);
    static_assert(kBytes <= 160 * 1024, "LDS");
};

// One direct load of 4 bytes (BYTES = 1: a byte, zero-extended) per lane to LDS bytes lds + 4 lane; of 16 bytes to lds + 16 lane.
template <int BYTES>
__device__ __forceinline__ void fb_load(const void *addr, unsigned lds)
{
    if constexpr (BYTES == 16)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(addr) : "memory", "m0");
    else if constexpr (BYTES == 4)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(addr) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_ubyte %1, off" ::"s"(lds), "v"(addr) : "memory", "m0");
}

// 16 bytes per lane from base + voff to LDS bytes lds + 16 lane.
__device__ __forceinline__ void fb_load_at(const void *base, unsigned voff, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}

template <int RB, bool MASK>
__global__ __launch_bounds__(64 * kFbWaves, 2) void fipa_factor_backward_kernel(const int *__restrict__ nbr_idx, const int *__restrict__ nbr_bin,
                                                                               const bf16_t *__restrict__ d_z, const uint8_t *__restrict__ mask,
                                                                               float *__restrict__ d_e_bin, float *__restrict__ d_e_pos,
                                                                               float *__restrict__ d_bias, int rows, int L, int k, int n_bins,
                                                                               int n_pos, int pos_mode, int n_out)
{
    extern __shared__ __attribute__((aligned(16))) char fb_smem[];
    const int s = blockIdx.y, col0 = blockIdx.x * 64;  // (512 columns: each of the 8 XCDs streams the same 64 for every slot)
    const int lane = threadIdx.x & 63, li = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int R = n_bins + n_pos + 1, half = (n_pos - 1) >> 1;
    using C = FbCfg<RB>;
    char *const mine = fb_smem + wave * C::kWaveBytes;
    const unsigned mine_lds = lds_address(mine);
    const int ntiles = (rows + 31) / 32;
    const int own = wave < ntiles ? (ntiles - wave + kFbWaves - 1) / kFbWaves : 0;  // tiles wave, wave + 8, ...

    // ---- the wave's tiles, those without a residue that counts left out: 64 of them looked at at a time, a lane each --------------
    int base = 0;  // the first of those 64
    unsigned long long rest = 0ull;
    auto look = [&] {
        const int r0 = 32 * min(wave + kFbWaves * (base + lane), ntiles - 1), words = rows >> 2;
        const unsigned *const m = reinterpret_cast<const unsigned *>(mask);
        unsigned any = 0u;
        if ((reinterpret_cast<uintptr_t>(mask) & 3u) != 0) {
            any = 1u;
        } else if ((rows & 31) == 0) {
#pragma unroll
            for (int x = 0; x < 8; ++x) any |= m[r0 / 4 + x];
        } else {  // (one round trip here too; words past the end are the last one again, and the last tile takes the bytes behind it)
            unsigned tail = 0u;
#pragma unroll
            for (int x = 0; x < 3; ++x) tail |= mask[min(4 * words + x, rows - 1)];
            if (words > 0)
#pragma unroll
                for (int x = 0; x < 8; ++x) any |= m[min(r0 / 4 + x, words - 1)];
            if (r0 + 32 > rows) any |= tail;
        }
        if (base + lane >= own) any = 0u;
        rest = __ballot(any != 0u);
    };
    int seen = 0;  // (no mask: the next tile)
    auto next_tile = [&]() -> int {  // -1: no more
        if constexpr (!MASK) return seen < own ? wave + kFbWaves * seen++ : -1;
        while (rest == 0ull) {
            if (base + 64 >= own) return -1;
            base += 64;
            look();
        }
        const int n = base + __builtin_ctzll(rest);
        rest &= rest - 1ull;
        return wave + kFbWaves * n;
    };
    if constexpr (MASK) look();

    // Loads of a tile's indices, bins and mask, and of its d_z (past the last tile: the last one again, so that every step has as many).
    // Rows and columns past the end: addresses of existing ones, what they bring is not used.
    constexpr int kLoads = MASK ? 6 : 5;
    unsigned vz[4];
    const int l8 = lane >> 3, l7 = lane & 7;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int rr = 8 * q + l8;
        vz[q] = (unsigned)(rr * n_out + min(8 * (l7 ^ (((rr >> 1) & 1) << 2)), n_out - 8 - col0)) * 2;
    }
    const int *const codes = (g ? nbr_bin : nbr_idx) + s;
    auto issue_codes = [&](int tile, int stage) {
        const unsigned st = mine_lds + stage * kFbCodes + C::kStages * kFbZ;
        const size_t res = min(32 * tile + li, rows - 1);
        fb_load<4>(codes + res * k, st);
        if constexpr (MASK) fb_load<1>(mask + res, st + 256);
    };
    auto issue_z = [&](int tile, int stage) {
        const unsigned st = mine_lds + stage * kFbZ;
        const bf16_t *from = d_z + (size_t)tile * 32 * n_out + col0;
        if (32 * tile + 32 <= rows) {
#pragma unroll
            for (int q = 0; q < 4; ++q) fb_load_at(from, vz[q], st + 1024 * q);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) fb_load_at(from, vz[q] - (unsigned)(max(8 * q + l8 - (rows - 1 - 32 * tile), 0) * n_out) * 2, st + 1024 * q);
        }
    };

    f32x16 acc[RB][2];
#pragma unroll
    for (int mb = 0; mb < RB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.f;

    char *const ones = mine + C::kOnes;
    for (int x = lane; x < 32 * RB * 4; x += 64) *reinterpret_cast<uint4 *>(ones + 16 * x) = (uint4){0u, 0u, 0u, 0u};
    // residue q of a group of 16 is value q mod 4 + 4 (q / 8) of the lanes of half q / 4 mod 2 (the order of the transposing read)
    const int slot = 2 * (li >> 4) + ((li >> 2) & 1), within = 2 * (4 * ((li >> 3) & 1) + (li & 3));
    auto one_at = [&](int row) { return row * 64 + ((slot ^ ((row >> 2) & 3)) << 4) + within; };
    const int aone = li * 64 + ((g ^ ((li >> 2) & 3)) << 4);  // (k-step t: slot 2 t + g)
    const int e4 = (lane & 15) >> 2, grp2 = (lane >> 4) & 1, j4 = lane & 3;
    int az[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) az[nb] = (4 * g + e4) * 128 + (nb ^ (e4 >> 1)) * 64 + (16 * grp2 + 4 * j4) * 2;

    // of a tile, from its indices, bins and mask: where this lane's one goes (a residue whose slot is empty or that does not count: to a place
    // in the masks' room that nothing reads), and which residues count
    const int nowhere = C::kStages * kFbZ + 384 + within - C::kOnes, bias_one = one_at(R - 1);
    const bool my_table = g == 0 || n_pos > 0;
    const int pos_lo = pos_mode ? -half : 0, pos_hi = pos_mode ? half : n_pos - 1, pos_0 = n_bins + (pos_mode ? half : 0);
    const int row_lo = g ? pos_lo : 0, row_hi = g ? pos_hi : n_bins - 1, row_0 = g ? pos_0 : 0;
    const unsigned inv_L = 0xFFFFFFFFu / (unsigned)L;
    const int li_L = li % L;
    int one = nowhere, j, bn, mk = 1;
    unsigned vmask = 0u;
    auto read_codes = [&](int stage) {
        const char *const st = mine + C::kStages * kFbZ + stage * kFbCodes;
        j = *reinterpret_cast<const int *>(st + 4 * li);
        bn = *reinterpret_cast<const int *>(st + 128 + 4 * li);
        if constexpr (MASK) mk = *reinterpret_cast<const int *>(st + 256 + 4 * li);
    };
    auto decode = [&](int tile) {
        const bool valid = 32 * tile + li < rows && mk != 0;
        vmask = (unsigned)__ballot(valid);  // (the two halves agree)
        unsigned r0 = 32u * tile;  // place of the tile's first residue in its chain
        r0 -= __umulhi(r0, inv_L) * (unsigned)L;
        if (r0 >= (unsigned)L) r0 -= L;
        int i = (int)r0 + li_L;
        if (i >= L) i -= L;
        const int code = g ? (pos_mode ? j - i : j) : bn;
        const bool filled = valid && (unsigned)j < (unsigned)L && my_table;
        one = filled ? one_at(min(max(code, row_lo), row_hi) + row_0) : nowhere;
    };
    auto advance = [](int stage, int n) { return stage + 1 == n ? 0 : stage + 1; };
    // tiles n, n + 1, .. of the wave (n: the one that is multiplied); where there is none, the one before again
    constexpr int S = C::kStages;
    int now = next_tile(), ahead[S], zs = 0, cs = 0;  // stages of tile n
    if (now >= 0) {
        bool more = true;
        int prev = now;
#pragma unroll
        for (int x = 0; x < S; ++x) {
            ahead[x] = more ? next_tile() : -1;
            more = ahead[x] >= 0;
        }
        issue_codes(now, 0);
#pragma unroll
        for (int x = 0; x < S - 1; ++x) {  // codes of tile n + 1 + x, d_z of tile n + x
            const int z_tile = prev;
            if (ahead[x] >= 0) prev = ahead[x];
            issue_codes(prev, x + 1);
            issue_z(z_tile, x);
        }
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * kLoads) : "memory");
        read_codes(0);
        decode(now);
    }
    int last = now;  // the tile whose loads are repeated past the end
#pragma unroll
    for (int x = 0; x < S - 1; ++x) last = now >= 0 && ahead[x] >= 0 ? ahead[x] : last;  // tile n + S - 1, or the last one
    // The operands of a tile are read while the tile before is multiplied, each into the registers of the one that has just been used.
    // (Not with five row blocks and a mask, where registers of the loop were spilled for it: 4 chains of 8192, 130 rows 123 us, 111 so; one
    // of 500 14.2, 12.6.  Without a mask, 2 spilled outside of the loop: 108, 134 so.)
    constexpr bool kReadAhead = RB <= 4 || !MASK;
    bf16x8 bz[2][2], a[2][RB];
    auto multiply = [&](int t, int mb) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t][mb], bz[t][nb], acc[mb][nb], 0, 0, 0);
    };
    auto step = [&](auto First) {
        constexpr bool first = !kReadAhead || decltype(First)::value;
        // d_z of tile n and the codes of tile n + 1 have landed; the reads of tile n - 1, whose stage the next loads take, are done
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * kLoads) : "memory");
        {
            const int z_tile = last;
            if (ahead[S - 1] >= 0) last = ahead[S - 1];
            issue_codes(last, (cs + S) & (C::kCodeStages - 1));
            issue_z(z_tile, zs == 0 ? S - 1 : zs - 1);
        }
        unsigned z0 = zs * kFbZ;
        asm volatile("" : "+s"(z0));  // (so that what follows is an address and constants)
        char *const st = mine + z0;
        read_codes((cs + 1) & (C::kCodeStages - 1));  // (past the last tile: not used)
        const bool counts = (vmask >> li) & 1u;
        auto set = [&](bf16_t v) {
            *reinterpret_cast<bf16_t *>(ones + one) = v;
            if (s == 0 && g == 0 && counts) *reinterpret_cast<bf16_t *>(ones + bias_one) = v;
            asm volatile("" ::: "memory");  // (the LDS accesses of a wave execute in order)
        };
        set(0x3F80);
        if (vmask != 0xFFFFFFFFu) {
            // what a masked or missing residue holds must not reach the products: 0 x NaN would
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (!((vmask >> (8 * q + l8)) & 1u)) *reinterpret_cast<uint4 *>(st + 1024 * q + 16 * lane) = (uint4){0u, 0u, 0u, 0u};
            asm volatile("" ::: "memory");
        }
        const char *const zp[2] = {st + az[0], st + az[1]};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int mb = 0; mb < RB; ++mb) {
                if constexpr (!first) {
                    multiply(t, mb);
                    __builtin_amdgcn_sched_barrier(0);
                }
                a[t][mb] = *reinterpret_cast<const bf16x8 *>(ones + 32 * 64 * mb + (aone ^ (32 * t)));
            }
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) bz[t][nb] = lds_read_tr(zp[nb] + 16 * t * 128, zp[nb] + (16 * t + 8) * 128);
            if constexpr (!first) __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("" ::: "memory");
        set(0);
        if constexpr (!kReadAhead) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int mb = 0; mb < RB; ++mb) multiply(t, mb);
        }
        now = ahead[0];
        decode(now);  // (past the last tile: not used)
#pragma unroll
        for (int x = 0; x < S - 1; ++x) ahead[x] = ahead[x + 1];
        ahead[S - 1] = ahead[S - 1] >= 0 ? next_tile() : -1;
        zs = advance(zs, S);
        cs = (cs + 1) & (C::kCodeStages - 1);
    };
    if (now >= 0) {
        step(std::true_type{});
        while (now >= 0) step(std::false_type{});
        if constexpr (kReadAhead) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int mb = 0; mb < RB; ++mb) multiply(t, mb);
        }
    }
    wait_vmem<0>();  // (loads past the last tile still write LDS)
    // the waves' sums, in a fixed order: 4..7 to 0..3, 2..3 to 0..1, 1 to 0
    constexpr int kSum = C::kSum;
#pragma unroll
    for (int w = kFbWaves / 2; w >= 1; w >>= 1) {
        __syncthreads();
        if (wave >= w && wave < 2 * w)
#pragma unroll
            for (int mb = 0; mb < RB; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<f32x4 *>(fb_smem + (wave - w) * kSum + ((mb * 2 + nb) * 4 + q) * 1024 + 16 * lane) =
                            (f32x4){acc[mb][nb][4 * q], acc[mb][nb][4 * q + 1], acc[mb][nb][4 * q + 2], acc[mb][nb][4 * q + 3]};
        __syncthreads();
        if (wave < w)
#pragma unroll
            for (int mb = 0; mb < RB; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(fb_smem + wave * kSum + ((mb * 2 + nb) * 4 + q) * 1024 + 16 * lane);
#pragma unroll
                        for (int x = 0; x < 4; ++x) acc[mb][nb][4 * q + x] += v[x];
                    }
    }
    // out through LDS, all threads storing: accumulator register r of a lane is row 8 (r / 4) + 4 g + r % 4 of the row block,
    // column li of the column block
    constexpr int kOutStride = 68 * 4;
    __syncthreads();
    if (wave == 0)
#pragma unroll
        for (int mb = 0; mb < RB; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    *reinterpret_cast<float *>(fb_smem + (32 * mb + 8 * (r >> 2) + 4 * g + (r & 3)) * kOutStride + (32 * nb + li) * 4) = acc[mb][nb][r];
    __syncthreads();
    for (int x = threadIdx.x; x < 16 * R; x += 64 * kFbWaves) {
        const int row = x >> 4, c = 4 * (x & 15), col = col0 + c;
        if (col >= n_out) continue;  // (n_out is a multiple of 8)
        const f32x4 v = *reinterpret_cast<const f32x4 *>(fb_smem + row * kOutStride + 4 * c);
        float *dst = nullptr;
        if (row < n_bins) dst = d_e_bin + ((size_t)s * n_bins + row) * n_out;
        else if (row < R - 1) dst = d_e_pos + ((size_t)s * n_pos + (row - n_bins)) * n_out;
        else if (s == 0) dst = d_bias;
        if (dst) *reinterpret_cast<f32x4 *>(dst + col) = v;
    }
}

template <int RB, bool MASK>
hipError_t launch_factor_backward(dim3 grid, hipStream_t stream, const int *nbr_idx, const int *nbr_bin, const bf16_t *d_z, const uint8_t *mask,
                                  float *d_e_bin, float *d_e_pos, float *d_bias, int rows, int L, int k, int n_bins, int n_pos, int pos_mode,
                                  int n_out)
{
    constexpr int lds = FbCfg<RB>::kBytes;
    static LdsLimit limit;
    const hipError_t e = raise_lds_limit(limit, (const void *)fipa_factor_backward_kernel<RB, MASK>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fipa_factor_backward_kernel<RB, MASK>), grid, dim3(64 * kFbWaves), lds, stream, nbr_idx, nbr_bin, d_z, mask, d_e_bin, d_e_pos,
                       d_bias, rows, L, k, n_bins, n_pos, pos_mode, n_out);
    return hipGetLastError();
}

}  // namespace
}  // namespace fipa

extern "C" int fipa_factor_project(int32_t B, int32_t L, int32_t k, int32_t n_bins, int32_t n_pos, int32_t pos_mode,
                                   int32_t n_out, const int32_t *nbr_idx, const int32_t *nbr_bin, const void *e_bin,
                                   const void *e_pos, const float *bias, void *z, void *hip_stream)
{
    if (B <= 0 || L <= 0 || k <= 0 || n_bins < 1 || n_out <= 0 || n_pos < 0) return FIPA_ERR_INVALID_ARG;
    if (!nbr_idx || !nbr_bin || !e_bin || !z) return FIPA_ERR_INVALID_ARG;
    if ((n_pos > 0) != (e_pos != nullptr)) return FIPA_ERR_INVALID_ARG;
    if (pos_mode != 0 && pos_mode != 1) return FIPA_ERR_INVALID_ARG;
    if (n_pos > 0 && pos_mode == 1 && n_pos % 2 == 0) return FIPA_ERR_INVALID_ARG;  // offsets -h .. +h
    if (n_out % 8 != 0 || k > 64 || (long long)B * L * k >= (1LL << 31)) return FIPA_ERR_UNSUPPORTED;
    const long long rows = (long long)B * L, threads = rows * (n_out / 8);
    if ((threads + 255) / 256 >= (1LL << 31)) return FIPA_ERR_UNSUPPORTED;
    const void *al16[] = {e_bin, e_pos, z, bias};
    for (const void *ptr : al16)
        if (ptr && !fipa::aligned16(ptr)) return FIPA_ERR_ALIGNMENT;
    if ((reinterpret_cast<uintptr_t>(nbr_idx) & 3u) != 0 || (reinterpret_cast<uintptr_t>(nbr_bin) & 3u) != 0) return FIPA_ERR_ALIGNMENT;
    const dim3 grid((unsigned)((threads + 255) / 256));
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    // One workgroup per compute unit and 32 columns; worth the loading of its table (about 100 KB) from factor_rows residues on.
    const int groups = (n_out + 31) / 32, parts = groups < 256 ? 256 / groups : 1;
    const size_t lds = fipa::factor_lds_bytes(k, n_bins, n_pos);
    if (lds <= 160 * 1024 && (long long)k * (n_bins + n_pos) < 0xFFFF && rows >= (long long)parts * fipa::factor_rows(k) && rows <= (1LL << 30)) {
        static fipa::LdsLimit limit;
        if (fipa::raise_lds_limit(limit, (const void *)fipa::fipa_factor_project_lds_kernel, (int)lds) != hipSuccess) return FIPA_ERR_LAUNCH;
        hipLaunchKernelGGL(fipa::fipa_factor_project_lds_kernel, dim3(groups, parts), dim3(fipa::kFpThreads), lds, stream, nbr_idx, nbr_bin,
                           (const fipa::bf16_t *)e_bin, (const fipa::bf16_t *)e_pos, bias, (fipa::bf16_t *)z, (int)rows, L, k, n_bins, n_pos,
                           pos_mode, n_out);
        return hipGetLastError() == hipSuccess ? FIPA_OK : FIPA_ERR_LAUNCH;
    }
    if (n_pos > 0)
        hipLaunchKernelGGL(fipa::fipa_factor_project_kernel<true>, grid, dim3(256), 0, stream, nbr_idx, nbr_bin,
                           (const fipa::bf16_t *)e_bin, (const fipa::bf16_t *)e_pos, bias, (fipa::bf16_t *)z, rows, L, k,
                           n_bins, n_pos, pos_mode, n_out / 8);
    else
        hipLaunchKernelGGL(fipa::fipa_factor_project_kernel<false>, grid, dim3(256), 0, stream, nbr_idx, nbr_bin,
                           (const fipa::bf16_t *)e_bin, (const fipa::bf16_t *)nullptr, bias, (fipa::bf16_t *)z, rows, L, k,
                           n_bins, 1, pos_mode, n_out / 8);
    return hipGetLastError() == hipSuccess ? FIPA_OK : FIPA_ERR_LAUNCH;
}

extern "C" int fipa_factor_project_backward(int32_t B, int32_t L, int32_t k, int32_t n_bins, int32_t n_pos, int32_t pos_mode,
                                            int32_t n_out, const int32_t *nbr_idx, const int32_t *nbr_bin, const void *d_z,
                                            const uint8_t *mask, float *d_e_bin, float *d_e_pos, float *d_bias,
                                            void *hip_stream)
{
    if (B <= 0 || L <= 0 || k <= 0 || n_bins < 1 || n_out <= 0 || n_pos < 0) return FIPA_ERR_INVALID_ARG;
    if (!nbr_idx || !nbr_bin || !d_z || !d_e_bin) return FIPA_ERR_INVALID_ARG;
    if ((n_pos > 0) != (d_e_pos != nullptr)) return FIPA_ERR_INVALID_ARG;
    if (pos_mode != 0 && pos_mode != 1) return FIPA_ERR_INVALID_ARG;
    if (n_pos > 0 && pos_mode == 1 && n_pos % 2 == 0) return FIPA_ERR_INVALID_ARG;
    if (n_out % 8 != 0 || k > 64 || (long long)B * L * k >= (1LL << 31)) return FIPA_ERR_UNSUPPORTED;
    // the one-hot tile holds 32-row blocks of the slot's rows (bins, position codes, one for the bias)
    const int RB = (n_bins + n_pos + 1 + 31) / 32;
    if (RB > fipa::kFbMaxRowBlocks) return FIPA_ERR_UNSUPPORTED;
    const void *al16[] = {d_z, d_e_bin, d_e_pos, d_bias};
    for (const void *ptr : al16)
        if (ptr && !fipa::aligned16(ptr)) return FIPA_ERR_ALIGNMENT;
    if ((reinterpret_cast<uintptr_t>(nbr_idx) & 3u) != 0 || (reinterpret_cast<uintptr_t>(nbr_bin) & 3u) != 0) return FIPA_ERR_ALIGNMENT;
    const dim3 grid((unsigned)((n_out + 63) / 64), (unsigned)k);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const auto with = [&](auto M) {
        constexpr bool masked = decltype(M)::value;
        return RB == 1   ? fipa::launch_factor_backward<1, masked>
               : RB == 2 ? fipa::launch_factor_backward<2, masked>
               : RB == 3 ? fipa::launch_factor_backward<3, masked>
               : RB == 4 ? fipa::launch_factor_backward<4, masked>
                         : fipa::launch_factor_backward<5, masked>;
    };
    const auto launch = mask ? with(std::true_type{}) : with(std::false_type{});
    return launch(grid, stream, nbr_idx, nbr_bin, (const fipa::bf16_t *)d_z, mask, d_e_bin, n_pos > 0 ? d_e_pos : nullptr, d_bias, B * L, L, k,
                  n_bins, n_pos, pos_mode, n_out) == hipSuccess
               ? FIPA_OK
               : FIPA_ERR_LAUNCH;
}
