// Exact int8-MFMA exemplar-search tile on gfx950 (see search_mfma.hip for
// the arithmetic): staging of a 64 x 64 candidate tile, the B operands of a
// target, and the scoring loop, shared by the one-search-per-launch kernel
// and the persistent fill kernel.
#pragma once

#include "search_tile.h"

namespace inpaint {
namespace mtile {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef v4i v4i_dw __attribute__((aligned(4)));   // at any dword of LDS

constexpr int kMfmaTileH = 64;   // candidate rows of a tile

// The staged window of a 64 x 64 tile.  A wave scores 16 candidate columns as
// four MFMA accumulators s = 0 .. 3 of the candidate rows 4 m + s (m = 0 ..
// 15): accumulator s then needs, for patch row dy, the window rows 4 m + s +
// dy, so one A operand (rows 4 m + v) serves every (s, dy) with s + dy = v.
// P + 3 operands replace the 4 P that four blocks of 16 consecutive rows
// need; the LDS reads of the operands are what bounds the scoring otherwise.
// The rows are stored by residue mod 4 so that the 16 lanes of an operand
// read rows a fixed stride apart: strides of 4 (mod 8) words touch every
// bank once per 8 lanes.
template <int R>
struct MfmaGeom {
    static constexpr int P = 2 * R + 1;
    static constexpr int ROWS = kMfmaTileH + 2 * R;
    static constexpr int RP = (ROWS + 3) / 4;                   // stored rows per residue
    static constexpr int COLS = kTileW + 2 * R;                 // staged columns that meet nonzero B entries
    static constexpr int QA = (COLS + 3) / 4;                   // 16-byte quads per row
    // Patches up to 9 pixels wide meet 24 window pixels per row of a block of
    // 16 columns: 16 pixels of one row fill one MFMA, and the other 8 pixels
    // of two rows share one.  Wider ones take two MFMAs per row.
    static constexpr bool PAIR = R <= 4;
    static constexpr int SA = PAIR ? 76 : 84;                   // words per stored row
    static constexpr int SL = 80;                               // bytes per stored row of |s'|^2 low bytes
    static constexpr int NA = ROWS * QA;
    static constexpr int AIT = (NA + kSearchWaves * 64 - 1) / (kSearchWaves * 64);
    // Stored row of window row y, relative to the operand's lane row (m = 0).
    static constexpr int slot(int y) { return (y & 3) * RP + (y >> 2); }
};

// Byte 3 of a staged word and the byte of the low plane are the two bytes of
// q = |s'|^2 (0 .. 49152), each minus 128 as int8.
template <int R>
struct MfmaTile {
    alignas(16) uint32_t a[4 * MfmaGeom<R>::RP * MfmaGeom<R>::SA];   // (R', G', B', q high)
    alignas(16) uint8_t lo[4 * MfmaGeom<R>::RP * MfmaGeom<R>::SL];   // q low
};

// The target as every wave reads its B operands from.  With T(dy, x) the
// target word at patch column x of row dy -- (R', G', B', -128) where known, 0
// elsewhere, also outside 0 <= x < P and for dy = P -- and M(dy, x) its 0/1
// known flag: t[s][dy][i] = T(dy, i - 16 - s) and m[s][dy][i] = M(dy, i - 16 -
// s), so that what lane (n, g) needs, four words or sixteen bytes starting at
// x = const - n, starts at a multiple of four in copy s = n mod 4.  Only the
// entries of 0 <= x < P are ever written after clear_tables().
template <int R>
struct FragTables {
    static constexpr int P = 2 * R + 1;
    alignas(16) uint32_t t[4][P + 1][48];
    alignas(16) uint8_t m[4][P + 1][48];
    int t2p[kSearchWaves], k[kSearchWaves];
};

// Zeroes the tables (whole work-group, once before the first build; the
// caller's barrier publishes it).
template <int R>
__device__ __forceinline__ void clear_tables(FragTables<R> *ft) {
    uint32_t *w = &ft->t[0][0][0];
    for (int i = threadIdx.x; i < (int)(sizeof(ft->t) / 4); i += kSearchWaves * 64) w[i] = 0;
    uint32_t *b = (uint32_t *)&ft->m[0][0][0];
    for (int i = threadIdx.x; i < (int)(sizeof(ft->m) / 4); i += kSearchWaves * 64) b[i] = 0;
}

// Writes the target's entries from its words (column-major slots x * P + dy)
// and known flags -- `word(slot, round)` and `known(slot, round)` read them
// wherever they are, round r covering slots r * 256 .. -- with the per-wave
// partial sums of T2' and k.  The caller's barrier publishes the tables.
template <int R, class Word, class Known>
__device__ __forceinline__ void build_tables(FragTables<R> *ft, Word word, Known known) {
    constexpr int P = 2 * R + 1, N = P * P, T = kSearchWaves * 64;
    int t2 = 0, kk = 0;
#pragma unroll
    for (int r = 0; r < (N + T - 1) / T; ++r) {
        const int sl = threadIdx.x + r * T;
        const bool in = sl < N, kn = in && known(in ? sl : 0, r);
        const uint32_t w = kn ? (word(sl, r) & 0x00ffffffu) ^ 0x00808080u : 0u;
        t2 = __builtin_amdgcn_sdot4((int)w, (int)w, t2, false);
        kk += __popcll(__ballot(kn));
        if (in) {
            const int x = sl / P, dy = sl - x * P;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                ft->t[s][dy][x + 16 + s] = kn ? w | 0x80000000u : 0u;
                ft->m[s][dy][x + 16 + s] = kn ? 1 : 0;
            }
        }
    }
    t2 = (int)dpp::sum_u32((uint32_t)t2);
    if ((threadIdx.x & 63) == 0) {
        ft->t2p[threadIdx.x >> 6] = t2;
        ft->k[threadIdx.x >> 6] = kk;
    }
}

// First tile column and row of tile `tile` of the MFMA tiling of the rect.
template <int R>
__device__ __forceinline__ void tile_origin(int rx0, int ry0, int ntx, int tile, int *tx0, int *ty0) {
    *tx0 = mfma_tile_x0(rx0, R) + (tile % ntx) * kTileW;
    *ty0 = ry0 + (tile / ntx) * kMfmaTileH;
}

// Issues every load of the tile at (tx0, ty0) -- staged window (padded rows
// ty0 - R + kPadT .., columns tx0 - R + kPadL .., a multiple of 4) and the
// validity radii of this lane's candidates (rows 16 g + j of the tile, column
// tx0 + 16 wave + n) -- then writes the window to LDS in the offset domain
// with the bytes of |s'|^2.  They are formed here, from the source plane the
// SIMT search reads too, rather than kept as planes of their own: a third
// less to load per tile (4 instead of 6 bytes a pixel) for four dot products
// and a few byte moves per 16-byte load.  Returns the lane's validity bits
// (bit j); the caller publishes with a barrier.
template <int R>
__device__ __forceinline__ uint32_t stage_tile(const JobDev &d, int tx0, int ty0, int rx0, int rx1, int ry1,
                                               MfmaTile<R> &L) {
    using G = MfmaGeom<R>;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int pitch = d.pitch;
    const int cx = tx0 + 16 * wave + n;
    const uint4 *src = (const uint4 *)(d.srcp + (int64_t)(ty0 - R + kPadT) * pitch + (tx0 - R + kPadL));
    uint4 va[G::AIT];
#pragma unroll
    for (int k = 0; k < G::AIT; ++k) {
        const int i = min(tid + k * kSearchWaves * 64, G::NA - 1);
        const int ly = i / G::QA, lq = i - ly * G::QA;
        va[k] = src[ly * (pitch >> 2) + lq];
    }
    const uint8_t *vr = d.vradp + (int64_t)(ty0 + 16 * g + kPadT) * pitch + (cx + kPadL);
    uint32_t vv[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) vv[j] = vr[j * pitch];

#pragma unroll
    for (int k = 0; k < G::AIT; ++k) {
        const int i = min(tid + k * kSearchWaves * 64, G::NA - 1);
        const int ly = i / G::QA, lq = i - ly * G::QA;
        const int row = (ly & 3) * G::RP + (ly >> 2);
        const uint32_t in[4] = {va[k].x, va[k].y, va[k].z, va[k].w};
        uint32_t w[4], q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t v = (in[j] & 0x00ffffffu) ^ 0x00808080u;
            q[j] = (uint32_t)__builtin_amdgcn_sdot4((int)v, (int)v, 0, false);
            w[j] = v | (((q[j] << 16) & 0xff000000u) ^ 0x80000000u);
        }
        *(uint4 *)&L.a[row * G::SA + 4 * lq] = make_uint4(w[0], w[1], w[2], w[3]);
        const uint32_t l01 = (q[0] & 255u) | (q[1] & 255u) << 8, l23 = (q[2] & 255u) | (q[3] & 255u) << 8;
        *(uint32_t *)&L.lo[row * G::SL + 4 * lq] = (l01 | l23 << 16) ^ 0x80808080u;
    }
    uint32_t vmask = 0;
    const bool colok = cx >= rx0 && cx < rx1;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (colok && ty0 + 16 * g + j < ry1 && vv[j] >= (uint32_t)R) vmask |= 1u << j;
    return vmask;
}

// Scores this lane's candidates of a staged tile and returns their minimum
// key (~0 if none is valid).  Accumulator s, element i of lane (n, g) is the
// candidate at tile row 16 g + 4 i + s, column 16 wave + n.
//
// Per 16 candidate rows and columns, patches up to 9 pixels wide take P + R + 1
// MFMAs for the cross term and the high byte of |s'|^2 (which rides in the
// words' fourth byte against a B byte of -128: -2 acc then carries 256 q_hi)
// and R + 1 for the low byte (32 bytes of two rows each): 19 at 9x9, where
// operands of four full rows and separate byte planes took 36.  LDS reads per
// wave fall from 108 + 54 to 36 + 19 at 9x9.
template <int R>
__device__ __forceinline__ uint64_t score_tile_rows(const JobDev &d, const FragTables<R> *ft, int tx0, int ty0,
                                                    uint32_t vmask, const MfmaTile<R> &L) {
    using G = MfmaGeom<R>;
    constexpr int P = G::P, V = P + 3;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, g = lane >> 4, s4 = n & 3;
    const int W = d.W, cx = tx0 + 16 * wave + n;
    int t2 = 0, kk = 0;
#pragma unroll
    for (int w = 0; w < kSearchWaves; ++w) {
        t2 += ft->t2p[w];
        kk += ft->k[w];
    }
    t2 = __builtin_amdgcn_readfirstlane(t2);
    kk = __builtin_amdgcn_readfirstlane(kk);
    v4i acc[4], al[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        acc[s] = v4i{0, 0, 0, 0};
        al[s] = v4i{0, 0, 0, 0};
    }
    // Operands over two rows: lanes g >= 2 read the next row, which is RP
    // stored rows on, or (after residue 3) back to residue 0.
    const int g1 = g & 1, gh = g >> 1;
    const uint32_t *ax = &L.a[n * G::SA + 16 * wave + 4 * g];
    const uint32_t *ay = &L.a[n * G::SA + 16 * wave + 16 + 4 * g1];
    const uint8_t *lb = &L.lo[n * G::SL + 16 * wave + 16 * g1];
    const int step = gh * G::RP, wrap = gh * (1 - 3 * G::RP);
    const uint32_t *bx = &ft->t[s4][0][16 + 4 * g - 4 * (n >> 2)];
    const uint32_t *by = &ft->t[s4][gh][32 + 4 * g1 - 4 * (n >> 2)];
    const uint8_t *bm = &ft->m[s4][gh][16 + 16 * g1 - 4 * (n >> 2)];
    v4i b0[P], b1[P], bp[R + 1], bl[R + 1];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int row = G::slot(v), next = (v & 3) == 3 ? wrap : step;
        const v4i a0 = *(const v4i *)&ax[row * G::SA];
        const v4i a1 = G::PAIR ? *(const v4i *)&ay[(row + next) * G::SA] : *(const v4i *)&ax[row * G::SA + 16];
        const v4i a2 = *(const v4i *)&lb[(row + next) * G::SL];
        if (v < P) {
            b0[v] = *(const v4i *)&bx[v * 48];
            if (!G::PAIR) b1[v] = *(const v4i *)&bx[v * 48 + 16];
            if ((v & 1) == 0) {
                if (G::PAIR) bp[v >> 1] = *(const v4i *)&by[v * 48];
                bl[v >> 1] = *(const v4i_dw *)&bm[v * 48];
            }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int dy = v - s;
            if (dy < 0 || dy >= P) continue;
            acc[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, b0[dy], acc[s], 0, 0, 0);
            if (!G::PAIR) acc[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, b1[dy], acc[s], 0, 0, 0);
            if (dy & 1) continue;
            if (G::PAIR) acc[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, bp[dy >> 1], acc[s], 0, 0, 0);
            al[s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a2, bl[dy >> 1], al[s], 0, 0, 0);
        }
    }
    // SSD = base + al - 2 acc.  The lane's candidates share a column and its
    // bits run down the rows, so the first minimum is that of (SSD - base +
    // kBias, bit) packed in one word: -base <= SSD - base <= 3 P^2 255^2, and
    // both fit 28 bits with the bias at every radius.  One word per candidate
    // in place of a 64-bit key, a compare and two selects: 6 instructions of 14.
    constexpr int kBias = 1 << 25;
    static_assert(P * P * (49152 + 256 * 128 + 128) < kBias && kBias + 3 * 255 * 255 * P * P < (1 << 28), "28 + 4 bits");
    const uint32_t gone = ~vmask;
    uint32_t low = ~0u;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t j = 4 * i + s, v = (uint32_t)(al[s][i] - 2 * acc[s][i] + kBias);
            low = min(low, v << 4 | j | (uint32_t)((int)(gone << (31 - j)) >> 31));
        }
    }
    const int base = t2 + kk * (256 * 128 + 128) - kBias;
    const uint32_t ssd = (low >> 4) + (uint32_t)base, y = (uint32_t)(ty0 + 16 * g) + (low & 15u);
    return vmask ? (uint64_t)ssd << 32 | (y * (uint32_t)W + (uint32_t)cx) : ~0ull;
}

}  // namespace mtile
}  // namespace inpaint
