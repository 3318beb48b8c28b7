// One fill iteration around the exemplar search on gfx950: the LDS copy of
// the target's neighbourhood, the search-independent half of the commit, the
// half that needs the source patch, the choice of the next target and the
// upkeep of the priority maxima.  Shared by the stream-form commit kernels
// and the persistent committer; one work-group of kCommitThreads per image.
//
// A commit is a chain of short steps on at most a few thousand pixels, so
// what bounds it is the number of instructions on that chain and the number
// of barriers and memory round trips in it, not bandwidth: four waves issue
// one vector instruction each per four cycles.  Hence the layout below: no
// integer division by a run-time value, one 32-bit word per pixel for colour
// and state, gradients kept instead of being formed again, and
// the maxima of untouched priority blocks kept in superblocks.  Persistent
// MFMA form, 1080p, us an iteration: 14.2 -> 8.2 at 9x9, 18.1 -> 11.7 at 13x13;
// the stream-form commit 13.2 -> 9.8 us a launch (640x480, 9x9).
//
// Priorities are binary64 and must match a plain sequential CPU evaluation
// bit for bit: FP contraction is off and every sum runs in the fixed raster
// order of the patch offsets.
#pragma once

#include "search_tile.h"

#pragma clang fp contract(off)

namespace inpaint {

// The functions below take the thread's number.  What they derive from it is
// the same in every iteration, far more than the registers hold; the loop of
// the persistent committer hands them a number that the compiler cannot see
// through, so that it is formed again instead of spilled (1080p 9x9: SIMT form
// 74.7 -> 56.4 ms a removal, MFMA form level).
__device__ __forceinline__ int thread_number() {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}

constexpr int kSlots = 2;   // patch slots per thread: 17 x 17 over 256 threads

// Neighbourhood staged around the target: the refresh window reaches 2r+1
// from it, a priority reads its patch (r) and the gradients there.
template <int R>
struct Stage {
    static constexpr int P = 2 * R + 1;
    static constexpr int half = 3 * R + 2;
    static constexpr int side = 2 * half + 1;
    static constexpr int cols = side <= 32 ? 32 : side;    // staged per row: a power of two where it is cheap
    static constexpr int pitch = cols | 1;                 // odd: a column of pixels spreads over the LDS banks
    static constexpr int n = cols * side;
    static constexpr int reach = 2 * R + 1;
    static constexpr int WIN = 2 * reach + 1;              // refresh window side
    static constexpr int NBA = (WIN + 6) / 8 + 1;          // 8x8 blocks it can touch per axis
    static constexpr int KP = 8 * NBA;                     // side of the touched blocks' pixels
    static constexpr int BP = KP % 16 ? KP : KP + 8;       // their pitch in LDS: rows of two blocks on other banks
    static constexpr int at(int dx, int dy) { return (dy + half) * pitch + (dx + half); }
};

// Pixel state in the fourth byte of an image word.
constexpr uint32_t kStateHole = 1u << 24, kStateOut = 2u << 24, kColour = 0x00ffffffu;
__device__ __forceinline__ uint32_t state_of(uint32_t w) { return w >> 24; }

// Integer BT.601 gray of an RGBX word.
__device__ __forceinline__ int gray_of(uint32_t w) {
    return (int)((299 * (w & 255) + 587 * ((w >> 8) & 255) + 114 * ((w >> 16) & 255) + 500) / 1000);
}

// A gradient as kept: gx in the low and gy in the high 16 bits, 0 where the
// pixel or one of its four neighbours is not known (a zero gradient and none
// give the same isophote).  In global memory a known pixel's gradient sits in
// the priority terms' D, which only front pixels, never known ones, use.
__device__ __forceinline__ uint32_t pack_grad(int gx, int gy) { return (uint32_t)(gx & 0xffff) | (uint32_t)gy << 16; }
typedef const uint32_t __attribute__((may_alias)) GradWord;   // read there
__device__ __forceinline__ GradWord *grad_word(const double2 *cd) { return (GradWord *)&cd->y; }
__device__ __forceinline__ double2 off_front(uint32_t grad) {
    return make_double2(-1.0, __longlong_as_double((long long)grad));
}
typedef short short2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int grad_size(uint32_t g) {
    const short2_t v = __builtin_bit_cast(short2_t, g);
    return __builtin_amdgcn_sdot2(v, v, 0, false);
}

__device__ __forceinline__ bool in_img(const JobDev &d, int x, int y) {
    return (unsigned)x < (unsigned)d.W && (unsigned)y < (unsigned)d.H;
}

// Column and row of a raster index (0 <= i < W * H < 2^31) by a reciprocal
// taken once: m = floor(2^32 / W) gives the row or one less, as i < 2^32.
struct Raster {
    uint32_t W, m;
    __device__ explicit Raster(int w) : W((uint32_t)w), m(0xffffffffu / (uint32_t)w) {}
    __device__ __forceinline__ void split(uint32_t i, int *x, int *y) const {
        uint32_t q = __umulhi(i, m), r = i - q * W;
        while (r >= W) {   // at most twice: m may be one below floor(2^32 / W)
            r -= W;
            ++q;
        }
        *x = (int)r;
        *y = (int)q;
    }
};

// Barrier over LDS contents alone.  __syncthreads also waits for every global
// store in flight, half a microsecond when one was just issued; the commit's
// stores are read back only after the full barrier that ends an iteration.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- (key, index) maxima: the greater key wins, equal keys go to the lower
// index, a strict total order.  Keys are -1 (none) or the bits of a
// non-negative double.
struct Best {
    int64_t key;
    uint32_t idx;
};
__device__ __forceinline__ Best no_best() { return {-1, 0xffffffffu}; }
__device__ __forceinline__ bool better(int64_t ka, uint32_t ia, int64_t kb, uint32_t ib) {
    return ka > kb || (ka == kb && ia < ib);
}
__device__ __forceinline__ void take(Best &b, int64_t key, uint32_t idx) {
    if (better(key, idx, b.key, b.idx)) b = {key, idx};
}
__device__ __forceinline__ uint32_t max_u32(uint32_t v) {
    return dpp::fold_wave(v, [](uint32_t a, uint32_t b) { return b > a ? b : a; });
}
// The wave's maximum, in every lane (all lanes active): the key's high word,
// then its low word and the index among the lanes that still match.  Three
// one-word folds of single DPP instructions are a third of the instructions of
// a fold over the pairs.
__device__ __forceinline__ Best wave_best(Best b) {
    const uint64_t e = (uint64_t)(b.key + 1);   // 0: none
    const uint32_t hi = (uint32_t)(e >> 32), lo = (uint32_t)e;
    const uint32_t mh = max_u32(hi);
    const uint32_t ml = max_u32(hi == mh ? lo : 0u);
    const uint32_t mi = max_u32(hi == mh && lo == ml ? ~b.idx : 0u);
    return {(int64_t)((uint64_t)mh << 32 | ml) - 1, ~mi};
}
// The wave's minimum of 64-bit words.
__device__ __forceinline__ uint64_t wave_min(uint64_t v) {
    const uint64_t e = ~v;
    const uint32_t hi = (uint32_t)(e >> 32), lo = (uint32_t)e;
    const uint32_t mh = max_u32(hi), ml = max_u32(hi == mh ? lo : 0u);
    return ~((uint64_t)mh << 32 | ml);
}

// State of the fill loop at the start of an iteration; uniform.
struct Snap {
    int64_t iter, limit, remaining;
    uint32_t p;
    double C, D, Pr;
    int32_t done, err, pending;
};

__device__ __forceinline__ Snap load_snap(const IterState *st) {
    return {st->iter, st->iter_limit, st->remaining, (uint32_t)st->p_idx, st->C, st->D, st->Pr,
            st->done, st->error, st->pending};
}

// Superblocks: 2^sshift x 2^sshift priority blocks of the priority range,
// d.nsx per row, at most kMaxSuper.
__device__ __forceinline__ int super_count(const JobDev &d) { return d.nsx * d.nsy; }

template <int R>
struct CommitLds {
    using S = Stage<R>;
    double conf[S::pitch * S::side];   // C of known pixels, +0.0 elsewhere
    uint32_t img[S::pitch * S::side];  // colour and state
    uint32_t grad[S::pitch * S::side]; // pack_grad
    int64_t bkey[S::BP * S::KP];  // priority keys of the touched blocks' pixels
    double fC[S::WIN * S::WIN];   // confidence term of each listed front pixel
    int16_t front[S::WIN * S::WIN];   // window index of each front pixel of the refresh window
    int nfront;
    uint8_t gray[(S::P + 4) * (S::P + 4)];   // of the patch and two pixels around it
    // work-group folds, one set of words per use
    int64_t fk[2][4];
    uint32_t fi[2][4];
    double wC[4], wD[4];          // terms of each wave's best new front pixel
    uint64_t smin[4];
    int cnt[4], late[4];
    Best part[4];                 // untouched blocks of each touched superblock
    int64_t bmk[S::NBA * S::NBA];     // maxima of the touched blocks
    uint32_t bmi[S::NBA * S::NBA];
    uint32_t tword[S::P * S::P];  // the staged target words (colour, known in bit 31)
};

// Geometry of one iteration: the window of pixels whose priority can change
// (within 2r+1 of the filled target, clipped to the image), the 8x8 blocks
// it touches and the superblocks they lie in (at most two per axis).
struct Refresh {
    int wx0, wx1, wy0, wy1;
    int abx0, aby0, nabx, naby;
    int sx0, sy0, sx1, sy1;
};
template <int R>
__device__ __forceinline__ Refresh refresh_geometry(const JobDev &d, int px, int py) {
    constexpr int reach = Stage<R>::reach;
    Refresh g;
    g.wx0 = max(px - reach, 0);
    g.wx1 = min(px + reach + 1, d.W);
    g.wy0 = max(py - reach, 0);
    g.wy1 = min(py + reach + 1, d.H);
    g.abx0 = g.wx0 >> 3;
    g.aby0 = g.wy0 >> 3;
    g.nabx = ((g.wx1 - 1) >> 3) - g.abx0 + 1;
    g.naby = ((g.wy1 - 1) >> 3) - g.aby0 + 1;
    // (the window lies in the priority range: the hole's box grown by 2r+1)
    g.sx0 = (g.abx0 - d.pbx0) >> d.sshift;
    g.sy0 = (g.aby0 - d.pby0) >> d.sshift;
    g.sx1 = (g.abx0 + g.nabx - 1 - d.pbx0) >> d.sshift;
    g.sy1 = (g.aby0 + g.naby - 1 - d.pby0) >> d.sshift;
    return g;
}

// Priority key from the cached terms: bits of P = C * D (Eq. 1), -1 off the
// front.  Non-negative doubles order like their bit patterns.
__device__ __forceinline__ int64_t key_of(double2 cd) {
    return cd.x < 0.0 ? -1 : __double_as_longlong(cd.x * cd.y);
}

// Reads everything of the commit that does not depend on the search: the
// target's neighbourhood and the touched blocks' keys into LDS, and this
// thread's share of the maximum over every pixel whose priority stays --
// superblocks that are not touched (`sup`, in LDS or global memory), the
// untouched blocks of the touched ones (wave w scans the w-th) and the
// touched blocks' pixels outside the window.  All loads are issued, from
// clamped addresses, before any is consumed.
template <int R>
__device__ __forceinline__ Best gather(int tid, const JobDev &d, int px, int py, const Refresh &g, const BlockBest *sup,
                                       CommitLds<R> &L) {
    using S = Stage<R>;
    constexpr int T = kCommitThreads;
    constexpr int NIT = (S::n + T - 1) / T, KIT = (S::KP * S::KP + T - 1) / T;
    const int lane = tid & 63, wave = tid >> 6;
    const int ox = px - S::half, oy = py - S::half;
    const int W = d.W;

    // the w-th touched superblock, its blocks one per lane and round
    const int sx = g.sx0 + (wave & 1), sy = g.sy0 + (wave >> 1);
    const bool has = sx <= g.sx1 && sy <= g.sy1;
    const int sh = d.sshift;
    const int bx0 = d.pbx0 + (sx << sh), by0 = d.pby0 + (sy << sh);
    const int brow = lane >> 3, bcol = lane & 7;   // 8 x 8 blocks per round
    BlockBest bb = {-1, INT64_MAX};
    const auto load_block = [&](int bx, int by) {
        BlockBest v = d.blk[min(by, d.pby1 - 1) * d.nbw + min(bx, d.pbx1 - 1)];
        const bool touched = (unsigned)(bx - g.abx0) < (unsigned)g.nabx && (unsigned)(by - g.aby0) < (unsigned)g.naby;
        if (bx >= d.pbx1 || by >= d.pby1 || touched) v.key = -1;
        return v;
    };
    if (has) bb = load_block(bx0 + bcol, by0 + brow);

    uint32_t im[NIT], gr[NIT];
    double c[NIT];
    double2 cd[KIT];
    const int kx0 = g.abx0 * 8, ky0 = g.aby0 * 8;
    // Away from the image border every slot of the thread grid is a pixel:
    // no clamps, and small byte offsets from uniform bases.
    constexpr int SR = (NIT * T + S::cols - 1) / S::cols, KR = (KIT * T + S::KP - 1) / S::KP;   // rows of the grids
    const bool inner = W <= 65536 && ox >= 0 && oy >= 0 && ox + S::cols <= W && oy + SR <= d.H && kx0 + S::KP <= W &&
                       ky0 + KR <= d.H;
    if (inner) {
        const int64_t o = (int64_t)oy * W + ox, ko = (int64_t)ky0 * W + kx0;
        const uint32_t *pi = d.img + o;
        GradWord *pg = grad_word(d.pcd + o);
        const double *pc = d.conf + o;
        const double2 *pk = d.pcd + ko;
#pragma unroll
        for (int k = 0; k < NIT; ++k) {
            const int t = tid + k * T;
            const uint32_t i = (uint32_t)(t / S::cols) * (uint32_t)W + (uint32_t)(t % S::cols);
            im[k] = *(const uint32_t *)((const char *)pi + 4 * i);
            c[k] = *(const double *)((const char *)pc + 8 * i);
            gr[k] = *(GradWord *)((const char *)pg + 16 * i);
        }
#pragma unroll
        for (int k = 0; k < KIT; ++k) {
            const int t = tid + k * T;
            cd[k] = *(const double2 *)((const char *)pk + 16 * ((uint32_t)(t / S::KP) * (uint32_t)W + (uint32_t)(t % S::KP)));
        }
    } else {
#pragma unroll
        for (int k = 0; k < NIT; ++k) {
            const int t = tid + k * T, lx = ox + t % S::cols, ly = oy + t / S::cols;
            const uint32_t i = (uint32_t)(min(max(ly, 0), d.H - 1) * W + min(max(lx, 0), W - 1));
            im[k] = in_img(d, lx, ly) ? d.img[i] : kStateOut;
            c[k] = d.conf[i];
            gr[k] = *grad_word(d.pcd + i);
        }
#pragma unroll
        for (int k = 0; k < KIT; ++k) {
            const int t = tid + k * T, x = kx0 + t % S::KP, y = ky0 + t / S::KP;
            cd[k] = d.pcd[(uint32_t)(min(y, d.H - 1) * W + min(x, W - 1))];
            if (x >= W || y >= d.H) cd[k].x = -1.0;
        }
    }

    // ---- consume
    Best best = no_best();
    const int ns = super_count(d);
    const int e0 = g.sy0 * d.nsx + g.sx0, e1 = g.sy0 * d.nsx + g.sx1, e2 = g.sy1 * d.nsx + g.sx0,
              e3 = g.sy1 * d.nsx + g.sx1;
    for (int e = tid; e < ns; e += T) {
        const BlockBest v = sup[e];
        if (e != e0 && e != e1 && e != e2 && e != e3) take(best, v.key, (uint32_t)v.idx);
    }
    Best part = {bb.key, (uint32_t)bb.idx};
    if (has)
        for (int q = 1; q < 1 << (2 * (sh - 3)); ++q) {   // larger superblocks of very large holes
            const BlockBest v = load_block(bx0 + bcol + 8 * (q & ((1 << (sh - 3)) - 1)), by0 + brow + 8 * (q >> (sh - 3)));
            take(part, v.key, (uint32_t)v.idx);
        }
    part = wave_best(part);
    if (lane == 0) L.part[wave] = part;
    take(best, part.key, part.idx);
#pragma unroll
    for (int k = 0; k < NIT; ++k) {
        const int t = tid + k * T;
        if ((k + 1) * T <= S::n || t < S::n) {
            const int li = (t / S::cols) * S::pitch + t % S::cols;
            L.img[li] = im[k];
            L.grad[li] = state_of(im[k]) == 0 ? gr[k] : 0u;
            L.conf[li] = state_of(im[k]) == 0 ? c[k] : 0.0;
        }
    }
    // pixels outside the window keep their keys (those in it are filled, off
    // the front or evaluated again)
    const uint32_t vx0 = g.wx0 - kx0, vy0 = g.wy0 - ky0, vw = g.wx1 - g.wx0, vh = g.wy1 - g.wy0;
#pragma unroll
    for (int k = 0; k < KIT; ++k) {
        const int t = tid + k * T;
        if ((k + 1) * T <= S::KP * S::KP || t < S::KP * S::KP) {
            const int col = t % S::KP, row = t / S::KP;
            const bool in = col < 8 * g.nabx && row < 8 * g.naby;
            const int64_t key = in ? key_of(cd[k]) : -1;
            L.bkey[row * S::BP + col] = key;
            if ((uint32_t)col - vx0 >= vw || (uint32_t)row - vy0 >= vh)
                take(best, key, (uint32_t)((ky0 + row) * W + kx0 + col));
        }
    }
    return best;
}

// A patch in registers, raster slots tid + 256 j ... (dx = t % P - R): which of
// them the copy fills.
struct FillSlots {
    bool fill[kSlots];
};

// The target patch's hole pixels take the target's confidence and leave the
// hole and, in LDS, the front; their colours follow with copy_colours, their
// terms in device memory with refresh_grads (one writer: nothing orders two
// waves' stores to one word within an iteration).  keep(t): whether hole slot
// t is filled (INTERSECT scoring fills only those whose source pixel
// qualifies).  L.cnt gets each wave's count of filled slots.
template <int R, class Keep>
__device__ __forceinline__ FillSlots mark_filled(int tid, const JobDev &d, int px, int py, double C, const Refresh &g,
                                                 CommitLds<R> &L, Keep keep) {
    using S = Stage<R>;
    constexpr int P = S::P;
    FillSlots f;
    int n = 0;
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
        f.fill[j] = false;
        if (j * kCommitThreads >= P * P) continue;
        const int t = tid + j * kCommitThreads;
        const int dx = t % P - R, dy = t / P - R, li = S::at(dx, dy);
        if (t < P * P && (L.img[li] & kStateHole) && keep(t)) {
            f.fill[j] = true;
            const int x = px + dx, y = py + dy;
            const uint32_t dst = (uint32_t)(y * d.W + x);
            d.conf[dst] = C;
            d.hole[dst] = 0;
            L.img[li] = 0;
            L.conf[li] = C;
            L.bkey[(y - 8 * g.aby0) * S::BP + (x - 8 * g.abx0)] = -1;
        }
        n += __popcll(__ballot(f.fill[j]));
    }
    if ((tid & 63) == 0) L.cnt[tid >> 6] = n;
    return f;
}

__device__ __forceinline__ int filled_count(const int *cnt) { return cnt[0] + cnt[1] + cnt[2] + cnt[3]; }

// Pixels of the refresh window on the front (a hole pixel with a known
// in-image 4-neighbour) go to a compact list, one atomic per wave.  Pixels
// off the front already carry C = -1 in global memory and key -1 in LDS: a
// hole pixel off the front has never been on it (the front only gains hole
// pixels), a known one was set when it was filled or at initialisation (one
// that this iteration fills gets C = -1 with its gradient).
//
// PATCH: the target's whole patch counts as known, so the list does not wait
// for mark_filled, which clears those pixels at the same time.
template <int R, bool PATCH>
__device__ __forceinline__ void list_front(int tid, CommitLds<R> &L) {
    using S = Stage<R>;
    constexpr int N = S::WIN * S::WIN;
#pragma unroll
    for (int k = 0; k < (N + kCommitThreads - 1) / kCommitThreads; ++k) {
        const int t = tid + k * kCommitThreads;
        const int dx = min(t, N - 1) % S::WIN - S::reach, dy = min(t, N - 1) / S::WIN - S::reach, li = S::at(dx, dy);
        const uint32_t c = L.img[li], e = L.img[li + 1], w = L.img[li - 1], n = L.img[li - S::pitch],
                       s = L.img[li + S::pitch];
        bool on = t < N && state_of(c) == 1;
        if (PATCH) {
            const uint32_t ux = dx + R, uy = dy + R;   // 0 .. 2R inside the patch
            const bool cx = ux <= 2 * R, cy = uy <= 2 * R;
            const auto known = [](uint32_t v, bool in_patch) { return in_patch ? state_of(v) != 2 : state_of(v) == 0; };
            on = on && !(cx && cy) &&
                 (known(e, ux + 1 <= 2 * R && cy) || known(w, ux - 1 <= 2 * R && cy) || known(n, cx && uy - 1 <= 2 * R) ||
                  known(s, cx && uy + 1 <= 2 * R));
        } else {
            on = on && (state_of(e) == 0 || state_of(w) == 0 || state_of(n) == 0 || state_of(s) == 0);
        }
        const uint64_t b = __ballot(on);
        if (b == 0) continue;
        int at = 0;
        if ((tid & 63) == 0) at = atomicAdd(&L.nfront, (int)__popcll(b));
        at = __builtin_amdgcn_readfirstlane(at);
        if (on) L.front[at + __popcll(b & ((1ull << (tid & 63)) - 1))] = (int16_t)t;
    }
}

// Confidence term of each listed front pixel (Eq. 2): the sum of C over the
// known pixels of its patch in raster order of the offsets (unknown ones add
// +0.0, which leaves the running sum bit-identical), over the constant patch
// area.  One pixel per lane.
template <int R>
__device__ __forceinline__ void confidence_terms(int tid, CommitLds<R> &L) {
    using S = Stage<R>;
    constexpr int P = S::P;
    const int nf = L.nfront;
    for (int f = tid; f < nf; f += kCommitThreads) {
        const int wi = L.front[f];
        const double *cf = &L.conf[S::at(wi % S::WIN - S::reach - R, wi / S::WIN - S::reach - R)];
        double sum = 0.0;
        // (a few rows of loads in flight; P is odd, so the rounds end with single rows)
        constexpr int RB = P <= 9 ? 3 : 2;
#pragma unroll 1
        for (int dy = 0; dy + RB <= P; dy += RB) {
            double v[RB][P];
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int dx = 0; dx < P; ++dx) v[r][dx] = cf[(dy + r) * S::pitch + dx];
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int dx = 0; dx < P; ++dx) sum = sum + v[r][dx];
        }
#pragma unroll
        for (int dy = P / RB * RB; dy < P; ++dy)
#pragma unroll
            for (int dx = 0; dx < P; ++dx) sum = sum + cf[dy * S::pitch + dx];
        L.fC[f] = sum / (double)(P * P);
    }
}

// Gray values of the patch and two pixels around it, before the copy.
template <int R>
__device__ __forceinline__ void stage_gray(int tid, CommitLds<R> &L) {
    using S = Stage<R>;
    constexpr int G = S::P + 4;
#pragma unroll
    for (int k = 0; k < (G * G + kCommitThreads - 1) / kCommitThreads; ++k) {
        const int t = tid + k * kCommitThreads;
        if (t < G * G) L.gray[t] = (uint8_t)gray_of(L.img[S::at(t % G - R - 2, t / G - R - 2)]);
    }
}

// Copies the source patch's colours into the filled slots.
template <int R>
__device__ __forceinline__ void copy_colours(int tid, const JobDev &d, int px, int py, int qx, int qy, const FillSlots &f,
                                             CommitLds<R> &L) {
    using S = Stage<R>;
    constexpr int P = S::P, G = P + 4;
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
        if (j * kCommitThreads >= P * P) continue;
        const int t = tid + j * kCommitThreads;
        if (f.fill[j]) {
            const int dx = t % P - R, dy = t / P - R;
            const uint32_t pix = d.img[(uint32_t)((qy + dy) * d.W + (qx + dx))], dst = (uint32_t)((py + dy) * d.W + (px + dx));
            const uint8_t gv = (uint8_t)gray_of(pix);
            d.img[dst] = pix;
            d.gray[dst] = gv;
            L.img[S::at(dx, dy)] = pix;
            L.gray[(dy + R + 2) * G + (dx + R + 2)] = gv;
        }
    }
}

// Gradients the copy changed: those within one pixel of the patch, which holds
// every pixel that left the front.  An iteration that empties the hole skips
// this: no later one reads its terms, and an import forms them all again.
template <int R>
__device__ __forceinline__ void refresh_grads(int tid, const JobDev &d, int px, int py, CommitLds<R> &L) {
    using S = Stage<R>;
    constexpr int Q = S::P + 2, G = S::P + 4;
#pragma unroll
    for (int k = 0; k < (Q * Q + kCommitThreads - 1) / kCommitThreads; ++k) {
        const int t = tid + k * kCommitThreads;
        if (t < Q * Q) {
            const int dx = t % Q - R - 1, dy = t / Q - R - 1, li = S::at(dx, dy);
            const uint8_t *gp = &L.gray[(dy + R + 2) * G + (dx + R + 2)];
            const uint32_t any = (L.img[li] | L.img[li + 1] | L.img[li - 1] | L.img[li + S::pitch] | L.img[li - S::pitch]) >> 24;
            const uint32_t v = any == 0 ? pack_grad((int)gp[1] - (int)gp[-1], (int)gp[G] - (int)gp[-G]) : 0u;
            L.grad[li] = v;
            if (state_of(L.img[li]) == 0) d.pcd[(uint32_t)((py + dy) * d.W + (px + dx))] = off_front(v);
        }
    }
}

// D of Eq. 2: the isophote (-gy, gx) / 2 at the known pixel of the patch with
// the largest central-difference gradient, dotted with the unit normal of the
// front (central differences of the hole indicator, out-of-image pixels
// counted as hole), absolute value, over 255.
__device__ __forceinline__ double data_term(uint32_t grad, int nx, int ny, double norm1, double norm2) {
    const int kn = nx * nx + ny * ny;
    const int gx = (int)(int16_t)(grad & 0xffff), gy = (int)grad >> 16;
    int a = gx * ny - gy * nx;
    if (a < 0) a = -a;
    return kn == 0 ? 0.0 : (0.5 * (double)a) / (kn == 1 ? norm1 : norm2);
}

// New terms of the listed front pixels, four lanes per pixel: each lane
// searches a quarter of the patch rows for the largest gradient (first in
// raster order on ties).  Terms go to global memory and the touched blocks'
// keys; each wave leaves its best pixel in L.fk[1] / fi[1] / wC / wD.
template <int R>
__device__ __forceinline__ void data_terms(int tid, const JobDev &d, int px, int py, const Refresh &g, CommitLds<R> &L) {
    using S = Stage<R>;
    constexpr int P = S::P;
    const int part = tid & 3, nf = L.nfront;
    Best best = no_best();
    double bC = 0.0, bD = 0.0;
    const int y0 = part * P / 4, y1 = (part + 1) * P / 4;
    // (every lane of a wave takes every round: the quarters combine across lanes)
    for (int f0 = (tid >> 6) * 16; f0 < nf; f0 += kCommitThreads / 4) {
        const int f = f0 + ((tid & 63) >> 2);
        const bool on = f < nf;
        const int wi = on ? L.front[f] : 0;
        const int wx = wi % S::WIN - S::reach, wy = wi / S::WIN - S::reach;
        // size << 9 | (511 - position): the larger gradient, the earlier
        // position on ties.  Rows past the lane's quarter repeat its last one.
        uint32_t b = 0;
        const uint32_t *gp = &L.grad[S::at(wx - R, wy - R)];
#pragma unroll
        for (int r = 0; r < (P + 3) / 4; ++r) {
            const int dy = max(min(y0 + r, y1 - 1), 0);
            const uint32_t *row = gp + dy * S::pitch;
            const uint32_t at = 511 - dy * P;
#pragma unroll
            for (int dx = 0; dx < P; ++dx) b = max(b, (uint32_t)grad_size(row[dx]) << 9 | (at - dx));
        }
        b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0xb1, 0xf, 0xf, true));   // quad lanes 1, 0, 3, 2
        b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0x4e, 0xf, 0xf, true));   // 2, 3, 0, 1
        const int best_at = 511 - (int)(b & 511);
        const uint32_t bg = gp[best_at / P * S::pitch + best_at % P];
        if (on && part == 0) {
            const int li = S::at(wx, wy);
            const int nx = (state_of(L.img[li + 1]) != 0) - (state_of(L.img[li - 1]) != 0);
            const int ny = (state_of(L.img[li + S::pitch]) != 0) - (state_of(L.img[li - S::pitch]) != 0);
            const double C = L.fC[f], D = data_term(bg, nx, ny, d.norm1, d.norm2);
            const int x = px + wx, y = py + wy;
            const uint32_t idx = (uint32_t)(y * d.W + x);
            d.pcd[idx] = make_double2(C, D);
            const int64_t key = __double_as_longlong(C * D);
            L.bkey[(y - 8 * g.aby0) * S::BP + (x - 8 * g.abx0)] = key;
            if (better(key, idx, best.key, best.idx)) {
                best = {key, idx};
                bC = C;
                bD = D;
            }
        }
    }
    const Best w = wave_best(best);
    const int wave = tid >> 6;
    if ((tid & 63) == 0) {
        L.fk[1][wave] = w.key;
        L.fi[1][wave] = w.idx;
    }
    if (w.key >= 0 && best.key == w.key && best.idx == w.idx) {   // (an index is one lane's)
        L.wC[wave] = bC;
        L.wD[wave] = bD;
    }
}

// This thread's share of a work-group maximum, posted; after a barrier
// posted_best() reads the whole.
template <int R>
__device__ __forceinline__ void post_best(CommitLds<R> &L, Best b) {
    b = wave_best(b);
    if (threadIdx.x == 0) L.nfront = 0;   // (for the list that follows the barrier)
    if ((threadIdx.x & 63) == 0) {
        L.fk[0][threadIdx.x >> 6] = b.key;
        L.fi[0][threadIdx.x >> 6] = b.idx;
    }
}
template <int R>
__device__ __forceinline__ Best posted_best(const CommitLds<R> &L, int set, int *wave = nullptr) {
    Best b = {L.fk[set][0], L.fi[set][0]};
    int at = 0;
#pragma unroll
    for (int q = 1; q < 4; ++q)
        if (better(L.fk[set][q], L.fi[set][q], b.key, b.idx)) {
            b = {L.fk[set][q], L.fi[set][q]};
            at = q;
        }
    if (wave) *wave = at;
    return b;
}

// Brings the block maxima of the touched blocks and the maxima of their
// superblocks (d.sup and, when not null, the LDS copy `sup`) up to date from
// L.bkey, and fills no part of the choice of the next target: the persistent
// committer runs it while the next search is under way.  16 threads per
// block, 4 keys each; then wave w folds the w-th touched superblock.
template <int R>
__device__ __forceinline__ void update_blocks(int tid, const JobDev &d, const Refresh &g, CommitLds<R> &L, BlockBest *sup) {
    using S = Stage<R>;
    constexpr int NB = S::NBA * S::NBA;
    const int sub = tid & 15;
#pragma unroll
    for (int b0 = 0; b0 < NB; b0 += kCommitThreads >> 4) {
        const int b = b0 + (tid >> 4), bc = b % S::NBA, br = b / S::NBA;
        const bool live = b < NB && bc < g.nabx && br < g.naby;
        const int64_t *kp = &L.bkey[(8 * min(br, S::NBA - 1) + (sub >> 3)) * S::BP + 8 * bc + (sub & 7)];   // rows + 0, 2, 4, 6
        const uint32_t i0 = (uint32_t)((8 * (g.aby0 + br) + (sub >> 3)) * d.W + 8 * (g.abx0 + bc) + (sub & 7));
        Best best = {kp[0], i0};
#pragma unroll
        for (int j = 1; j < 4; ++j) {
            // (indices rise with j, so an equal key keeps the earlier one)
            const int64_t key = kp[2 * j * S::BP];
            best.idx = key > best.key ? i0 + (uint32_t)(2 * j * d.W) : best.idx;
            best.key = key > best.key ? key : best.key;
        }
        // the block's 16 threads are one DPP row: lane 15 ends with the maximum
        const uint64_t e = (uint64_t)(best.key + 1);
        const auto row_max = [](uint32_t v) {
            v = dpp::fold_rows(v, [](uint32_t a, uint32_t c) { return c > a ? c : a; });
            return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x15f, 0xf, 0xf, true);   // lane 15 of the row
        };
        const uint32_t hi = (uint32_t)(e >> 32), lo = (uint32_t)e;
        const uint32_t mh = row_max(hi), ml = row_max(hi == mh ? lo : 0u);
        const uint32_t mi = row_max(hi == mh && lo == ml ? ~best.idx : 0u);
        if (live && sub == 15) {
            const int64_t key = (int64_t)((uint64_t)mh << 32 | ml) - 1;
            const uint32_t idx = ~mi;
            d.blk[(g.aby0 + br) * d.nbw + g.abx0 + bc] = BlockBest{key, key < 0 ? INT64_MAX : (int64_t)idx};
            L.bmk[b] = key;
            L.bmi[b] = idx;
        }
    }
    lds_barrier();
    const int wave = tid >> 6, lane = tid & 63;
    const int sx = g.sx0 + (wave & 1), sy = g.sy0 + (wave >> 1);
    if (sx > g.sx1 || sy > g.sy1) return;   // (uniform over the wave)
    Best b = no_best();
    if (lane < NB) {
        const int bc = lane % S::NBA, br = lane / S::NBA;
        if (bc < g.nabx && br < g.naby && ((g.abx0 + bc - d.pbx0) >> d.sshift) == sx &&
            ((g.aby0 + br - d.pby0) >> d.sshift) == sy)
            b = {L.bmk[lane], L.bmi[lane]};
    } else if (lane == 63) {
        b = L.part[wave];
    }
    static_assert(NB <= 63, "one touched block per lane, the last lane holds the rest");
    b = wave_best(b);
    if (lane == 0) {
        const BlockBest v = {b.key, b.key < 0 ? INT64_MAX : (int64_t)b.idx};
        d.sup[sy * d.nsx + sx] = v;
        if (sup) sup[sy * d.nsx + sx] = v;
    }
}

// The patch at raster index idx, column-major slots tid + 256 j, as words with
// the state in byte 3 (out-of-image slots kStateOut): load it while other
// work goes on.
struct PatchWords {
    uint32_t w[kSlots];
};
template <int R>
__device__ __forceinline__ PatchWords load_patch(int tid, const JobDev &d, int tx, int ty) {
    constexpr int P = 2 * R + 1;
    PatchWords f{};
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
        if (j * kCommitThreads >= P * P) continue;
        const int t = min(tid + j * kCommitThreads, P * P - 1);
        const int x = tx + t / P - R, y = ty + t % P - R;
        const uint32_t w = d.img[(uint32_t)(min(max(y, 0), d.H - 1) * d.W + min(max(x, 0), d.W - 1))];
        f.w[j] = in_img(d, x, y) ? w : kStateOut;
    }
    return f;
}

}  // namespace inpaint
