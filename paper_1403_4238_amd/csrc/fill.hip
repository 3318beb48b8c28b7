// Initialisation, selection, target staging, and the kernels around a fill
// iteration of exemplar-based object removal on gfx950: the stream-form commit
// (one work-group of 256 threads per image, after each search) and the
// persistent forms, whose committer runs the same steps (commit.h) while the
// search groups score.
//
// Priorities are binary64 and must match a plain sequential CPU evaluation
// bit for bit, so this file is compiled with FP contraction off and every
// sum runs in the fixed raster order of the patch offsets.
#pragma clang fp contract(off)

#include <algorithm>

#include "commit.h"
#include "search_mfma_tile.h"

// This file is compiled once per part so that the parts build in parallel:
// 0 holds the initialisation, commit, query and persistent SIMT kernels and
// every launcher, 1 to 3 one family of persistent MFMA kernels each.
#ifndef INPAINT_FILL_PART
#error "INPAINT_FILL_PART (0 .. 3) selects what this compilation holds"
#endif

namespace inpaint {

namespace {

// ---- pixel views: what a priority evaluation reads -------------------------

// Column and row of a raster index (0 <= i < W * H < 2^31, so a 32-bit
// unsigned division, much shorter than a 64-bit one).
__device__ __forceinline__ int col_of(int64_t i, int W) { return (int)((uint32_t)i % (uint32_t)W); }
__device__ __forceinline__ int row_of(int64_t i, int W) { return (int)((uint32_t)i / (uint32_t)W); }

// Straight from global memory.
struct GlobalView {
    const JobDev &d;
    __device__ bool known(int x, int y) const { return in_img(d, x, y) && d.hole[(int64_t)y * d.W + x] == 0; }
    // hole indicator with out-of-image pixels counted as hole (the normal)
    __device__ int hole_or_out(int x, int y) const {
        return (!in_img(d, x, y) || d.hole[(int64_t)y * d.W + x]) ? 1 : 0;
    }
    // Central-difference gradient of the gray image at a known pixel whose
    // four neighbours are known: returns gx^2 + gy^2, or -1 otherwise.
    __device__ int grad(int x, int y, int *gx, int *gy) const {
        if (!known(x, y) || !known(x + 1, y) || !known(x - 1, y) || !known(x, y + 1) || !known(x, y - 1))
            return -1;
        const uint8_t *p = d.gray + (int64_t)y * d.W + x;
        *gx = (int)p[1] - (int)p[-1];
        *gy = (int)p[d.W] - (int)p[-d.W];
        return *gx * *gx + *gy * *gy;
    }
};

// Fill front: a hole pixel with at least one in-image 4-neighbour known.
// (x, y) is always inside the image here.
__device__ __forceinline__ bool on_front(const GlobalView &v, int x, int y) {
    if (v.hole_or_out(x, y) == 0) return false;
    return v.known(x + 1, y) || v.known(x - 1, y) || v.known(x, y + 1) || v.known(x, y - 1);
}

// Scratch of a target staging.
struct Scratch {
    uint32_t t2[4];
    uint32_t mbits[16];
};

// The words of the persistent form's records carry their own freshness: each
// is the target word (RGB) with a 7-bit tag of the fill iteration it belongs
// to in bits 24-30 and its known flag in bit 31.  Consecutive iterations of
// a job have different tags, and every word of a record is rewritten each
// iteration, so a word that carries the expected tag is that iteration's.
__device__ __forceinline__ uint32_t rec_tag(int64_t iter) { return (uint32_t)(iter % 127) + 1u; }
__device__ __forceinline__ uint32_t lean_word(uint32_t pix, bool known, uint32_t tag) {
    return (pix & kColour) | (tag << 24) | (known ? 0x80000000u : 0u);
}

// Column-run bits of mask word w (of mw) of a P x P patch in column-major
// slot order: a known slot starts a run when the slot above it in its column
// is unknown or outside the patch, and ends one when the slot below is.
__device__ __forceinline__ void run_bits(const uint32_t *mbits, int w, int mw, int P, uint32_t *sb, uint32_t *eb) {
    const uint32_t m = mbits[w];
    const uint32_t up = (m << 1) | (w > 0 ? mbits[w - 1] >> 31 : 0u);        // slot - 1 known
    const uint32_t dn = (m >> 1) | (w + 1 < mw ? mbits[w + 1] << 31 : 0u);   // slot + 1 known
    uint32_t cs = 0, ce = 0;   // slots at the top / bottom of their column
    const int base = 32 * w;
    for (int c = (base + P - 1) / P * P; c < base + 32; c += P) cs |= 1u << (c - base);
    for (int c = (base + P) / P * P - 1; c < base + 32; c += P) ce |= 1u << (c - base);
    *sb = m & (cs | ~up);
    *eb = m & (ce | ~dn);
}

// Target staging core: slot(t, round, &pix) says whether patch slot t (column-major,
// (dx + r) * P + (dy + r)) is known and gives its RGB word.  One pass over
// the slots writes the words and takes the known mask with a wave ballot per
// 64 slots (no atomics), then one barrier; the column-run bits follow from
// the mask words: a known slot starts a run when the slot above it in its
// column is unknown or outside the patch, and ends one when the slot below
// is.  Returns the known count k; T2 = sum of squared known values.
template <class F>
__device__ void stage_slots(int r, int tx, int ty, TargetStage *tg, Scratch &s, F slot) {
    const int P = 2 * r + 1, n = P * P, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t t2 = 0;
    for (int j = 0; j * kCommitThreads < n; ++j) {
        const int t = j * kCommitThreads + threadIdx.x;
        uint32_t pix = 0;
        const bool kn = t < n && slot(t, j, &pix);
        if (t < n) tg->tpix[t] = pix;
        if (kn) {
            const uint32_t R = pix & 255, G = (pix >> 8) & 255, B = (pix >> 16) & 255;
            t2 += R * R + G * G + B * B;
        }
        const uint64_t bal = __ballot(kn);
        const int w0 = (j * kCommitThreads >> 5) + 2 * wave;
        if (lane == 0 && w0 < 16) {
            s.mbits[w0] = (uint32_t)bal;
            if (w0 + 1 < 16) s.mbits[w0 + 1] = (uint32_t)(bal >> 32);
        }
    }
    t2 = dpp::sum_u32(t2);
    if (lane == 0) s.t2[wave] = t2;
    lds_barrier();
    const int mw = (n + 31) / 32;
    if ((int)threadIdx.x < mw) {
        const int w = threadIdx.x;
        uint32_t sb, eb;
        run_bits(s.mbits, w, mw, P, &sb, &eb);
        tg->mbits[w] = s.mbits[w];
        tg->sbits[w] = sb;
        tg->ebits[w] = eb;
    }
    if (threadIdx.x == 0) {
        int kk = 0;
        for (int w = 0; w < mw; ++w) kk += __popc(s.mbits[w]);
        tg->tx = tx;
        tg->ty = ty;
        tg->r = r;
        tg->k = kk;
        tg->t2 = s.t2[0] + s.t2[1] + s.t2[2] + s.t2[3];
    }
}

// Stages the target patch at (tx, ty) with radius r into *tg: known mask,
// RGBX words and T2 = sum of squared known target values, in column-major
// slot order (dx + r) * P + (dy + r).
__device__ void stage_target(const JobDev &d, int tx, int ty, int r, TargetStage *tg, Scratch &s) {
    const int P = 2 * r + 1;
    const GlobalView v{d};
    stage_slots(r, tx, ty, tg, s, [&](int t, int, uint32_t *pix) {
        const int x = tx + t / P - r, y = ty + t % P - r;
        if (!v.known(x, y)) return false;
        *pix = d.img[(int64_t)y * d.W + x] & kColour;
        return true;
    });
}

// Argmax over the superblocks, then stages the winner as the next target.
__device__ void select_and_stage(const JobDev &d, Scratch &s, int64_t *fk, uint32_t *fi) {
    Best b = no_best();
    for (int t = threadIdx.x; t < super_count(d); t += kCommitThreads) take(b, d.sup[t].key, (uint32_t)d.sup[t].idx);
    b = wave_best(b);
    if ((threadIdx.x & 63) == 0) {
        fk[threadIdx.x >> 6] = b.key;
        fi[threadIdx.x >> 6] = b.idx;
    }
    lds_barrier();
    for (int q = 0; q < 4; ++q) take(b, fk[q], fi[q]);
    IterState *st = d.st;
    if (b.key < 0) {
        // No front pixel although the hole is not empty: cannot happen for a
        // valid state; flag it instead of looping.
        if (threadIdx.x == 0) st->error = INPAINT_DEVICE;
        return;
    }
    stage_target(d, col_of(b.idx, d.W), row_of(b.idx, d.W), d.r, d.tgt, s);
    if (threadIdx.x == 0) {
        const double2 cd = d.pcd[b.idx];
        st->p_idx = b.idx;
        st->C = cd.x;
        st->D = cd.y;
        st->Pr = cd.x * cd.y;
        st->pending = 1;
    }
}

}  // namespace

// ----------------------------------------------------------------- kernels

#if INPAINT_FILL_PART == 0
// Cleared results, the loop state of a fresh removal (nothing staged), and no
// go or slot word of an earlier use of the workspace.
__global__ __launch_bounds__(256) void k_init_info(JobDev d, int64_t remaining, int nslots, uint32_t nonce) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x), n = (int)(gridDim.x * blockDim.x);
    for (int t = i; t < nslots; t += n) d.fslot[t] = 0;
    for (int t = i; t < (int)(sizeof(FillSync) / 4); t += n) ((uint32_t *)d.sync)[t] = 0;
    for (int t = i; t < (int)(sizeof(IterState) / 4); t += n) ((uint32_t *)d.st)[t] = 0;
    __syncthreads();
    if (i == 0) {   // (block 0 cleared the state: it has more threads than that has words)
        static_assert(sizeof(IterState) / 4 <= 256, "one block clears the state");
        d.st->remaining = remaining;
        d.st->iter_limit = INT64_MAX;
        InitInfo *info = d.info;
        info->hole_count = 0;
        info->bad = 0;
        info->bx0 = INT32_MAX;
        info->by0 = INT32_MAX;
        info->bx1 = INT32_MIN;
        info->by1 = INT32_MIN;
        info->valid_count = 0;
        info->nonce = nonce;
        info->seal = 0;
        info->blocks = 0;
    }
}

__global__ void k_seal(InitInfo *info, uint32_t nonce) { info->seal = nonce; }

// Initialisation: zero the hole pixels, RGBX image with the pixel state, integer
// BT.601 gray, hole map, confidence 1 / 0, hole count and bounding box.  Four
// pixels per thread and round, at most kInitBlocks work-groups: one thread per
// pixel moved single bytes and counted 8100 work-groups at one address (1080p:
// 144 us, now 41).
constexpr unsigned kInitBlocks = 512;
__device__ __forceinline__ void unpack_rgb(const uint8_t *rgb, int ch, int64_t i, bool whole, int left, uint32_t *w) {
    if (whole && ch == 4) {
        const uint4 v = *(const uint4 *)(rgb + 4 * i);
        w[0] = v.x & kColour, w[1] = v.y & kColour, w[2] = v.z & kColour, w[3] = v.w & kColour;
    } else if (whole) {
        const uint32_t *p = (const uint32_t *)(rgb + 3 * i);
        const uint32_t a = p[0], b = p[1], c = p[2];
        w[0] = a & kColour;
        w[1] = a >> 24 | (b & 0xffffu) << 8;
        w[2] = b >> 16 | (c & 0xffu) << 16;
        w[3] = c >> 8;
    } else {
        for (int j = 0; j < 4; ++j) {
            const uint8_t *p = rgb + (i + min(j, left - 1)) * ch;
            w[j] = p[0] | (uint32_t)p[1] << 8 | (uint32_t)p[2] << 16;
        }
    }
}

__global__ __launch_bounds__(256) void k_init_pixels(JobDev d, const uint8_t *rgb, int ch, const uint8_t *mask) {
    const int64_t n = (int64_t)d.W * d.H;
    __shared__ int s_cnt, s_x0, s_y0, s_x1, s_y1;
    if (threadIdx.x == 0) {
        s_cnt = 0;
        s_x0 = INT32_MAX;
        s_y0 = INT32_MAX;
        s_x1 = INT32_MIN;
        s_y1 = INT32_MIN;
    }
    __syncthreads();
    int cnt = 0, x0 = INT32_MAX, y0 = INT32_MAX, x1 = INT32_MIN, y1 = INT32_MIN;
    for (int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x); i < n; i += 4 * 256 * (int64_t)gridDim.x) {
        const int left = (int)min(n - i, (int64_t)4);
        const bool whole = left == 4;
        uint32_t w[4], m = 0;
        unpack_rgb(rgb, ch, i, whole, left, w);
        if (whole) m = *(const uint32_t *)(mask + i);
        else
            for (int j = 0; j < left; ++j) m |= (uint32_t)mask[i + j] << (8 * j);
        uint32_t g = 0, hole = 0;
        double c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool h = ((m >> (8 * j)) & 255u) != 0;
            g |= h ? 0u : (uint32_t)gray_of(w[j]) << (8 * j);
            hole |= h ? 1u << (8 * j) : 0u;
            w[j] = h ? kStateHole : w[j];
            c[j] = h ? 0.0 : 1.0;
        }
        if (whole) {
            *(uint4 *)(d.img + i) = make_uint4(w[0], w[1], w[2], w[3]);
            *(uint32_t *)(d.gray + i) = g;
            *(uint32_t *)(d.hole + i) = hole;
            *(uint32_t *)(d.hole0 + i) = hole;
            *(double2 *)(d.conf + i) = make_double2(c[0], c[1]);
            *(double2 *)(d.conf + i + 2) = make_double2(c[2], c[3]);
        } else {
            for (int j = 0; j < left; ++j) {
                d.img[i + j] = w[j];
                d.gray[i + j] = (uint8_t)(g >> (8 * j));
                d.hole[i + j] = d.hole0[i + j] = (uint8_t)(hole >> (8 * j));
                d.conf[i + j] = c[j];
            }
        }
        if (hole) {
            int x = col_of(i, d.W), y = row_of(i, d.W);
            for (int j = 0; j < left; ++j) {
                if ((hole >> (8 * j)) & 1u) {
                    ++cnt;
                    x0 = min(x0, x), x1 = max(x1, x + 1), y0 = min(y0, y), y1 = max(y1, y + 1);
                }
                if (++x == d.W) x = 0, ++y;
            }
        }
    }
    if (cnt) {
        atomicAdd(&s_cnt, cnt);
        atomicMin(&s_x0, x0);
        atomicMin(&s_y0, y0);
        atomicMax(&s_x1, x1);
        atomicMax(&s_y1, y1);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt > 0) {
        atomicAdd((unsigned long long *)&d.info->hole_count, (unsigned long long)s_cnt);
        atomicMin(&d.info->bx0, s_x0);
        atomicMin(&d.info->by0, s_y0);
        atomicMax(&d.info->bx1, s_x1);
        atomicMax(&d.info->by1, s_y1);
    }
    if (threadIdx.x == 0) atomicAdd(&d.info->blocks, 1u);
}

// The colours of `count` pixels, packed, 4 pixels per thread.
__global__ __launch_bounds__(256) void k_pack_rgb(const uint32_t *img, int64_t count, uint8_t *out) {
    const int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
    if (i >= count) return;
    if (i + 4 <= count) {
        const uint4 v = *(const uint4 *)(img + i);
        uint32_t *o = (uint32_t *)(out + 3 * i);
        o[0] = (v.x & kColour) | v.y << 24;
        o[1] = ((v.y >> 8) & 0xffffu) | v.z << 16;
        o[2] = ((v.z >> 16) & 0xffu) | v.w << 8;
    } else {
        for (int64_t j = i; j < count; ++j)
            for (int c = 0; c < 3; ++c) out[3 * j + c] = (uint8_t)(img[j] >> (8 * c));
    }
}

// ---- checkpoint import (resume / iterative editing) ------------------------

// Counts the pixels of a checkpoint that fail its checks: a hole pixel
// outside the original hole, or a filled pixel of the original hole whose
// confidence is not in [0, 1] (NaN included).  Writes nothing else.
__global__ __launch_bounds__(256) void k_import_check(JobDev d, const uint8_t *hole, const double *conf) {
    const int64_t n = (int64_t)d.W * d.H;
    int bad = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += 256 * (int64_t)gridDim.x) {
        const bool h = hole[i] != 0, h0 = d.hole0[i] != 0;
        const double c = conf[i];
        bad += (h && !h0) || (h0 && !h && !(c >= 0.0 && c <= 1.0));
    }
    if (bad) atomicAdd((unsigned long long *)&d.info->bad, (unsigned long long)bad);
    if (threadIdx.x == 0) atomicAdd(&d.info->blocks, 1u);
}

// Overlays a checked checkpoint on the original-hole pixels: those still in
// its hole become hole again (zeroed), the others take its colour, the gray
// value of that colour and its confidence.  Other pixels keep their values.
__global__ __launch_bounds__(256) void k_import_apply(JobDev d, const uint8_t *rgb, int ch, const uint8_t *hole,
                                                      const double *conf) {
    const int64_t n = (int64_t)d.W * d.H;
    __shared__ int s_cnt;
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    int cnt = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += 256 * (int64_t)gridDim.x) {
        if (!d.hole0[i]) continue;
        const bool h = hole[i] != 0;
        const uint32_t R = h ? 0 : rgb[i * ch], G = h ? 0 : rgb[i * ch + 1], B = h ? 0 : rgb[i * ch + 2];
        d.img[i] = R | (G << 8) | (B << 16) | (h ? kStateHole : 0u);
        d.gray[i] = (uint8_t)gray_of(R | (G << 8) | (B << 16));
        d.hole[i] = h ? 1 : 0;
        d.conf[i] = h ? 0.0 : conf[i];
        cnt += h;
    }
    if (cnt) atomicAdd(&s_cnt, cnt);
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt > 0) atomicAdd((unsigned long long *)&d.info->hole_count, (unsigned long long)s_cnt);
    if (threadIdx.x == 0) atomicAdd(&d.info->blocks, 1u);
}

__global__ void k_import_reset(InitInfo *info, uint32_t nonce) {
    info->hole_count = 0;
    info->bad = 0;
    info->nonce = nonce;
    info->seal = 0;
    info->blocks = 0;
}

// Validity radii and the padded search planes, one 64 x 16 tile of the padded
// plane per work-group.
//
// vrad = (Chebyshev distance to the nearest hole or out-of-image pixel) - 1,
// clamped to [0, 8]: the patch of radius r at a centre lies inside the image
// and the original known region iff vrad >= r.  A row's holes are two wave
// ballots (64 columns and 9 on either side), from which each lane takes the
// distance to the nearest along the row (capped at 10) with a shift and two
// bit scans; the rows combine through LDS.  The padded planes hold the
// original image (hole pixels zero) and vrad, zero outside the image; with
// INTERSECT scoring the 4th byte of a source pixel's word is 1 and the
// validity plane only flags source pixels (a candidate centre needs to be
// one).  hdist (or null) keeps the row distances.  In place of three kernels
// that read the holes byte by byte (1080p: 52 us together, now 18).
__global__ __launch_bounds__(256) void k_init_planes(JobDev d, uint8_t *hdist) {
    constexpr int TH = 16, RD = 9;
    __shared__ uint8_t hd[TH + 2 * RD][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // (a grid of one dimension: images that are accepted have more rows of tiles
    // than the 65535 that the second one is documented to take)
    const int nx = (d.pitch + 63) / 64;
    const int x0 = (int)(blockIdx.x % nx) * 64 - kPadL, y0 = (int)(blockIdx.x / nx) * TH - kPadT, x = x0 + lane;
    const auto bad = [&](int px, int py) { return !in_img(d, px, py) || d.hole[(int64_t)py * d.W + px] != 0; };
    for (int r = wave; r < TH + 2 * RD; r += 4) {
        const int y = y0 - RD + r;
        const uint64_t b0 = __ballot(bad(x - RD, y)), b1 = __ballot(lane < 2 * RD && bad(x - RD + 64, y));
        // bits 0 .. 18: columns x - 9 .. x + 9
        const uint32_t w = (uint32_t)((b0 >> lane) | (lane ? b1 << (64 - lane) : 0ull)) & 0x7ffffu;
        const uint32_t right = w >> RD, leftw = w & 0x3ffu;
        const int dr = right ? __builtin_ctz(right) : 10, dl = leftw ? __builtin_clz(leftw) - 22 : 10;
        const uint8_t h = (uint8_t)min(dr, dl);
        hd[r][lane] = h;
        if (hdist && r >= RD && r < TH + RD && in_img(d, x, y)) hdist[(int64_t)y * d.W + x] = h;
    }
    __syncthreads();
    if (x + kPadL >= d.pitch) return;
    for (int q = 0; q < TH / 4; ++q) {
        const int r = wave * (TH / 4) + q, y = y0 + r;
        if (y + kPadT >= padded_rows(d.H)) return;
        int dist = 10;
#pragma unroll
        for (int dy = -RD; dy <= RD; ++dy) dist = min(dist, max(dy < 0 ? -dy : dy, (int)hd[r + RD + dy][lane]));
        uint32_t pix = 0;
        uint8_t vr = 0;
        if (in_img(d, x, y)) {
            const int64_t i = (int64_t)y * d.W + x;
            vr = (uint8_t)min(max(dist - 1, 0), kMaxRadius);
            d.vrad[i] = vr;
            const uint32_t w = d.img[i];
            pix = w & kColour;
            if (d.isect) {
                vr = state_of(w) == 0 ? 1 : 0;
                pix |= (uint32_t)vr << 24;
            }
        }
        const int64_t o = (int64_t)(y + kPadT) * d.pitch + (x + kPadL);
        d.srcp[o] = pix;
        d.vradp[o] = vr;
    }
}

// Number of valid source centres in the search rectangle, a row per work-group
// and round (1080p: 12 us; a shared-memory atomic per centre took 97).
__global__ __launch_bounds__(256) void k_count_valid(JobDev d) {
    __shared__ int s_cnt[4];
    int cnt = 0;
    for (int y = d.ry0 + (int)blockIdx.x; y < d.ry1; y += (int)gridDim.x)
        for (int x = d.rx0 + (int)threadIdx.x; x < d.rx1; x += 256) {
            const int64_t j = (int64_t)y * d.W + x;
            cnt += d.isect ? d.hole[j] == 0 : d.vrad[j] >= d.r;
        }
    cnt = (int)dpp::sum_u32((uint32_t)cnt);
    if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = cnt;
    __syncthreads();
    cnt = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
    if (threadIdx.x == 0 && cnt) atomicAdd((unsigned long long *)&d.info->valid_count, (unsigned long long)cnt);
}
#endif  // INPAINT_FILL_PART 0

// Gradients, priority terms (Eq. 2) and block maxima of every block of the
// priority range; one wave per 8x8 block.  Only blocks with a front pixel need
// more than a pixel's own gradient: such a wave stages the block with R + 1
// pixels around it in LDS and evaluates its front pixels there, one per lane,
// as confidence_terms and data_terms do.  1080p: 12 us at 9x9, 20 at 17x17.
// (Reading each offset of each patch from global memory took 46 and 139.)
template <int R>
__global__ __launch_bounds__(256) void k_prio_init(JobDev d) {
    constexpr int P = 2 * R + 1, H = R + 1, S = kBlock + 2 * H;
    __shared__ double s_conf[4][S * S];
    __shared__ uint32_t s_img[4][S * S], s_grad[4][S * S];
    const int bw = d.pbx1 - d.pbx0, nb = bw * (d.pby1 - d.pby0);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, b = (int)blockIdx.x * 4 + wave;
    if (b >= nb) return;
    const int bx = d.pbx0 + b % bw, by = d.pby0 + b / bw;
    const int x = bx * kBlock + (lane & (kBlock - 1)), y = by * kBlock + lane / kBlock;
    const GlobalView v{d};
    const bool in = in_img(d, x, y), front = in && on_front(v, x, y);
    double2 cd = off_front(0);
    if (__ballot(front) == 0) {
        int gx = 0, gy = 0;
        if (in && v.grad(x, y, &gx, &gy) >= 0) cd = off_front(pack_grad(gx, gy));
    } else {
        double *conf = s_conf[wave];
        uint32_t *img = s_img[wave], *grad = s_grad[wave];
        for (int t = lane; t < S * S; t += 64) {
            const int px = bx * kBlock - H + t % S, py = by * kBlock - H + t / S;
            const uint32_t w = in_img(d, px, py) ? d.img[(int64_t)py * d.W + px] : kStateOut;
            img[t] = w;
            conf[t] = state_of(w) == 0 ? d.conf[(int64_t)py * d.W + px] : 0.0;
        }
        // (one wave: its LDS accesses are in order, the fence keeps the compiler's)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int t = lane; t < (S - 2) * (S - 2); t += 64) {
            const int li = (t / (S - 2) + 1) * S + t % (S - 2) + 1;
            const uint32_t any = (img[li] | img[li + 1] | img[li - 1] | img[li + S] | img[li - S]) >> 24;
            grad[li] = any == 0 ? pack_grad(gray_of(img[li + 1]) - gray_of(img[li - 1]),
                                            gray_of(img[li + S]) - gray_of(img[li - S]))
                                : 0u;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int li = (lane / kBlock + H) * S + (lane & (kBlock - 1)) + H;
        if (!front) {
            cd = off_front(grad[li]);   // 0 for hole pixels
        } else {
            double sum = 0.0;
            uint32_t best = 0;
#pragma unroll 1
            for (int dy = 0; dy < P; ++dy) {
                const int row = li + (dy - R) * S - R;
#pragma unroll
                for (int dx = 0; dx < P; ++dx) {
                    sum = sum + conf[row + dx];
                    best = max(best, (uint32_t)grad_size(grad[row + dx]) << 9 | (uint32_t)(511 - dy * P - dx));
                }
            }
            const int at = 511 - (int)(best & 511);
            const int nx = (state_of(img[li + 1]) != 0) - (state_of(img[li - 1]) != 0);
            const int ny = (state_of(img[li + S]) != 0) - (state_of(img[li - S]) != 0);
            cd.x = sum / (double)(P * P);
            cd.y = data_term(grad[li + (at / P - R) * S + at % P - R], nx, ny, d.norm1, d.norm2);
        }
    }
    Best m = no_best();
    if (in) {
        d.pcd[(int64_t)y * d.W + x] = cd;
        m = {key_of(cd), (uint32_t)(y * d.W + x)};
    }
    m = wave_best(m);
    if (lane == 0) d.blk[by * d.nbw + bx] = BlockBest{m.key, m.key < 0 ? INT64_MAX : (int64_t)m.idx};
}

#if INPAINT_FILL_PART == 0
// Superblock maxima from the block maxima, one wave per superblock.
__global__ __launch_bounds__(256) void k_super_init(JobDev d) {
    const int e = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (e >= super_count(d)) return;
    const int bx0 = d.pbx0 + ((e % d.nsx) << d.sshift), by0 = d.pby0 + ((e / d.nsx) << d.sshift), n = 1 << d.sshift;
    Best b = no_best();
    for (int t = threadIdx.x & 63; t < n * n; t += 64) {
        const int bx = bx0 + (t & (n - 1)), by = by0 + (t >> d.sshift);
        if (bx >= d.pbx1 || by >= d.pby1) continue;
        const BlockBest v = d.blk[by * d.nbw + bx];
        take(b, v.key, (uint32_t)v.idx);
    }
    b = wave_best(b);
    if ((threadIdx.x & 63) == 0) d.sup[e] = BlockBest{b.key, b.key < 0 ? INT64_MAX : (int64_t)b.idx};
}
#endif  // INPAINT_FILL_PART 0

// What the stream-form commit reports about its copy: the target and the
// number of pixels filled.
struct CommitNote {
    uint32_t p;
    int32_t filled;
};

// CURRENT source policy: the pixels this iteration filled become source
// pixels.  Writes their words into the padded source plane and brings the
// validity plane up to date around the patch: the horizontal distances of the
// patch rows, then the validity radii of every centre whose radius can have
// changed (as k_init_planes computes them).  The hole map changed only inside
// the patch, which the LDS neighbourhood holds; every other pixel is read from
// device memory, unchanged since earlier launches.
template <int R, bool ISECT>
__device__ void add_filled_sources(const JobDev &d, const CommitLds<R> &L, int px, int py) {
    constexpr int P = 2 * R + 1, half = Stage<R>::half, side = Stage<R>::side, pitch_l = Stage<R>::pitch;
    constexpr int HW = 2 * R + 19;   // columns px - R - 9 .. px + R + 9
    const int W = d.W, H = d.H, pitch = d.pitch;
    auto known = [&](int x, int y) -> bool {
        if ((unsigned)x >= (unsigned)W || (unsigned)y >= (unsigned)H) return false;
        const int lx = x - px + half, ly = y - py + half;
        if ((unsigned)lx < (unsigned)side && (unsigned)ly < (unsigned)side) return state_of(L.img[ly * pitch_l + lx]) == 0;
        return d.hole[(int64_t)y * W + x] == 0;
    };
    // the patch's known pixels (rewriting the unchanged ones is harmless)
    for (int t = threadIdx.x; t < P * P; t += blockDim.x) {
        const int x = px + t % P - R, y = py + t / P - R;
        if (!known(x, y)) continue;
        const int64_t pi = (int64_t)(y + kPadT) * pitch + (x + kPadL);
        d.srcp[pi] = L.img[(y - py + half) * pitch_l + (x - px + half)] | (ISECT ? 1u << 24 : 0u);
        if (ISECT) d.vradp[pi] = 1;
    }
    if (ISECT) return;   // INTERSECT candidates only need their centre to be a source pixel
    __shared__ uint8_t hrow[P * HW];
    for (int t = threadIdx.x; t < P * HW; t += blockDim.x) {
        const int x = px - R - 9 + t % HW, y = py - R + t / HW;
        uint8_t h = 0;
        if ((unsigned)x < (unsigned)W && (unsigned)y < (unsigned)H) {
            int hh = 10;
            for (int dx = 0; dx < 10; ++dx)
                if (!known(x - dx, y) || !known(x + dx, y)) {
                    hh = dx;
                    break;
                }
            h = (uint8_t)hh;
            d.hdist[(int64_t)y * W + x] = h;
        }
        hrow[t] = h;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < HW * HW; t += blockDim.x) {
        const int x = px - R - 9 + t % HW, y = py - R - 9 + t / HW;
        if ((unsigned)x >= (unsigned)W || (unsigned)y >= (unsigned)H) continue;
        int dist = 10;
        for (int dy = -9; dy <= 9; ++dy) {
            const int yy = y + dy, ady = dy < 0 ? -dy : dy;
            int h;
            if (yy < 0 || yy >= H) h = 0;
            else if (yy >= py - R && yy <= py + R) h = hrow[(yy - py + R) * HW + (x - px + R + 9)];
            else h = d.hdist[(int64_t)yy * W + x];
            const int m = ady > h ? ady : h;
            dist = m < dist ? m : dist;
        }
        int v = dist - 1;
        v = v < 0 ? 0 : (v > kMaxRadius ? kMaxRadius : v);
        d.vradp[(int64_t)(y + kPadT) * pitch + (x + kPadL)] = (uint8_t)v;
    }
}

// One fill iteration after the search: reduce the search partials, fill the
// target patch, refresh the priorities near it, select and stage the next
// target.  With no staged target (right after create) it only selects and
// stages.
template <int R, bool ISECT = false>
__device__ __forceinline__ void commit_body(const JobDev &d, Scratch &s, CommitLds<R> &L, CommitNote *note) {
    using S = Stage<R>;
    constexpr int P = S::P, T = kCommitThreads;
    Snap v = load_snap(d.st);
    if (v.done || v.err) return;
    if (!v.pending) {
        select_and_stage(d, s, L.fk[0], L.fi[0]);
        return;
    }
    if (v.iter >= v.limit) return;
    const Raster raster(d.W);
    int px, py;
    raster.split(v.p, &px, &py);
    const Refresh g = refresh_geometry<R>(d, px, py);
    const int known_k = d.tgt->k, tid = threadIdx.x;

    // the search partials, eight loads in flight, with the gather's
    const int ntiles = d.ntx * d.nty;
    uint64_t pv[8], best = ~0ull;
#pragma unroll
    for (int k = 0; k < 8; ++k) pv[k] = d.partials[min((int)threadIdx.x + k * T, ntiles - 1)];
    post_best(L, gather<R>(tid, d, px, py, g, d.sup, L));
#pragma unroll
    for (int k = 0; k < 8; ++k) best = pv[k] < best ? pv[k] : best;   // clamped repeats are harmless
    // (many tiles: eight in flight again; the 11750 SIMT tiles of a 24 Mpixel
    // image at radius 1, us an iteration: 49.2 one by one, 42.1 now)
    for (int t0 = threadIdx.x + 8 * T; t0 < ntiles; t0 += 8 * T) {
#pragma unroll
        for (int k = 0; k < 8; ++k) pv[k] = d.partials[min(t0 + k * T, ntiles - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k) best = pv[k] < best ? pv[k] : best;
    }
    best = wave_min(best);
    if ((threadIdx.x & 63) == 0) L.smin[threadIdx.x >> 6] = best;
    lds_barrier();
#pragma unroll
    for (int q = 0; q < 4; ++q) best = L.smin[q] < best ? L.smin[q] : best;
    IterState *st = d.st;
    if (best == ~0ull) {
        if (threadIdx.x == 0) st->error = INPAINT_NO_CANDIDATE;
        return;
    }
    // the best pixel that keeps its priority: the usual next target when that
    // is far; its patch and terms are loaded now
    const Best far = posted_best(L, 0);
    const uint32_t fidx = far.key >= 0 ? far.idx : v.p;
    int fx, fy;
    raster.split(fidx, &fx, &fy);
    const PatchWords fw = load_patch<R>(tid, d, fx, fy);
    const double2 fcd = d.pcd[fidx];

    const uint32_t q = (uint32_t)best;
    int qx, qy;
    raster.split(q, &qx, &qy);
    const FillSlots fs = mark_filled<R>(tid, d, px, py, v.C, g, L, [&](int t) {
        // INTERSECT: the flag byte of the source word, read before any of
        // this copy's writes (the padded plane covers R pixels around the image)
        return !ISECT || (d.srcp[(int64_t)(qy + t / P - R + kPadT) * d.pitch + (qx + t % P - R + kPadL)] >> 24) != 0;
    });
    stage_gray<R>(tid, L);
    if (!ISECT) list_front<R, true>(tid, L);
    lds_barrier();
    copy_colours<R>(tid, d, px, py, qx, qy, fs, L);
    const int filled = filled_count(L.cnt);
    if (ISECT) list_front<R, false>(tid, L);
    lds_barrier();
    refresh_grads<R>(tid, d, px, py, L);
    confidence_terms<R>(tid, L);
    const int64_t remaining = v.remaining - filled;
    if (threadIdx.x == 0) {
        if (note) {
            note->p = v.p;
            note->filled = filled;
        }
        StepRec rec;
        rec.target_index = v.p;
        rec.source_index = q;
        rec.ssd = (uint32_t)(best >> 32);
        rec.known_k = known_k;
        rec.n_filled = filled;
        rec.reserved = 0;
        rec.priority = v.Pr;
        rec.confidence = v.C;
        rec.data_term = v.D;
        rec.remaining = remaining;
        if (v.iter < d.log_cap) d.log[v.iter] = rec;
        st->last = rec;
        st->remaining = remaining;
        st->iter = v.iter + 1;
        st->pending = 0;
        if (remaining == 0) st->done = 1;
    }
    if (remaining == 0) return;
    lds_barrier();
    data_terms<R>(tid, d, px, py, g, L);
    lds_barrier();
    int wv;
    const Best near = posted_best(L, 1, &wv);
    const bool is_far = better(far.key, far.idx, near.key, near.idx);
    const Best next = is_far ? far : near;
    if (next.key < 0) {
        // No front pixel although the hole is not empty: cannot happen for a
        // valid state; flag it instead of looping.
        if (threadIdx.x == 0) st->error = INPAINT_DEVICE;
        return;
    }
    int tx, ty;
    raster.split(next.idx, &tx, &ty);
    stage_slots(R, tx, ty, d.tgt, s, [&](int t, int j, uint32_t *pix) {
        const uint32_t w = is_far ? (j == 0 ? fw.w[0] : fw.w[1]) : L.img[S::at(tx - px + t / P - R, ty - py + t % P - R)];
        if (state_of(w) != 0) return false;
        *pix = w;
        return true;
    });
    if (threadIdx.x == 0) {
        const double C = is_far ? fcd.x : L.wC[wv], D = is_far ? fcd.y : L.wD[wv];
        st->p_idx = next.idx;
        st->C = C;
        st->D = D;
        st->Pr = C * D;
        st->pending = 1;
    }
    update_blocks<R>(tid, d, g, L, nullptr);
}

// ---- persistent fill: one dispatch runs many iterations ------------------
//
// Work-group 0 commits; work-group 1 + t owns search tile t for the whole
// dispatch, staged in LDS once (its source pixels never change).  Per
// iteration k: the committer publishes go = (epoch, k + 1) once target k is
// staged; every search group copies the target to LDS, scores its tile and
// writes its minimum key, tagged with k, to its own slot; meanwhile the committer
// issues the search-independent loads of the commit (gather).  When every
// slot carries iteration k's tag it reduces the keys and finishes the
// iteration.  go carries the launch epoch, so values left by an earlier
// dispatch never match.  Every wait is bounded: a search group gives up
// after kSpinLimit polls; the committer then flags a device error and
// publishes stop, and every group exits.

constexpr uint32_t kSpinLimit = 1u << 22;

// Go words: the launch epoch in the high half; in the low half either stop
// (all ones) or k + 1 (k < 2^25 - 1, the dispatch's iteration) in bits 0-24
// with the record tag of that iteration in bits 25-31.
constexpr uint32_t kGoK = (1u << 25) - 1;
__device__ __forceinline__ uint64_t go_word(uint32_t epoch, uint32_t k1, uint32_t tag) {
    return ((uint64_t)epoch << 32) | (tag << 25) | k1;
}
__device__ __forceinline__ uint64_t go_stop(uint32_t epoch) { return ((uint64_t)epoch << 32) | 0xffffffffu; }
__device__ __forceinline__ bool go_is(uint64_t v, uint32_t epoch, uint32_t k1) {
    return (v >> 32) == epoch && (uint32_t)v != 0xffffffffu && (v & kGoK) == k1;
}
__device__ __forceinline__ uint32_t go_tag(uint64_t v) { return (uint32_t)(v >> 25) & 0x7fu; }

// Committer (all threads): writes every copy of the go word.
__device__ __forceinline__ void publish_go(FillSync *sy, uint64_t word) {
    if (threadIdx.x < kGoCopies)
        __hip_atomic_store(&sy->rec[threadIdx.x].go, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t slot_tag(uint32_t k) { return k % 255u + 1u; }

__device__ __forceinline__ uint64_t slot_word(uint64_t key, uint32_t tag) {
    if (key == ~0ull) return (~0ull << 8) | tag;
    const uint64_t ssd = key >> 32, idx = key & 0xffffffffu;
    return (ssd << (kSlotIndexBits + 8)) | (idx << 8) | tag;
}

// Committer (all threads): waits until every search slot carries `tag` and
// leaves each wave's minimum (ssd, index) word in L.smin and whether it timed
// out in L.late; the caller's barrier publishes them.  Each slot word is
// self-contained, so plain device-scope loads suffice (no acquire, no cache
// invalidation).
template <int R>
__device__ __forceinline__ void collect_slots(const uint64_t *fs, int ntiles, uint32_t tag, CommitLds<R> &L) {
    // The first wave sums confidences meanwhile.
    constexpr int T = kCommitThreads - 64, U = 4;
    uint64_t best = ~0ull;
    bool pend = false;
    // Each thread polls its own slots (no barrier per round), so the last
    // report is seen one load latency after it lands; U loads in flight cover
    // the resident tiles of a single image.
    for (uint32_t spin = 0; threadIdx.x >= 64 && spin < kSpinLimit; ++spin) {
        best = ~0ull;
        pend = false;
        for (int t = (int)threadIdx.x - 64; t < ntiles; t += U * T) {
            uint64_t w[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                w[u] = __hip_atomic_load(&fs[t + u * T < ntiles ? t + u * T : t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                pend |= (w[u] & 255u) != tag;
                best = (w[u] >> 8) < best ? (w[u] >> 8) : best;
            }
        }
        if (!pend) break;
        __builtin_amdgcn_s_sleep(1);
    }
    const bool late = __ballot(pend) != 0;
    best = wave_min(best);
    if ((threadIdx.x & 63) == 0) {
        L.smin[threadIdx.x >> 6] = best;
        L.late[threadIdx.x >> 6] = late;
    }
}

// A word of a StepRec, whose fields are wider.
typedef uint32_t __attribute__((may_alias)) RecordWord;

// LDS of the persistent committer: the commit's, the superblock maxima (the
// scan of the blocks that keep their priorities reads them every iteration)
// and the last record.
template <int R>
struct FillCommitLds {
    CommitLds<R> c;
    BlockBest sup[kMaxSuper];
    Scratch s;
    StepRec last;
};

// The committer of one job.  Per iteration: publish the staged target, bring
// the block maxima of the last refresh up to date, gather, mark the patch's
// hole pixels filled and sum the new front's confidences -- which pixels the
// copy fills and the confidence they take do not depend on the source patch
// under the original source region with whole-window scoring, the only domain
// this form runs -- all while the search goes on; then collect the slots,
// copy the colours, and choose and stage the next target.  The loop state
// stays in registers, the same in every thread.
template <int R>
__device__ __forceinline__ void fill_commit(const JobDev &d, int ntiles, int n_iters, uint32_t epoch, FillCommitLds<R> &C) {
    using S = Stage<R>;
    constexpr int P = S::P, T = kCommitThreads;
    CommitLds<R> &L = C.c;
    FillSync *sy = d.sync;
    int tid = threadIdx.x;
    Snap v = load_snap(d.st);
    if (!v.done && !v.err && !v.pending) v.err = INPAINT_DEVICE;   // (create and import stage a target)
    const Raster raster(d.W);
    for (int e = tid; e < super_count(d); e += T) C.sup[e] = d.sup[e];
    // the target that an earlier dispatch or kernel staged
    const auto write_word = [&](int t, uint32_t w, bool known, uint32_t tag) {
        const uint32_t word = lean_word(w, known, tag);
        L.tword[t] = known ? (w & kColour) | 0x80000000u : 0u;
#pragma unroll
        for (int c = 0; c < kGoCopies; ++c)
            __hip_atomic_store(&sy->rec[c].tpix[t], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    for (int t = tid; t < P * P; t += T)
        write_word(t, d.tgt->tpix[t], (d.tgt->mbits[t >> 5] >> (t & 31)) & 1u, rec_tag(v.iter));
    for (int i = tid; i < ntiles; i += T)
        __hip_atomic_store(&d.fslot[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // (complete before the first go: a search group's report must not be
    // overtaken by the reset of its slot)
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    bool ran = false;
    bool logged = false, stale = false;   // the log and the block maxima lag the last iteration
    Refresh g{};
    for (uint32_t k = 0;; ++k) {
        tid = thread_number();
        // The words of a record say themselves which iteration they belong
        // to, so go needs no order after them.
        const bool stop = v.done || v.err || !v.pending || v.iter >= v.limit || (int)k >= n_iters;
        if (k == 0) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");   // the slot resets
        publish_go(sy, stop ? go_stop(epoch) : go_word(epoch, k + 1, rec_tag(v.iter)));
        if (logged && tid >= T - 64 && tid < T - 64 + (int)sizeof(StepRec) / 4 && v.iter <= d.log_cap)
            ((RecordWord *)&d.log[v.iter - 1])[tid - (T - 64)] = ((const RecordWord *)&C.last)[tid - (T - 64)];
        logged = false;
        if (stale) update_blocks<R>(tid, d, g, L, C.sup);
        stale = false;
        // every store of the last iteration is visible to the loads below
        __syncthreads();
        if (stop) break;

        int px, py;
        raster.split(v.p, &px, &py);
        px = __builtin_amdgcn_readfirstlane(px);
        py = __builtin_amdgcn_readfirstlane(py);
        g = refresh_geometry<R>(d, px, py);
        post_best(L, gather<R>(tid, d, px, py, g, C.sup, L));
        lds_barrier();
        // the best pixel that keeps its priority: the usual next target when
        // that is far; its patch and terms are loaded while the search runs
        const Best far = posted_best(L, 0);
        const uint32_t fidx = far.key >= 0 ? far.idx : v.p;
        int fx, fy;
        raster.split(fidx, &fx, &fy);
        const PatchWords fw = load_patch<R>(tid, d, fx, fy);
        const double2 fcd = d.pcd[fidx];
        const FillSlots fs = mark_filled<R>(tid, d, px, py, v.C, g, L, [](int) { return true; });
        stage_gray<R>(tid, L);
        list_front<R, true>(tid, L);
        lds_barrier();
        const int filled = filled_count(L.cnt);
        confidence_terms<R>(tid, L);   // (wave 0, unless the front is long)
        collect_slots<R>(d.fslot, ntiles, slot_tag(k), L);   // (the other waves)
        lds_barrier();
        uint64_t best = ~0ull;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            best = L.smin[q] < best ? L.smin[q] : best;
            if (L.late[q]) v.err = INPAINT_DEVICE;
        }
        const uint32_t ssd = (uint32_t)(best >> kSlotIndexBits), q = (uint32_t)best & ((1u << kSlotIndexBits) - 1);
        if (ssd == (1u << 26) - 1) v.err = INPAINT_NO_CANDIDATE;
        if (v.err) continue;   // publishes stop
        int qx, qy;
        raster.split(q, &qx, &qy);
        copy_colours<R>(tid, d, px, py, qx, qy, fs, L);
        const int64_t remaining = v.remaining - filled;
        if (tid == T - 64) {   // (the last wave has few slots to copy)
            StepRec &rec = C.last;
            rec.target_index = v.p;
            rec.source_index = q;
            rec.ssd = ssd;
            // the patch's in-image pixels that were not filled
            rec.known_k = (min(px + R + 1, d.W) - max(px - R, 0)) * (min(py + R + 1, d.H) - max(py - R, 0)) - filled;
            rec.n_filled = filled;
            rec.reserved = 0;
            rec.priority = v.Pr;
            rec.confidence = v.C;
            rec.data_term = v.D;
            rec.remaining = remaining;
        }
        ran = logged = true;
        v.iter += 1;
        v.remaining = remaining;
        v.pending = 0;
        lds_barrier();   // also publishes C.last to the lanes that log it
        if (remaining == 0) {
            v.done = 1;
            continue;
        }
        refresh_grads<R>(tid, d, px, py, L);
        lds_barrier();
        data_terms<R>(tid, d, px, py, g, L);
        lds_barrier();
        stale = true;
        int wv;
        const Best near = posted_best(L, 1, &wv);
        const bool is_far = better(far.key, far.idx, near.key, near.idx);
        const Best next = is_far ? far : near;
        if (next.key < 0) {
            // No front pixel although the hole is not empty: cannot happen
            // for a valid state; flag it instead of looping.
            v.err = INPAINT_DEVICE;
            continue;
        }
        // ---- stage the next target: from the registers that hold the far
        // patch, or from the neighbourhood, which covers the patch of every
        // pixel of the refresh window
        int tx, ty;
        raster.split(next.idx, &tx, &ty);
        const uint32_t tag = rec_tag(v.iter);
#pragma unroll
        for (int j = 0; j < kSlots; ++j) {
            const int t = tid + j * T;
            if (j * T >= P * P || t >= P * P) continue;
            const uint32_t w = is_far ? fw.w[j] : L.img[S::at(tx - px + t / P - R, ty - py + t % P - R)];
            write_word(t, w, state_of(w) == 0, tag);
        }
        v.p = next.idx;
        v.C = is_far ? fcd.x : L.wC[wv];
        v.D = is_far ? fcd.y : L.wD[wv];
        v.Pr = v.C * v.D;
        v.pending = 1;
    }

    IterState *st = d.st;
    if (tid == 0) {
        if (v.err) st->error = v.err;
        if (ran) {
            st->remaining = v.remaining;
            st->iter = v.iter;
            st->done = v.done;
            st->pending = v.pending;
            st->p_idx = v.p;
            st->C = v.C;
            st->D = v.D;
            st->Pr = v.Pr;
            st->last = C.last;
        }
    }
    if (ran && v.pending && !v.err) {
        int tx, ty;
        raster.split(v.p, &tx, &ty);
        stage_slots(R, tx, ty, d.tgt, C.s, [&](int t, int, uint32_t *pix) {
            const uint32_t w = L.tword[t];
            *pix = w & kColour;
            return (w >> 31) != 0;
        });
    }
}

// Search groups: waits until the words of record `rec` carry `tag` and hands
// this thread's (column-major slots tid + 256 j); false after kSpinLimit
// polls.  Words are read with agent-scope loads, which eventually return the
// latest store, and each says which iteration it belongs to, so nothing rests
// on the order in which the committer's stores arrive.
template <int R>
struct RecWords {
    static constexpr int N = (2 * R + 1) * (2 * R + 1), J = (N + kSearchWaves * 64 - 1) / (kSearchWaves * 64);
    uint32_t w[J];
    __device__ __forceinline__ void load(const FillRec *rec) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int t = threadIdx.x + j * kSearchWaves * 64;
            if (t < N) w[j] = __hip_atomic_load(&rec->tpix[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __device__ __forceinline__ bool fresh(uint32_t tag) const {
        bool ok = true;
#pragma unroll
        for (int j = 0; j < J; ++j)
            if ((int)threadIdx.x + j * kSearchWaves * 64 < N) ok = ok && ((w[j] >> 24) & 0x7fu) == tag;
        return ok;
    }
    __device__ __forceinline__ bool known(int j) const { return (w[j] >> 31) != 0; }
};

// Bit i of column_slots<P>(base, k): slot base + i of a P x P patch in
// column-major order is the k-th of its column.
template <int P>
constexpr uint64_t column_slots(int base, int k) {
    uint64_t m = 0;
    for (int i = 0; i < 64; ++i) m |= (uint64_t)((base + i) % P == k) << i;
    return m;
}
// The slots of rounds of 64 that start and end a column.
template <int P>
struct ColumnEnds {
    uint64_t top[kMaxOffsets / 64 + 1], end[kMaxOffsets / 64 + 1];
    constexpr ColumnEnds() : top(), end() {
        for (int j = 0; j < kMaxOffsets / 64 + 1; ++j) {
            top[j] = column_slots<P>(64 * j, 0);
            end[j] = column_slots<P>(64 * j, P - 1);
        }
    }
};

// The target of a record as the SIMT search reads it: words, known mask,
// column-run bits (run_bits) and T2.  Every wave reads all the words, until
// they carry `tag`, so that each has the whole known mask in its ballots and
// forms its share of the bits from scalars: one barrier, the caller's, which
// publishes the target and every wave's ok[] (0 after kSpinLimit reads).
// (Shared reads with the mask put together in LDS took three barriers a
// target: 64 images, us an iteration, radius 3 127 -> 117, radius 6 429 -> 410.)
template <int R>
__device__ __forceinline__ void read_target(const FillRec *rec, uint32_t tag, tile::TargetLds *t, int32_t *ok) {
    constexpr int P = 2 * R + 1, N = P * P, J = (N + 63) / 64;
    constexpr ColumnEnds<P> ends;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t w[J];
    bool fresh = false;
    for (uint32_t spin = 0; !fresh && spin < kSpinLimit; ++spin) {
        bool mine = true;
#pragma unroll
        for (int j = 0; j < J; ++j)
            w[j] = __hip_atomic_load(&rec->tpix[min(lane + 64 * j, N - 1)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < J; ++j) mine = mine && ((w[j] >> 24) & 0x7fu) == tag;
        fresh = __ballot(!mine) == 0;
    }
    uint64_t known[J];
    uint32_t t2 = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const bool kn = lane + 64 * j < N && (w[j] >> 31) != 0;
        known[j] = __ballot(kn);
        w[j] = kn ? w[j] & kColour : 0u;
        t2 = __builtin_amdgcn_udot4(w[j], w[j], t2, false);
    }
    t2 = dpp::sum_u32(t2);
#pragma unroll
    for (int j = 0; j < J; ++j) {
        if ((j & 3) != wave) continue;
        if (lane + 64 * j < N) t->tpix[lane + 64 * j] = w[j];
        const uint64_t m = known[j];
        const uint64_t up = m << 1 | (j > 0 ? known[j > 0 ? j - 1 : 0] >> 63 : 0ull);              // slot - 1 known
        const uint64_t dn = m >> 1 | (j + 1 < J ? known[j + 1 < J ? j + 1 : j] << 63 : 0ull);      // slot + 1 known
        const uint64_t sb = m & (ends.top[j] | ~up), eb = m & (ends.end[j] | ~dn);
        if (lane == 0) {
            t->mbits[2 * j] = (uint32_t)m;
            t->mbits[2 * j + 1] = (uint32_t)(m >> 32);
            t->sbits[2 * j] = (uint32_t)sb;
            t->sbits[2 * j + 1] = (uint32_t)(sb >> 32);
            t->ebits[2 * j] = (uint32_t)eb;
            t->ebits[2 * j + 1] = (uint32_t)(eb >> 32);
        }
    }
    if (lane == 0) ok[wave] = fresh;
    if (threadIdx.x == 0) t->t2 = t2;
}
__device__ __forceinline__ bool all_ok(const int32_t *ok) { return ok[0] && ok[1] && ok[2] && ok[3]; }
static_assert(kSearchWaves == 4, "one ok word per wave");

// A SIMT search group's wait for iteration k (whole group): one lane polls
// the go word.  (Up to four such groups share a CU, a thousand the device:
// polling whole records slows the committer's own loads more than the round
// trip it saves.)  False on stop or time-out.
__device__ __forceinline__ bool wait_go(const FillRec *rec, uint32_t epoch, uint32_t k, int32_t *flag, uint32_t *tag) {
    if (threadIdx.x == 0) {
        int f = 0;
        for (uint32_t spin = 0; spin < kSpinLimit; ++spin) {
            const uint64_t v = __hip_atomic_load(&rec->go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (go_is(v, epoch, k + 1)) {
                *tag = go_tag(v);
                f = 1;
                break;
            }
            if (v == go_stop(epoch)) break;
            __builtin_amdgcn_s_sleep(1);
        }
        *flag = f;
    }
    __syncthreads();
    return *flag != 0;
}

// A search group's wait for iteration k (whole group): each poll reads the go
// word (thread 0) and the record's words together, so the target arrives with
// the go word instead of one memory round trip after it; stale words are read
// again.  False on stop or time-out.  `words`: whether this group needs them.
template <int R>
__device__ __forceinline__ bool wait_target(const FillRec *rec, uint32_t epoch, uint32_t k, bool words,
                                            RecWords<R> &rw, int32_t *flag, uint32_t *tag) {
    for (uint32_t spin = 0;; ++spin) {
        uint64_t gv = 0;
        if (threadIdx.x == 0) gv = __hip_atomic_load(&rec->go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (words) rw.load(rec);
        if (threadIdx.x == 0) {
            // 1: go for iteration k (its tag in *tag), 0: stop or time-out, -1: not yet
            *flag = go_is(gv, epoch, k + 1) ? 1 : (gv == go_stop(epoch) ? 0 : -1);
            if (spin >= kSpinLimit) *flag = 0;
            *tag = go_tag(gv);
        }
        __syncthreads();
        const int f = *flag;
        // (words of an earlier dispatch may carry the first iteration's tag:
        // there they are read after go, which the committer orders after them)
        if (f == 1 && k == 0 && words) rw.load(rec);
        if (f == 1 && __syncthreads_and(!words || rw.fresh(*tag))) return true;
        if (f == 0) return false;
        if (f == -1) __builtin_amdgcn_s_sleep(1);
        __syncthreads();   // thread 0 rewrites *flag only after everyone read it
    }
}

template <int R, int NY>
struct SearchLds {
    __attribute__((aligned(16))) uint32_t tile[tile::TileGeom<R, NY>::LDS_WORDS];
    tile::TargetLds tgt;
    uint64_t red[kSearchWaves];
    int32_t ok[kSearchWaves];
    int32_t flag;
    uint32_t tag;
};

template <int R, int NY>
union FillLds {
    FillCommitLds<R> c;
    SearchLds<R, NY> s;
};

template <int R, int NY>
__device__ __forceinline__ void fill_search(const JobDev &d, int ntiles, uint32_t epoch, SearchLds<R, NY> &S) {
    // The tile stays in this group's LDS for the whole dispatch, so the
    // order of tiles over the XCDs does not matter here.
    const int t = (int)blockIdx.x - 1;
    int tx0, ty0;
    tile::tile_origin<R, NY>(d.rx0, d.ry0, d.ntx, t, &tx0, &ty0);
    const uint32_t vmask = tile::stage_tile<R, NY>(d, tx0, ty0, d.rx1, d.ry1, S.tile);
    const bool anyv = __syncthreads_or(vmask != 0);
    const FillRec *rec = &d.sync->rec[t % kGoCopies];
    for (uint32_t k = 0;; ++k) {
        if (!wait_go(rec, epoch, k, &S.flag, &S.tag)) break;
        uint64_t best = ~0ull;
        if (anyv) {
            read_target<R>(rec, S.tag, &S.tgt, S.ok);
            __syncthreads();
            if (!all_ok(S.ok)) break;
            const tile::LdsTarget view{&S.tgt};
            best = tile::wave_min_u64(tile::score_tile<R, NY>(d, view, tx0, ty0, vmask, S.tile));
            if ((threadIdx.x & 63) == 0) S.red[threadIdx.x >> 6] = best;
            __syncthreads();
            if (threadIdx.x == 0)
                for (int w = 0; w < kSearchWaves; ++w) best = S.red[w] < best ? S.red[w] : best;
        }
        if (threadIdx.x == 0)
            __hip_atomic_store(&d.fslot[t], slot_word(best, slot_tag(k)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    }
}

// Search tiles a group of the batched MFMA dispatch keeps in LDS.  Two of
// radius up to 6 fit beside the tables with two groups per CU; the commit of
// radius 7 leaves room for one, that of radius 8 only lets one group onto a
// CU, which then holds three.
template <int R>
constexpr int kMultiTiles = R <= 6 ? 2 : (R == 7 ? 1 : 3);

template <int R, int NT = 1>
struct SearchLdsMfma {
    mtile::MfmaTile<R> tile[NT];
    mtile::FragTables<R> ft;
    uint64_t red[kSearchWaves];
    int32_t flag;
    uint32_t tag;
};

template <int R, int NT = 1>
union FillLdsMfma {
    FillCommitLds<R> c;
    SearchLdsMfma<R, NT> s;
};
static_assert(sizeof(FillLdsMfma<6, kMultiTiles<6>>) + 256 <= 80 * 1024 && sizeof(FillLdsMfma<7, kMultiTiles<7>>) + 256 <= 80 * 1024,
              "two work-groups per CU");
static_assert(sizeof(FillLdsMfma<8, kMultiTiles<8>>) + 256 <= 160 * 1024, "one work-group per CU");

// Search group of the MFMA form: one 64 x 64 tile of the MFMA tiling, staged
// once; per target it builds the B-operand tables in LDS from the record and
// scores the tile on the matrix cores.
template <int R>
__device__ __forceinline__ void fill_search_mfma(const JobDev &d, uint32_t epoch, SearchLdsMfma<R> &S) {
    const int t = (int)blockIdx.x - 1;
    int tx0, ty0;
    mtile::tile_origin<R>(d.rx0, d.ry0, d.ntx, t, &tx0, &ty0);
    mtile::clear_tables<R>(&S.ft);
    const uint32_t vmask = mtile::stage_tile<R>(d, tx0, ty0, d.rx0, d.rx1, d.ry1, S.tile[0]);
    const bool anyv = __syncthreads_or(vmask != 0);
    const FillRec *rec = &d.sync->rec[t % kGoCopies];
    for (uint32_t k = 0;; ++k) {
        RecWords<R> rw;
        if (!wait_target<R>(rec, epoch, k, anyv, rw, &S.flag, &S.tag)) break;
        uint64_t best = ~0ull;
        if (anyv) {
            // the target from the record words into the tables
            mtile::build_tables<R>(
                &S.ft, [&](int, int j) { return rw.w[j]; }, [&](int, int j) { return rw.known(j); });
            __syncthreads();
            best = tile::wave_min_u64(mtile::score_tile_rows<R>(d, &S.ft, tx0, ty0, vmask, S.tile[0]));
            if ((threadIdx.x & 63) == 0) S.red[threadIdx.x >> 6] = best;
            __syncthreads();
            if (threadIdx.x == 0)
                for (int w = 0; w < kSearchWaves; ++w) best = S.red[w] < best ? S.red[w] : best;
        }
        if (threadIdx.x == 0)
            __hip_atomic_store(&d.fslot[t], slot_word(best, slot_tag(k)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    }
}

// Waves per SIMD of the MFMA form: radius 8 has LDS for one group per CU.
constexpr int mfma_waves(int r) { return r <= 7 ? 2 : 1; }

template <int R>
__global__ __launch_bounds__(kCommitThreads) __attribute__((amdgpu_waves_per_eu(mfma_waves(R)))) void k_fill_mfma(JobDev d, int ntiles, int n_iters, uint32_t epoch) {
    __shared__ FillLdsMfma<R> lds;
    if (blockIdx.x == 0)
        fill_commit<R>(d, ntiles, n_iters, epoch, lds.c);
    else
        fill_search_mfma<R>(d, epoch, lds.s);
}

// Waves per SIMD of the SIMT form: what the LDS of its work-groups leaves room
// for (left to itself the compiler spends the registers of fewer, and the
// tiles of a large image no longer fit the resident groups).
constexpr int simt_waves(int r, bool multi) { return r <= 4 ? 4 : (r == 5 && multi ? 3 : (r <= 7 ? 2 : 1)); }

template <int R>
__global__ __launch_bounds__(kCommitThreads) __attribute__((amdgpu_waves_per_eu(simt_waves(R, false)))) void k_fill(JobDev d, int ntiles, int n_iters, uint32_t epoch) {
    __shared__ FillLds<R, kFillTileRows> lds;
    if (blockIdx.x == 0)
        fill_commit<R>(d, ntiles, n_iters, epoch, lds.c);
    else
        fill_search<R, kFillTileRows>(d, ntiles, epoch, lds.s);
}

// ---- batched persistent fill: many jobs in one dispatch -----------------
//
// Work-groups [0, n_commit) each commit one job (fill_commit, exactly as in
// the single-job kernels, on that job's own records and slot words).  Every
// other work-group is a search group owning a list of (job, tile) items; a
// job's tiles are spread over many groups and a group's items come from
// many jobs.  Wave 0 keeps one item per lane -- its job, tile and the job
// iteration it scores next -- and polls all its items' go words at once.
// The group then serves one ready item, taken round-robin: stage the tile
// unless it is the one already in LDS, read the job's record, score, and
// write the job's slot word of that tile.  So a search group never waits on
// one job while another has work for it, and a job's iteration is scored by
// whichever groups are free.  A group with a single item keeps its tile in
// LDS for the whole dispatch, as the single-job kernels do.  Every wait is
// bounded as there: committers time out on their slots and publish stop; a
// search group gives up after kSpinLimit empty polls in a row.

struct MultiPick {
    int32_t pick;       // item to serve, -1: none ready
    int32_t all_done;   // every item's job published stop
    int32_t slot, tile;
    uint32_t k;
    uint32_t tag;       // record tag the item's go word carries
};

// Wave 0: polls the go words of this group's items (lane i: item i) and
// publishes the next ready item after `rot` (round-robin) in *pk.  my_k is
// the job iteration lane i's item scores next; it advances for the item
// picked.  The caller's barrier publishes *pk.
__device__ __forceinline__ void multi_poll(const uint64_t *my_go, int my_slot, int my_tile, uint32_t &my_k,
                                           bool &my_done, int rot, uint32_t epoch, MultiPick *pk) {
    const int lane = threadIdx.x & 63;
    bool ready = false;
    uint64_t v = 0;
    if (!my_done) {
        v = __hip_atomic_load(my_go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ready = go_is(v, epoch, my_k + 1);
        my_done = v == go_stop(epoch);
    }
    const uint64_t rb = __ballot(ready), db = __ballot(my_done);
    const uint64_t hi = rb & (~0ull << rot);
    const int pick = hi ? __builtin_ctzll(hi) : (rb ? __builtin_ctzll(rb) : -1);
    if (lane == 0) {
        pk->pick = pick;
        pk->all_done = db == ~0ull;
    }
    if (lane == pick) {
        pk->slot = my_slot;
        pk->tile = my_tile;
        pk->k = my_k;
        pk->tag = go_tag(v);
        my_k += 1;
    }
}

// The record's words of the iteration with this tag; false after kSpinLimit
// reads.
template <int R>
__device__ __forceinline__ bool read_record(const FillRec *rec, uint32_t tag, RecWords<R> &rw) {
    for (uint32_t spin = 0; spin < kSpinLimit; ++spin) {
        rw.load(rec);
        if (__syncthreads_and(rw.fresh(tag))) return true;
    }
    return false;
}

// What a search group does with one item (job d, tile t) for iteration k.
struct ServeItem {
    int t;
    uint32_t k, tag;   // the job's iteration and the record tag its go word carried
    int at;            // LDS tile to use
    bool restage;      // that tile is not this item's
    bool build;        // the target's tables in LDS are not this job's for iteration k
};

// Scores an item of the MFMA form and reports in the job's slot word.  True
// when the target tables are now the job's of iteration k.
template <int R>
__device__ __forceinline__ bool multi_serve_mfma(const JobDev &d, const ServeItem &it, SearchLdsMfma<R, kMultiTiles<R>> &S,
                                                 uint32_t &vmask, bool &anyv) {
    int tx0, ty0;
    mtile::tile_origin<R>(d.rx0, d.ry0, d.ntx, it.t, &tx0, &ty0);
    mtile::MfmaTile<R> &tile = S.tile[it.at];
    if (it.restage) {
        vmask = mtile::stage_tile<R>(d, tx0, ty0, d.rx0, d.rx1, d.ry1, tile);
        anyv = __syncthreads_or(vmask != 0);
    }
    if (it.build && anyv) {
        // the record words of iteration k: read until every one carries the
        // go word's tag (bounded; on a time-out no slot word is written, and
        // the committer's bounded wait reports the device error)
        RecWords<R> rw;
        if (!read_record<R>(&d.sync->rec[it.t % kGoCopies], it.tag, rw)) return false;
        mtile::build_tables<R>(
            &S.ft, [&](int, int j) { return rw.w[j]; }, [&](int, int j) { return rw.known(j); });
        __syncthreads();
    }
    uint64_t best = ~0ull;
    if (anyv) {
        best = tile::wave_min_u64(mtile::score_tile_rows<R>(d, &S.ft, tx0, ty0, vmask, tile));
        if ((threadIdx.x & 63) == 0) S.red[threadIdx.x >> 6] = best;
        __syncthreads();
        if (threadIdx.x == 0)
            for (int w = 0; w < kSearchWaves; ++w) best = S.red[w] < best ? S.red[w] : best;
    }
    if (threadIdx.x == 0)
        __hip_atomic_store(&d.fslot[it.t], slot_word(best, slot_tag(it.k)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return anyv || !it.build;
}

// The same for the SIMT form.
template <int R>
__device__ __forceinline__ bool multi_serve_simt(const JobDev &d, const ServeItem &it, SearchLds<R, kFillTileRows> &S,
                                                 uint32_t &vmask, bool &anyv) {
    constexpr int NY = kFillTileRows;
    int tx0, ty0;
    tile::tile_origin<R, NY>(d.rx0, d.ry0, d.ntx, it.t, &tx0, &ty0);
    if (it.restage) {
        vmask = tile::stage_tile<R, NY>(d, tx0, ty0, d.rx1, d.ry1, S.tile);
        anyv = __syncthreads_or(vmask != 0);
    }
    if (it.build && anyv) {
        read_target<R>(&d.sync->rec[it.t % kGoCopies], it.tag, &S.tgt, S.ok);
        __syncthreads();
        if (!all_ok(S.ok)) return false;
    }
    uint64_t best = ~0ull;
    if (anyv) {
        const tile::LdsTarget view{&S.tgt};
        best = tile::wave_min_u64(tile::score_tile<R, NY>(d, view, tx0, ty0, vmask, S.tile));
        if ((threadIdx.x & 63) == 0) S.red[threadIdx.x >> 6] = best;
        __syncthreads();
        if (threadIdx.x == 0)
            for (int w = 0; w < kSearchWaves; ++w) best = S.red[w] < best ? S.red[w] : best;
    }
    if (threadIdx.x == 0)
        __hip_atomic_store(&d.fslot[it.t], slot_word(best, slot_tag(it.k)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return anyv || !it.build;
}

// Search group w of a batched dispatch; serve(d, item, vmask, anyv) scores
// one item.  Of NT LDS tiles, item i of a group with more than NT items uses
// tile min(i, NT - 1): the first NT - 1 items stay in LDS for the whole
// dispatch and the others take turns in the last tile (least-recently-used
// tiles would all miss, as items come round in turn).
template <int NT, class Serve>
__device__ __forceinline__ void multi_search(const MultiPlan &m, int w, uint32_t epoch, MultiPick *pk, Serve serve) {
    const int i0 = m.first[w], ni = m.first[w + 1] - i0;   // 0 <= ni <= kMultiMaxItems (host-checked)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int my_slot = 0, my_tile = 0;
    uint32_t my_k = 0;
    bool my_done = true;
    const uint64_t *my_go = nullptr;   // go word of the record this lane's item reads
    if (wave == 0 && lane < ni) {
        const WorkItem it = m.items[i0 + lane];
        my_slot = it.slot;
        my_tile = it.tile;
        my_go = &m.slots[my_slot].sync->rec[my_tile % kGoCopies].go;
        my_done = false;
    }
    uint32_t vmask[NT] = {};
    bool anyv[NT] = {};
    int staged[NT];   // items whose tiles are in LDS
#pragma unroll
    for (int j = 0; j < NT; ++j) staged[j] = -1;
    int built_slot = -1;   // the target tables in LDS are this job's
    uint32_t built_k = 0;  // for this iteration
    int rot = 0;
    for (uint32_t spin = 0; spin < kSpinLimit;) {
        if (wave == 0) multi_poll(my_go, my_slot, my_tile, my_k, my_done, rot, epoch, pk);
        __syncthreads();
        const int pick = __builtin_amdgcn_readfirstlane(pk->pick);
        if (pick < 0) {
            if (pk->all_done) break;
            ++spin;
            __builtin_amdgcn_s_sleep(1);
            __syncthreads();   // wave 0 rewrites *pk only after everyone read it
            continue;
        }
        spin = 0;
        rot = pick + 1 < ni ? pick + 1 : 0;
        // (uniform: the job's fields the search reads become scalar loads)
        const int slot = __builtin_amdgcn_readfirstlane(pk->slot);
        ServeItem it;
        it.t = __builtin_amdgcn_readfirstlane(pk->tile);
        it.k = (uint32_t)__builtin_amdgcn_readfirstlane((int)pk->k);
        it.tag = (uint32_t)__builtin_amdgcn_readfirstlane((int)pk->tag);
        it.at = min(pick, NT - 1);
        it.build = slot != built_slot || it.k != built_k;
        uint32_t vm = 0;
        bool av = false;
        it.restage = true;
#pragma unroll
        for (int j = 0; j < NT; ++j)
            if (j == it.at) {
                it.restage = staged[j] != pick;
                vm = vmask[j];
                av = anyv[j];
            }
        const JobDev d = m.slots[slot];
        const bool ok = serve(d, it, vm, av);
        built_slot = ok ? slot : -1;
        built_k = it.k;
#pragma unroll
        for (int j = 0; j < NT; ++j)
            if (j == it.at) {
                staged[j] = pick;
                vmask[j] = vm;
                anyv[j] = av;
            }
        __syncthreads();
    }
}

template <int R>
__global__ __launch_bounds__(kCommitThreads) __attribute__((amdgpu_waves_per_eu(mfma_waves(R)))) void k_fill_multi_mfma(
    MultiPlan m, int n_iters, uint32_t epoch) {
    __shared__ FillLdsMfma<R, kMultiTiles<R>> lds;
    __shared__ MultiPick pk;
    if ((int)blockIdx.x < m.n_commit) {
        // by value: held through a reference to device memory, the job's
        // fields would stay live in vector registers (and spill)
        const JobDev d = m.slots[m.commit[blockIdx.x]];
        fill_commit<R>(d, d.ntx * d.nty, n_iters, epoch, lds.c);
        return;
    }
    mtile::clear_tables<R>(&lds.s.ft);   // (published by the first poll's barrier)
    multi_search<kMultiTiles<R>>(m, (int)blockIdx.x - m.n_commit, epoch, &pk,
                              [&](const JobDev &d, const ServeItem &it, uint32_t &vmask, bool &anyv)
                                  __attribute__((always_inline)) { return multi_serve_mfma<R>(d, it, lds.s, vmask, anyv); });
}

template <int R>
__global__ __launch_bounds__(kCommitThreads) __attribute__((amdgpu_waves_per_eu(simt_waves(R, true)))) void k_fill_multi(
    MultiPlan m, int n_iters, uint32_t epoch) {
    __shared__ FillLds<R, kFillTileRows> lds;
    __shared__ MultiPick pk;
    if ((int)blockIdx.x < m.n_commit) {
        const JobDev d = m.slots[m.commit[blockIdx.x]];   // by value, see k_fill_multi_mfma
        fill_commit<R>(d, d.ntx * d.nty, n_iters, epoch, lds.c);
        return;
    }
    multi_search<1>(m, (int)blockIdx.x - m.n_commit, epoch, &pk,
                    [&](const JobDev &d, const ServeItem &it, uint32_t &vmask, bool &anyv)
                        __attribute__((always_inline)) { return multi_serve_simt<R>(d, it, lds.s, vmask, anyv); });
}

// The MFMA form for jobs of several radii in one dispatch: the LDS of the
// largest radius; each committer takes its job's radius, and each search
// group the radius of its items (the plan gives a search group items of one
// radius only), so every work-group runs the per-radius code of its own
// radius for the whole dispatch.
union MixLdsMfma {
    FillLdsMfma<1, kMultiTiles<1>> r1;
    FillLdsMfma<2, kMultiTiles<2>> r2;
    FillLdsMfma<3, kMultiTiles<3>> r3;
    FillLdsMfma<4, kMultiTiles<4>> r4;
    FillLdsMfma<5, kMultiTiles<5>> r5;
};
static_assert(kMultiMixMaxR == 5, "MixLdsMfma holds radii 1..5");

template <int R>
__device__ __forceinline__ void mixed_role(const MultiPlan &m, int n_iters, uint32_t epoch, FillLdsMfma<R, kMultiTiles<R>> &lds,
                                           MultiPick *pk) {
    if ((int)blockIdx.x < m.n_commit) {
        const JobDev d = m.slots[m.commit[blockIdx.x]];   // by value, see k_fill_multi_mfma
        fill_commit<R>(d, d.ntx * d.nty, n_iters, epoch, lds.c);
        return;
    }
    mtile::clear_tables<R>(&lds.s.ft);   // (published by the first poll's barrier)
    multi_search<kMultiTiles<R>>(m, (int)blockIdx.x - m.n_commit, epoch, pk,
                              [&](const JobDev &d, const ServeItem &it, uint32_t &vmask, bool &anyv)
                                  __attribute__((always_inline)) { return multi_serve_mfma<R>(d, it, lds.s, vmask, anyv); });
}

#if INPAINT_FILL_PART == 3
__global__ __launch_bounds__(kCommitThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_fill_multi_mfma_mixed(
    MultiPlan m, int n_iters, uint32_t epoch) {
    __shared__ MixLdsMfma lds;
    __shared__ MultiPick pk;
    // this work-group's radius: its job's, or its first item's (a search
    // group without items has nothing to serve)
    int r = 0;
    if ((int)blockIdx.x < m.n_commit) {
        r = m.slots[m.commit[blockIdx.x]].r;
    } else {
        const int w = (int)blockIdx.x - m.n_commit;
        if (m.first[w + 1] > m.first[w]) r = m.slots[m.items[m.first[w]].slot].r;
    }
    switch (r) {
        case 1: mixed_role<1>(m, n_iters, epoch, lds.r1, &pk); break;
        case 2: mixed_role<2>(m, n_iters, epoch, lds.r2, &pk); break;
        case 3: mixed_role<3>(m, n_iters, epoch, lds.r3, &pk); break;
        case 4: mixed_role<4>(m, n_iters, epoch, lds.r4, &pk); break;
        case 5: mixed_role<5>(m, n_iters, epoch, lds.r5, &pk); break;
        default: break;   // no items; the host plan holds only radii 1 .. 5
    }
}
#endif

template <int R, bool ISECT>
__global__ __launch_bounds__(kCommitThreads) void k_commit(JobDev d) {
    __shared__ Scratch s;
    __shared__ CommitLds<R> L;
    __shared__ CommitNote note;
    if (threadIdx.x == 0) note.filled = 0;
    commit_body<R, ISECT>(d, s, L, &note);
    if (d.policy == INPAINT_SOURCE_CURRENT) {
        __syncthreads();
        if (note.filled > 0) add_filled_sources<R, ISECT>(d, L, col_of(note.p, d.W), row_of(note.p, d.W));
    }
}

// One work-group per listed slot (all with patch radius R); the list length
// is read from device memory so the slot list can change between graph
// replays without re-capture.
template <int R>
__global__ __launch_bounds__(kCommitThreads) void k_commit_batched(const JobDev *slots, const int32_t *ids,
                                                                   const int32_t *n) {
    __shared__ Scratch s;
    __shared__ CommitLds<R> L;
    if ((int)blockIdx.x >= *n) return;
    const JobDev d = slots[ids[blockIdx.x]];
    if (d.st == nullptr) return;   // empty slot
    commit_body<R>(d, s, L, nullptr);
}

#if INPAINT_FILL_PART == 0
__global__ __launch_bounds__(kCommitThreads) void k_stage_query(JobDev d, int tx, int ty, int r) {
    __shared__ Scratch s;
    stage_target(d, tx, ty, r, d.qtgt, s);
}

__global__ __launch_bounds__(kCommitThreads) void k_reduce_partials(const uint64_t *partials, int n,
                                                                   uint64_t *out) {
    __shared__ uint64_t sh[16];
    uint64_t best = ~0ull;
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
        const uint64_t v = partials[t];
        best = v < best ? v : best;
    }
    best = wave_min(best);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 0; w < kCommitThreads / 64; ++w) best = sh[w] < best ? sh[w] : best;
        *out = best;
    }
}

// Number of attached images that are still unfinished and error-free, and
// each slot's state (0 empty, 1 running, 2 finished, 3 error).
__global__ void k_count_active(const JobDev *slots, int nslots, int64_t *out, int32_t *status) {
    __shared__ int cnt;
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < nslots; i += blockDim.x) {
        const IterState *st = slots[i].st;
        int v = 0;
        if (st) v = st->error ? 3 : (st->done ? 2 : 1);
        if (v == 1) atomicAdd(&cnt, 1);
        status[i] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) *out = cnt;
}
#endif  // INPAINT_FILL_PART 0

// ---------------------------------------------------------------- launchers

#if INPAINT_FILL_PART == 0

static inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

uint32_t init_pixel_blocks(const JobDev &d) {
    return std::min(blocks_for((int64_t)d.W * d.H, 1024), kInitBlocks);
}

static void launch_planes(const JobDev &d, hipStream_t s) {
    hipLaunchKernelGGL(k_init_planes, dim3(blocks_for(d.pitch, 64) * blocks_for(padded_rows(d.H), 16)), dim3(256), 0, s, d,
                       d.hdist);
}

hipError_t launch_seal(const JobDev &d, uint32_t nonce, hipStream_t s) {
    hipLaunchKernelGGL(k_seal, dim3(1), dim3(1), 0, s, d.info, nonce);
    return hipGetLastError();
}

hipError_t launch_init(const JobDev &d, const uint8_t *stage_rgb, int channels, const uint8_t *stage_mask,
                       int64_t remaining, int nslots, uint32_t nonce, hipStream_t s) {
    hipLaunchKernelGGL(k_init_info, dim3(std::min(blocks_for(nslots, 256), 64u)), dim3(256), 0, s, d, remaining, nslots,
                       nonce);
    hipLaunchKernelGGL(k_init_pixels, dim3(init_pixel_blocks(d)), dim3(256), 0, s, d, stage_rgb, channels, stage_mask);
    launch_planes(d, s);
    return hipGetLastError();
}

hipError_t launch_import_check(const JobDev &d, const uint8_t *hole, const double *conf, uint32_t nonce,
                               hipStream_t s) {
    hipLaunchKernelGGL(k_import_reset, dim3(1), dim3(1), 0, s, d.info, nonce);
    hipLaunchKernelGGL(k_import_check, dim3(init_pixel_blocks(d)), dim3(256), 0, s, d, hole, conf);
    return hipGetLastError();
}

hipError_t launch_import_apply(const JobDev &d, const uint8_t *rgb, int channels, const uint8_t *hole,
                               const double *conf, uint32_t nonce, hipStream_t s) {
    hipLaunchKernelGGL(k_import_reset, dim3(1), dim3(1), 0, s, d.info, nonce);
    hipLaunchKernelGGL(k_import_apply, dim3(init_pixel_blocks(d)), dim3(256), 0, s, d, rgb, channels, hole, conf);
    // (under the CURRENT policy the source region is the current known region)
    if (d.policy == INPAINT_SOURCE_CURRENT) launch_planes(d, s);
    return hipGetLastError();
}

hipError_t launch_count_valid(const JobDev &d, hipStream_t s) {
    if (d.rx1 <= d.rx0 || d.ry1 <= d.ry0) return hipSuccess;
    hipLaunchKernelGGL(k_count_valid, dim3(std::min((unsigned)(d.ry1 - d.ry0), kInitBlocks)), dim3(256), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_pack_rgb(const uint32_t *img, int64_t count, uint8_t *out, hipStream_t s) {
    hipLaunchKernelGGL(k_pack_rgb, dim3(blocks_for(count, 1024)), dim3(256), 0, s, img, count, out);
    return hipGetLastError();
}

#define INPAINT_RADIUS_SWITCH(r, CALL) \
    switch (r) {                          \
        case 1: CALL(1); break;           \
        case 2: CALL(2); break;           \
        case 3: CALL(3); break;           \
        case 4: CALL(4); break;           \
        case 5: CALL(5); break;           \
        case 6: CALL(6); break;           \
        case 7: CALL(7); break;           \
        case 8: CALL(8); break;           \
        default: return hipErrorInvalidValue; \
    }

hipError_t launch_prio_init(const JobDev &d, hipStream_t s) {
    const int nb = (d.pbx1 - d.pbx0) * (d.pby1 - d.pby0);
#define CALL(R) hipLaunchKernelGGL(k_prio_init<R>, dim3((nb + 3) / 4), dim3(256), 0, s, d)
    INPAINT_RADIUS_SWITCH(d.r, CALL)
#undef CALL
    hipLaunchKernelGGL(k_super_init, dim3((d.nsx * d.nsy + 3) / 4), dim3(256), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_commit(const JobDev &d, hipStream_t s) {
#define CALL(R)                                                                            \
    if (d.isect) hipLaunchKernelGGL((k_commit<R, true>), dim3(1), dim3(kCommitThreads), 0, s, d); \
    else hipLaunchKernelGGL((k_commit<R, false>), dim3(1), dim3(kCommitThreads), 0, s, d)
    INPAINT_RADIUS_SWITCH(d.r, CALL)
#undef CALL
    return hipGetLastError();
}

hipError_t launch_commit_batched(const JobDev *slots, const int32_t *ids, const int32_t *n, int grid, int r,
                                 hipStream_t s) {
    if (grid <= 0) return hipSuccess;
#define CALL(R) hipLaunchKernelGGL(k_commit_batched<R>, dim3(grid), dim3(kCommitThreads), 0, s, slots, ids, n)
    INPAINT_RADIUS_SWITCH(r, CALL)
#undef CALL
    return hipGetLastError();
}

#endif  // INPAINT_FILL_PART 0

// Kernels by radius, nullptr where there is none.
#if INPAINT_FILL_PART == 1
const void *fill_mfma_kernel(int r) {
    switch (r) {
        case 1: return (const void *)k_fill_mfma<1>;
        case 2: return (const void *)k_fill_mfma<2>;
        case 3: return (const void *)k_fill_mfma<3>;
        case 4: return (const void *)k_fill_mfma<4>;
        case 5: return (const void *)k_fill_mfma<5>;
        case 6: return (const void *)k_fill_mfma<6>;
        case 7: return (const void *)k_fill_mfma<7>;
        case 8: return (const void *)k_fill_mfma<8>;
        default: return nullptr;
    }
}
#endif
#if INPAINT_FILL_PART == 0
const void *fill_simt_kernel(int r) {
    switch (r) {
        case 1: return (const void *)k_fill<1>;
        case 2: return (const void *)k_fill<2>;
        case 3: return (const void *)k_fill<3>;
        case 4: return (const void *)k_fill<4>;
        case 5: return (const void *)k_fill<5>;
        case 6: return (const void *)k_fill<6>;
        case 7: return (const void *)k_fill<7>;
        case 8: return (const void *)k_fill<8>;
        default: return nullptr;
    }
}
#endif
#if INPAINT_FILL_PART == 2
const void *multi_mfma_kernel(int r) {
    switch (r) {
        case 1: return (const void *)k_fill_multi_mfma<1>;
        case 2: return (const void *)k_fill_multi_mfma<2>;
        case 3: return (const void *)k_fill_multi_mfma<3>;
        case 4: return (const void *)k_fill_multi_mfma<4>;
        case 5: return (const void *)k_fill_multi_mfma<5>;
        case 6: return (const void *)k_fill_multi_mfma<6>;
        case 7: return (const void *)k_fill_multi_mfma<7>;
        case 8: return (const void *)k_fill_multi_mfma<8>;
        default: return nullptr;
    }
}
#endif
#if INPAINT_FILL_PART == 0
const void *multi_simt_kernel(int r) {
    switch (r) {
        case 1: return (const void *)k_fill_multi<1>;
        case 2: return (const void *)k_fill_multi<2>;
        case 3: return (const void *)k_fill_multi<3>;
        case 4: return (const void *)k_fill_multi<4>;
        case 5: return (const void *)k_fill_multi<5>;
        case 6: return (const void *)k_fill_multi<6>;
        case 7: return (const void *)k_fill_multi<7>;
        case 8: return (const void *)k_fill_multi<8>;
        default: return nullptr;
    }
}
#endif
#if INPAINT_FILL_PART == 3
const void *multi_mixed_kernel() { return (const void *)k_fill_multi_mfma_mixed; }
#endif

#if INPAINT_FILL_PART == 0
static const void *fill_kernel(int r, bool mfma) { return mfma ? fill_mfma_kernel(r) : fill_simt_kernel(r); }

hipError_t fill_blocks_per_cu(int r, bool mfma, int *blocks) {
    const void *f = fill_kernel(r, mfma);
    if (!f) return hipErrorInvalidValue;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, f, kCommitThreads, 0);
}

int fill_grid(int ntiles) { return 1 + ntiles; }

hipError_t launch_fill(const JobDev &d, int ntiles, int n_iters, uint32_t epoch, hipStream_t s) {
    const void *f = fill_kernel(d.r, d.mfma != 0);
    if (!f) return hipErrorInvalidValue;
    JobDev dd = d;
    void *args[] = {&dd, &ntiles, &n_iters, &epoch};
    return hipLaunchKernel(f, dim3(fill_grid(ntiles)), dim3(kCommitThreads), args, 0, s);
}

static const void *fill_multi_kernel(bool mfma, int r) {
    if (!mfma) return multi_simt_kernel(r);
    return r == kMultiMixed ? multi_mixed_kernel() : multi_mfma_kernel(r);
}

hipError_t multi_blocks_per_cu(bool mfma, int r, int *blocks) {
    const void *f = fill_multi_kernel(mfma, r);
    if (!f) return hipErrorInvalidValue;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, f, kCommitThreads, 0);
}

hipError_t launch_fill_multi(const MultiPlan &m, bool mfma, int r, int grid, int n_iters, uint32_t epoch,
                             hipStream_t s) {
    const void *f = fill_multi_kernel(mfma, r);
    if (!f || grid <= m.n_commit) return hipErrorInvalidValue;
    MultiPlan mm = m;
    void *args[] = {&mm, &n_iters, &epoch};
    return hipLaunchKernel(f, dim3(grid), dim3(kCommitThreads), args, 0, s);
}

hipError_t launch_stage_query(const JobDev &d, int tx, int ty, int r, hipStream_t s) {
    hipLaunchKernelGGL(k_stage_query, dim3(1), dim3(kCommitThreads), 0, s, d, tx, ty, r);
    return hipGetLastError();
}

hipError_t launch_reduce_partials(const JobDev &d, int ntiles, uint64_t *out, hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_partials, dim3(1), dim3(kCommitThreads), 0, s,
                       (const uint64_t *)d.partials, ntiles, out);
    return hipGetLastError();
}

hipError_t launch_count_active(const JobDev *slots, int nslots, int64_t *out, int32_t *status, hipStream_t s) {
    hipLaunchKernelGGL(k_count_active, dim3(1), dim3(256), 0, s, slots, nslots, out, status);
    return hipGetLastError();
}
#endif  // INPAINT_FILL_PART 0

}  // namespace inpaint
