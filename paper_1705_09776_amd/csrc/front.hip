// Front end: every input image brought down to a longer side of at most
// kFrontLongSide (640) pixels before the scale space is built (Sec. III:
// the encoder first reduces the resolution so that the longer side is at
// most 640).
//
// Area averaging in exact integer arithmetic.  Along an axis of n input and
// m output pixels, input pixel i spans [i m, (i + 1) m) and output pixel j
// spans [j n, (j + 1) n) in units of 1 / (n m) of the image; their overlap
// is an integer, the output pixel's weighted sum N = sum over its
// footprint of overlap_x * overlap_y * I is an exact integer, and the u8
// output is the mean rounded half up, floor((2 N + W H) / (2 W H)).  An
// image whose longer side is at most 640 maps onto itself (every overlap
// is the whole pixel) and is copied.
//
// A wave takes a segment of the output's columns and a run of its rows, and
// streams their source rows once.  Per output row it first forms the column sums V_i = sum_k overlap_y I_ki of the
// segment's source columns, four columns per lane from 4-byte loads (the row
// weights are the same for every lane; V is below 2^24, so single precision
// sums it exactly), leaves them in LDS, and then each lane sums its outputs'
// footprints: all their columns whole, less the two ends' missing parts.
// Quotients (a footprint's first column, the rounded mean) are reciprocal
// estimates corrected by their remainders, so no integer division is left.
//
// Bound by vector instructions (about 3 per source byte and 40 per output).
// One lane per output pixel that gathered its footprint byte by byte, with
// four integer divisions, took 241 us for 64 camera images of mixed sizes up
// to 2048x1536 (117 MB, 0.48 TB/s); this takes 52 us (2.3 TB/s).  One
// 3264x2448 image: 139 -> 13 us; 64 of 800x600: 101 -> 33 us.  Three or four
// source rows on their way instead of two cost more in registers than they
// hide (76 and 92 us), and so do segments of 768 or 1280 columns (67, 60 us,
// against 60 with 1024, all before the tables of the footprints).
#include "cdvs_internal.h"

namespace cdvs {

namespace {

constexpr int kFrontWaves = 4;                  // per workgroup
constexpr int kFrontLoads = 4;                  // 4-byte loads per lane and source row
constexpr int kFrontCols = 256 * kFrontLoads;   // source columns of a segment
constexpr int kFrontAhead = 2;                  // source rows on their way (see above)

// floor(n / d) and n - d floor(n / d) for 0 <= n < 2^24, 1 <= d < 2^24.
__device__ __forceinline__ int div24(int n, int d, float inv, int& r) {
    int q = (int)((float)n * inv);   // within one of the quotient
    r = n - q * d;
    if (r < 0) {
        --q;
        r += d;
    }
    if (r >= d) {
        ++q;
        r -= d;
    }
    return q;
}

// floor((2 N + WH) / (2 WH)), N <= 255 WH: the estimate is within one of it,
// and the remainder (below 2^32 in magnitude where NARROW, whatever the
// products wrapped to) says which way.
template <bool NARROW>
__device__ __forceinline__ uint32_t rounded_mean(uint64_t N, uint64_t WH, float inv, double dinv) {
    if constexpr (NARROW) {
        const uint32_t n = (uint32_t)N, wh = (uint32_t)WH;
        uint32_t q = (uint32_t)((float)n * inv + 0.5f);
        const int32_t r = (int32_t)(2u * n + wh - q * 2u * wh);
        q += (r >= (int32_t)(2u * wh)) ? 1u : 0u;
        q -= (r < 0) ? 1u : 0u;
        return q;
    } else {
        uint32_t q = (uint32_t)((double)N * dinv + 0.5);
        const int64_t r = (int64_t)(2ull * N + WH - (uint64_t)q * 2ull * WH);
        q += (r >= (int64_t)(2ull * WH)) ? 1u : 0u;
        q -= (r < 0) ? 1u : 0u;
        return q;
    }
}

// One wave: output columns [x0, x1) of the rows [y0, y1).  T: the whole
// columns t0 of a footprint where they are known beforehand, else 0 (then any
// number).
template <bool NARROW, int T>
__device__ __forceinline__ void front_walk(const uint8_t* __restrict__ src, const cdvs_image_desc& s,
                                           uint8_t* __restrict__ dst, const cdvs_image_desc& d, int x0, int x1, int y0,
                                           int y1, uint32_t* V, uint32_t* xp, int lane) {
    const int W = s.width, H = s.height, wo = d.width, ho = d.height;
    const float iwo = 1.f / (float)wo, iho = 1.f / (float)ho;
    const uint64_t WH = (uint64_t)W * (uint64_t)H;
    const float inv = 1.f / (float)WH;
    const double dinv = 1.0 / (double)WH;
    int r;
    const int c0 = div24(x0 * W, wo, iwo, r) & ~3;                  // first source column staged
    const int c1 = div24(x1 * W - 1, wo, iwo, r) + 1;               // past the last one needed
    const int nj = min((c1 - c0 + 255) / 256, kFrontLoads);
    // a footprint is t0 + 1 or t0 + 2 source columns
    const int tq = div24(W - 1, wo, iwo, r), tr = r;                // (W - 1) = t0 wo + tr
    const int t0 = T > 0 ? T : tq;
    // output x starts at column i0, a = x W - i0 wo of whose wo parts lie
    // before it
    for (int x = x0 + lane; x < x1; x += 64) {
        int a;
        const int i0 = div24(x * W, wo, iwo, a);
        xp[x - x0] = (uint32_t)(i0 - c0) | ((uint32_t)a << 16);
    }
    // the source rows of all the output rows in one stream, kFrontAhead of
    // them on their way; a row that two output rows share is read once
    const uint8_t* base = src + s.offset + c0 + 4 * lane;
    const int cl = c0 + 4 * lane;
    uint32_t px[kFrontAhead][kFrontLoads];
    auto load = [&](uint32_t (&p)[kFrontLoads], int k) {
        const uint8_t* row = base + (int64_t)k * s.pitch;
#pragma unroll
        for (int j = 0; j < kFrontLoads; ++j) {
            p[j] = 0;
            if (j < nj && cl + 256 * j < W) {
                if (cl + 256 * j + 4 <= W) {
                    __builtin_memcpy(&p[j], row + 256 * j, 4);   // (of any alignment)
                } else {
                    for (int b = 0; b < 3; ++b)
                        if (cl + 256 * j + b < W) p[j] |= (uint32_t)row[256 * j + b] << (8 * b);
                }
            }
        }
    };
    float acc[kFrontLoads][4];
    auto add = [&](const uint32_t (&p)[kFrontLoads], float wt) {
#pragma unroll
        for (int j = 0; j < kFrontLoads; ++j)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[j][b] = fmaf((float)((p[j] >> (8 * b)) & 255u), wt, acc[j][b]);
    };
    auto clear = [&]() {
#pragma unroll
        for (int j = 0; j < kFrontLoads; ++j)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[j][b] = 0.f;
    };
    // output row y from its column sums
    auto finish = [&](int y) {
#pragma unroll
        for (int j = 0; j < kFrontLoads; ++j)
            if (j < nj)
                *reinterpret_cast<uint4*>(V + 4 * lane + 256 * j) =
                    make_uint4((uint32_t)acc[j][0], (uint32_t)acc[j][1], (uint32_t)acc[j][2], (uint32_t)acc[j][3]);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint8_t* orow = dst + d.offset + (int64_t)y * d.pitch;
#pragma unroll 1
        for (int xw = x0; xw < x1; xw += 64) {
            const uint32_t xa = xp[min(xw + lane, x1 - 1) - x0];
            const uint32_t* v = V + (xa & 0xffffu);
            const uint32_t a = xa >> 16;
            const int ai = (int)a;
            const uint32_t first = v[0];
            uint32_t sum = first, last = first;
            if constexpr (T > 0) {
#pragma unroll
                for (int t = 1; t <= T; ++t) {
                    last = v[t];
                    sum += last;
                }
            } else {
                for (int t = 1; t <= t0; ++t) {
                    last = v[t];
                    sum += last;
                }
            }
            // (a + W - 1) / wo columns after the first: t0, or one more
            const bool extra = ai + tr >= wo;
            const uint32_t e = v[t0 + 1];
            sum += extra ? e : 0u;
            last = extra ? e : last;
            const uint32_t b = (uint32_t)((t0 + 1 + (extra ? 1 : 0)) * wo - ai - W);   // parts past its end
            uint64_t N;
            if constexpr (NARROW) N = (uint32_t)wo * sum - a * first - b * last;
            else N = (uint64_t)(uint32_t)wo * sum - (uint64_t)a * first - (uint64_t)b * last;
            const uint32_t q = rounded_mean<NARROW>(N, WH, inv, dinv);
            if (xw + lane < x1) orow[xw + lane] = (uint8_t)q;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();   // V is rewritten by the next row
    };
    int before, after;
    const int kbeg = div24(y0 * H, ho, iho, before), kend = div24(y1 * H - 1, ho, iho, after);
#pragma unroll
    for (int u = 0; u < kFrontAhead; ++u) load(px[u], min(kbeg + u, kend));
    clear();
    // of each source row's ho parts, `part` are still to be given out, and the
    // output row y still needs `need` of its H
    int y = y0, need = H, part = ho - before;
    for (int k = kbeg; k <= kend; k += kFrontAhead) {
#pragma unroll
        for (int u = 0; u < kFrontAhead; ++u) {
            if (k + u <= kend) {   // uniform over the wave
                const int w = min(part, need);
                add(px[u], (float)w);
                need -= w;
                if (need == 0) {
                    finish(y);
                    ++y;
                    clear();
                    add(px[u], (float)(part - w));
                    need = H - (part - w);
                }
                part = ho;
                load(px[u], min(k + u + kFrontAhead, kend));
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_front(const uint8_t* __restrict__ src,
                                               const cdvs_image_desc* __restrict__ sdesc,
                                               uint8_t* __restrict__ dst, const cdvs_image_desc* __restrict__ ddesc,
                                               int n, int parts, int32_t* __restrict__ flags) {
    __shared__ __align__(16) uint32_t V[kFrontWaves][kFrontCols + 4];
    __shared__ uint32_t xp[kFrontWaves][kFrontLongSide];
    const int img = blockIdx.x / parts, part = blockIdx.x % parts;
    if (img >= n) return;
    const cdvs_image_desc s = sdesc[img], d = ddesc[img];
    const int W = s.width, H = s.height;
    int wo = -1, ho = -1;
    if (W >= 1 && H >= 1 && W <= CDVS_MAX_SIDE && H <= CDVS_MAX_SIDE && s.pitch >= W && s.offset >= 0)
        front_size(W, H, &wo, &ho);
    if (wo != d.width || ho != d.height) {   // uniform over the workgroup
        if (part == 0 && threadIdx.x == 0) atomicOr(flags, kFlagFrontShape);
        return;
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (W == 2 * wo && H == 2 * ho && ((s.offset | s.pitch | d.offset | d.pitch) & 7) == 0) {
        // An exact factor of 2 (e.g. 1280x960 -> 640x480): every overlap is
        // a whole source pixel, so N = wo ho S for the 2x2 sum S, W H =
        // 4 wo ho, and the rounded mean is (S + 2) / 4 -- the same integers
        // as below.  Each lane takes 4 outputs from 8 bytes of both source
        // rows (8-byte aligned: offsets and pitches are multiples of 8).
        for (int y = part * 4 + wave; y < ho; y += parts * 4) {
            const uint8_t* r0 = src + s.offset + (int64_t)(2 * y) * s.pitch;
            const uint8_t* r1 = r0 + s.pitch;
            uint8_t* orow = dst + d.offset + (int64_t)y * d.pitch;
            for (int x4 = 4 * lane; x4 < wo; x4 += 256) {
                if (x4 + 4 <= wo) {
                    const uint2 a = *reinterpret_cast<const uint2*>(r0 + 2 * x4);
                    const uint2 b = *reinterpret_cast<const uint2*>(r1 + 2 * x4);
                    uint32_t o = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t wa = k < 2 ? a.x : a.y, wb = k < 2 ? b.x : b.y;
                        const int sh = 16 * (k & 1);
                        const uint32_t sum = ((wa >> sh) & 255u) + ((wa >> (sh + 8)) & 255u) +
                                             ((wb >> sh) & 255u) + ((wb >> (sh + 8)) & 255u);
                        o |= ((sum + 2u) >> 2) << (8 * k);
                    }
                    *reinterpret_cast<uint32_t*>(orow + x4) = o;
                } else {
                    for (int x = x4; x < wo; ++x) {
                        const uint32_t sum = r0[2 * x] + r0[2 * x + 1] + r1[2 * x] + r1[2 * x + 1];
                        orow[x] = (uint8_t)((sum + 2u) >> 2);
                    }
                }
            }
        }
        return;
    }
    // the output's columns in as many equal segments as keep a segment's
    // source columns (and four of alignment and an end) within the loads
    const int per = max(1, (int)((int64_t)(kFrontCols - 8) * wo / W));
    const int nseg = (wo + per - 1) / per, len = (wo + nseg - 1) / nseg;
    const int unit = part * kFrontWaves + wave, groups = parts * kFrontWaves / nseg;
    const int rows = (ho + groups - 1) / groups;
    const int x0 = unit % nseg * len, y0 = unit / nseg * rows;
    if (y0 >= ho || x0 >= wo) return;   // uniform over the wave; there are no barriers
    const int x1 = min(x0 + len, wo), y1 = min(y0 + rows, ho);
    // 2 N + W H < 511 W H: 32-bit arithmetic while that stays below 2^32
    const bool narrow = (uint64_t)W * (uint64_t)H * 511u < (1ull << 32);
    const int t0 = (W - 1) / wo;
#define CDVS_WALK(N, T) front_walk<N, T>(src, s, dst, d, x0, x1, y0, y1, V[wave], xp[wave], lane)
    if (!narrow) CDVS_WALK(false, 0);
    else if (t0 == 1) CDVS_WALK(true, 1);
    else if (t0 == 2) CDVS_WALK(true, 2);
    else if (t0 == 3) CDVS_WALK(true, 3);
    else CDVS_WALK(true, 0);
#undef CDVS_WALK
}

}  // namespace

hipError_t launch_front(const uint8_t* src, const cdvs_image_desc* sdesc, uint8_t* dst,
                        const cdvs_image_desc* ddesc, int n, int32_t* flags, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    // workgroups per image: 32 (128 waves, a few rows each) once the batch
    // fills the chip, up to one wave per output row below that
    const int parts = std::min(160, std::max(32, 2048 / n));
    hipLaunchKernelGGL(k_front, dim3((unsigned)n * parts), dim3(64 * kFrontWaves), 0, s, src, sdesc, dst, ddesc, n, parts,
                       flags);
    return hipGetLastError();
}

}  // namespace cdvs
