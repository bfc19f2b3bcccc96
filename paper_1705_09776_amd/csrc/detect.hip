// ALP keypoint detection on gfx950 (Sec. III-A, Eqs. (2)-(3); Sec. IV-A,
// Algorithm 1 stages A-C).
//
// k_detect_strip: one wave per strip of 60 columns by 6 to 48 rows of centres of
//   one (image, octave), all octaves of all images in one launch; the wave
//   streams the five Gaussian images down its strip in registers (details at
//   the kernel).  Per centre: scale-normalised 5-point Laplacians, the four
//   ALP coefficients, extremal scale, contrast test, strict 8-neighbour test
//   at that scale, one quadratic refinement step; survivors go to the image's
//   candidate list, those that a workgroup's strips have left at the end with
//   one atomic for each image.  With a cell mask (the learned gate) only the
//   centres of active cells are examined and strips without any are skipped
//   before loading anything.
// k_finalize: one workgroup per image.  (Images with more candidates than it
//   holds: their strongest kCandCap by |p|.)  Stage C (cross-octave
//   duplicates) over cells of the adjacent octaves, a counting sort over bins
//   of |p| for the canonical order (|p| descending, octave, iy, ix) of what can
//   be among the top k, and the copy-out.  It leaves the detection's counters
//   at zero for the next one.
#include <algorithm>

#include "cdvs_internal.h"

namespace cdvs {

namespace {

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return min(max(v, lo), hi); }

__device__ __forceinline__ float horner(const float4 a, float s) { return fmaf(fmaf(fmaf(a.w, s, a.z), s, a.y), s, a.x); }

// Extremal scale of p(s) = a.x + a.y s + a.z s^2 + a.w s^3 in [lo, hi) where
// |p| has a maximum (p p'' < 0); larger |p| wins, then the smaller s.  The
// roots of p'(s) = A s^2 + B s + C come from the stable quadratic formula,
// s0 = q / A and s1 = C / q; when A = 0, q = -B and s1 is the linear root.
// Both candidates are evaluated and the choice is made by selects (no
// branches: every lane of a wave runs this), with correctly rounded
// quotients (the extremal scale is ill-conditioned, so the quotients are
// not replaced by reciprocal approximations).
__device__ __forceinline__ bool alp_extremum(const float4 a, float lo, float hi, float& s_out, float& p_out,
                                             float& pss_out) {
    const float A = 3.f * a.w, B = 2.f * a.z, C = a.y;
    const bool lin = A == 0.f;
    const float disc = B * B - 4.f * A * C;
    const float sq = __builtin_amdgcn_sqrtf(fmaxf(disc, 0.f));   // hardware square root (1 ulp)
    const float q = (B >= 0.f) ? -(B + sq) * 0.5f : -(B - sq) * 0.5f;
    const float s0 = q / A;
    const float s1 = C / (lin ? -B : q);
    const bool real = lin || disc >= 0.f;
    const float p0 = horner(a, s0), p1 = horner(a, s1);
    const float pss0 = 6.f * a.w * s0 + 2.f * a.z, pss1 = 6.f * a.w * s1 + 2.f * a.z;
    const bool ok0 = real & !lin & (s0 >= lo) & (s0 < hi) & (p0 * pss0 < 0.f);
    const bool ok1 = real & (s1 >= lo) & (s1 < hi) & (p1 * pss1 < 0.f);
    const float a0 = fabsf(p0), a1 = fabsf(p1);
    const bool take1 = ok1 & (!ok0 | (a1 > a0) | ((a1 == a0) & (s1 < s0)));
    // without an extremum the outputs are left as they fall (possibly not
    // finite): they then only feed this centre's own tests, which it fails
    s_out = take1 ? s1 : s0;
    p_out = take1 ? p1 : p0;
    pss_out = take1 ? pss1 : pss0;
    return ok0 | ok1;
}

// 5-point Laplacian sum (up + down + left + right - 4 centre), in one fixed
// order of operations for the plain and the gated detection.
__device__ __forceinline__ float lap5(float c, float up, float dn, float lf, float rt) {
    float s = up + dn;
    s = s + lf;
    s = s + rt;
    s = s - 4.f * c;
    return s;
}

// Adds scale k's normalised Laplacian sigma_k^2 lap to the ALP coefficients
// (sigma_k^2 is folded into the fitting weights on the host).
__device__ __forceinline__ void alpha_acc(float4& a, float lap, int k, const DetParams& dp) {
    a.x = fmaf(dp.bsig[k][0], lap, a.x);
    a.y = fmaf(dp.bsig[k][1], lap, a.y);
    a.z = fmaf(dp.bsig[k][2], lap, a.z);
    a.w = fmaf(dp.bsig[k][3], lap, a.w);
}

struct Cand {
    float s, p, pss, ox, oy, pr, rho;
};

// Strict extremum of the centre value p = v[4] against the eight
// neighbours' cubics v[] evaluated at the centre's scale (Algorithm 1 stage A).
// (All eight below p for a maximum, above it for a minimum: compared through
// their max and min, without branches; mn > p is tested as -mn < -p = |p|,
// so one float select and one comparison decide both cases exactly; the
// values are finite.)
__device__ __forceinline__ bool strict_extremum(const float (&v)[9], float p) {
    float mx = v[0], mn = v[0];
#pragma unroll
    for (int i = 1; i < 9; ++i)
        if (i != 4) {
            mx = fmaxf(mx, v[i]);
            mn = fminf(mn, v[i]);
        }
    return (p > 0.f ? mx : -mn) < fabsf(p);
}

// One quadratic refinement step on the 3x3 values v[] (row-major, centre
// v[4] = p): offset, edge test and interpolated response (Algorithm 1 stage B).
__device__ __forceinline__ bool refine_v(const float (&v)[9], float s, float p, float pss, const DetParams& dp,
                                         Cand& o) {
    const float c = v[4];
    const float gxd = (v[5] - v[3]) * 0.5f;
    const float gyd = (v[7] - v[1]) * 0.5f;
    const float hxx = v[5] - 2.f * c + v[3];
    const float hyy = v[7] - 2.f * c + v[1];
    const float hxy = (v[8] - v[6] - v[2] + v[0]) * 0.25f;
    const float det = hxx * hyy - hxy * hxy;
    if (!(det > 0.f)) return false;
    const float tr = hxx + hyy;
    const float ratio = __fdividef(tr * tr, det);
    if (!(ratio < dp.edge_lim)) return false;
    const float rdet = 1.f / det;
    const float dx = -(hyy * gxd - hxy * gyd) * rdet;
    const float dy = -(hxx * gyd - hxy * gxd) * rdet;
    if (fabsf(dx) > dp.max_off || fabsf(dy) > dp.max_off) return false;
    o.s = s;
    o.p = p;
    o.pss = pss;
    o.ox = dx;
    o.oy = dy;
    o.pr = c + (gxd * dx + gyd * dy) * 0.5f;
    o.rho = ratio;
    return true;
}

// A centre that came through the refinement (keep) or not.
struct Refined {
    Cand c;
    int gx, gy;
    bool keep;
};

// A survivor's record, at a slot of its image's candidates.
__device__ __forceinline__ void store_candidate(const Refined& v, int slot, const DetTile& job, const DetOut& out) {
    if (slot >= job.cand_cap) {
        atomicOr(out.flags, kFlagCandOverflow);
        return;
    }
    const float scale = (float)(1 << job.octave);
    cdvs_keypoint r;
    r.x = ((float)v.gx + v.c.ox) * scale;
    r.y = ((float)v.gy + v.c.oy) * scale;
    r.sigma = v.c.s * scale;
    r.p = v.c.pr;
    r.theta = 0.f;
    r.rho = v.c.rho;
    r.p_ss = v.c.pss;
    r.peak = 0.f;
    r.image = job.image;
    r.octave = job.octave;
    r.ix = v.gx;
    r.iy = v.gy;
    const int64_t at = (int64_t)job.cand_blk * kCandBlock + slot;
    out.cand[at] = r;
    if (out.absp) out.absp[at] = fabsf(v.c.pr);
}

// Wave-level compaction of survivors into the image's candidate list: one
// ballot and one atomic per wave.  Every lane of the wave must call it.
__device__ __forceinline__ void emit(const Refined& v, const DetTile& job, const DetOut& out) {
    const int lane = threadIdx.x & 63;
    const uint64_t m = __ballot(v.keep);
    if (!m) return;
    const int leader = __ffsll((unsigned long long)m) - 1;
    int base = 0;
    if (lane == leader) base = atomicAdd(&out.cnt[job.image * kCntStride], __popcll(m));
    base = __shfl(base, leader);
    if (v.keep) store_candidate(v, base + __popcll(m & ((1ull << lane) - 1ull)), job, out);
}

// ---------------------------------------------------------------------------
// k_detect_strip: the detection, one wave per strip of kStripW
// centre columns x strip_h centre rows of one (image, octave) inside the
// detection border; lane l holds image column x0 - 2 + l (lanes 0, 1, 62
// and 63 are halo).  The wave walks down its strip one row at a time with
// no LDS staging and no barriers: each row's five plane values arrive by one
// coalesced dword load per plane, issued a chunk of rows ahead; the
// Laplacians take their horizontal neighbours from the adjacent lanes (DPP
// wave shifts) and their vertical ones from the previous two rows held in
// registers, and the ALP coefficients of the last three rows stay in
// registers for the centre tests.  For the strict 3x3 test each lane
// evaluates its own column's cubics at its neighbours' scales and hands the
// values over, so no lane needs another lane's coefficients.  Centres that
// pass are queued in the wave's LDS list with their 3x3 values and refined
// in passes of up to 64 once more than 36 are waiting (dense lanes; one
// global atomic per pass).
constexpr int kStripW = kDetStripW;
constexpr int kQCap = 96;              // flushed above 36, and one row adds at most 60
constexpr int kQFlush = kQCap - 60;
constexpr int kQFields = 12;           // the eight neighbour values, s, p, pss, (x | y << 16)

__device__ __forceinline__ float lane_from_left(float v) {   // lane l gets lane l-1's value (lane 0: 0)
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_from_right(float v) {  // lane l gets lane l+1's value (lane 63: 0)
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}

struct StripRow {
    float g[kScales];
};

// The five planes of a strip's (image, octave): their bases are the same in
// every lane and kept in scalar registers, and a lane reads a row as one
// 32-bit byte offset from each (an octave's planes span less than 2^32
// bytes, as sides are at most CDVS_MAX_SIDE), so a row costs one vector add
// for its address instead of a 64-bit address per plane.
struct StripPlanes {
    const char* base[kScales];
    uint32_t col4;   // this lane's (clamped) column, in bytes
};

__device__ __forceinline__ StripPlanes strip_planes(const float* __restrict__ pyr, const DetTile& job, int gx) {
    StripPlanes sp;
    // (the offset, not the pointer, goes through the scalar unit: a pointer
    // rebuilt from an integer would lose its global address space)
#pragma unroll
    for (int k = 0; k < kScales; ++k) {
        const uint64_t o = (uint64_t)(job.plane0 + (int64_t)k * job.plane_stride);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)o);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(o >> 32));
        sp.base[k] = reinterpret_cast<const char*>(pyr + (int64_t)(((uint64_t)hi << 32) | lo));
    }
    sp.col4 = (uint32_t)clampi(gx, 0, job.w - 1) * 4u;
    return sp;
}

// Plane row y (clamped to the image) of this lane's column.
__device__ __forceinline__ void load_row(const StripPlanes& sp, const DetTile& job, int y, StripRow& r) {
    const uint32_t off = (uint32_t)clampi(y, 0, job.h - 1) * (uint32_t)job.pitch * 4u + sp.col4;
#pragma unroll
    for (int k = 0; k < kScales; ++k) r.g[k] = *reinterpret_cast<const float*>(sp.base[k] + off);
}

// ALP coefficients of the middle row from three consecutive rows.
__device__ __forceinline__ float4 strip_alpha(const StripRow& u, const StripRow& m, const StripRow& d,
                                              const DetParams& dp) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < kScales; ++k)
        alpha_acc(a, lap5(m.g[k], u.g[k], d.g[k], lane_from_left(m.g[k]), lane_from_right(m.g[k])), k, dp);
    return a;
}

// The refinement of this lane's queued centre, base + lane, of n in all.
__device__ __forceinline__ Refined strip_refine(float (*q)[kQCap], int base, int n, const DetParams& dp) {
    Refined r{};
    const int e = base + (threadIdx.x & 63);
    if (e < n) {
        float v[9];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = q[i][e];
        v[4] = q[9][e];   // the centre: p
#pragma unroll
        for (int i = 5; i < 9; ++i) v[i] = q[i - 1][e];
        const int xy = __float_as_int(q[11][e]);
        r.gx = xy & 0xffff;
        r.gy = xy >> 16;
        r.keep = refine_v(v, q[8][e], q[9][e], q[10][e], dp, r.c);
    }
    return r;
}

// Refines everything queued (in passes of 64), appends the survivors to the
// image's candidates and empties the queue.  Every lane of the wave calls it.
__device__ __forceinline__ void strip_drain(float (*q)[kQCap], int& qn, const DetTile& job, const DetParams& dp,
                                            const DetOut& out) {
    for (int base = 0; base < qn; base += 64) emit(strip_refine(q, base, qn, dp), job, out);
    qn = 0;
}

// What the four strips of a workgroup have left in their queues, appended
// with one atomic for all those of one image (a large image's strips would
// otherwise queue up at its counter: 5,600 additions of 7 ns for 4000x3000
// pixels).  Every lane of the workgroup calls it.
__device__ __forceinline__ void workgroup_drain(float (*q)[kQCap], int qn, const DetTile& job, const DetParams& dp,
                                                const DetOut& out) {
    __shared__ int cnt_s[4], img_s[4], base_s[4];
    static_assert(kQFlush <= 64, "one pass: a strip leaves no more than that");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const Refined r = strip_refine(q, 0, qn, dp);
    const uint64_t m = __ballot(r.keep);
    if (lane == 0) {
        cnt_s[wave] = __popcll(m);
        img_s[wave] = job.image;
    }
    __syncthreads();
    if (lane == 0 && (wave == 0 || img_s[wave - 1] != job.image)) {
        // the first wave of an image's run (strips are image by image)
        int sum = 0;
        for (int w = wave; w < 4 && img_s[w] == job.image; ++w) sum += cnt_s[w];
        base_s[wave] = sum ? atomicAdd(&out.cnt[job.image * kCntStride], sum) : 0;
    }
    __syncthreads();
    int before = 0, first = wave;
    while (first > 0 && img_s[first - 1] == job.image) before += cnt_s[--first];
    if (r.keep) store_candidate(r, base_s[first] + before + __popcll(m & ((1ull << lane) - 1ull)), job, out);
}

// Centre tests of one row y from the coefficients of rows y-1, y, y+1;
// strict extrema are queued (qn: the wave's queue length, uniform).
__device__ __forceinline__ void strip_centres(const float4& aU, const float4& aM, const float4& aD, bool col_ok, int gx,
                                              int y, float (*q)[kQCap], int& qn, const DetTile& job,
                                              const DetParams& dp, const DetOut& out) {
    float s = 0.f, p = 0.f, pss = 0.f;
    const bool found = alp_extremum(aM, dp.lo, dp.hi, s, p, pss);
    const bool pass = col_ok & found & (fabsf(p) >= dp.contrast);   // no branch: every lane evaluates
    if (!__ballot(pass)) return;   // uniform over the wave
    // this lane's column at the scale of the centre to its right (for which
    // it is the left column) and of the centre to its left
    const float s_r = lane_from_right(s), s_l = lane_from_left(s);
    const float l0 = horner(aU, s_r), l1 = horner(aM, s_r), l2 = horner(aD, s_r);
    const float r0 = horner(aU, s_l), r1 = horner(aM, s_l), r2 = horner(aD, s_l);
    float v[9];
    v[0] = lane_from_left(l0);
    v[3] = lane_from_left(l1);
    v[6] = lane_from_left(l2);
    v[2] = lane_from_right(r0);
    v[5] = lane_from_right(r1);
    v[8] = lane_from_right(r2);
    v[1] = horner(aU, s);
    v[4] = p;
    v[7] = horner(aD, s);
    const bool keep = pass & strict_extremum(v, p);   // both evaluated: no branch
    const uint64_t m = __ballot(keep);
    if (!m) return;
    const int lane = threadIdx.x & 63;
    if (keep) {
        const int i = qn + __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
        for (int f = 0; f < 4; ++f) q[f][i] = v[f];
#pragma unroll
        for (int f = 5; f < 9; ++f) q[f - 1][i] = v[f];
        q[8][i] = s;
        q[9][i] = p;
        q[10][i] = pss;
        q[11][i] = __int_as_float(gx | (y << 16));
    }
    qn += __popcll(m);
    if (qn > kQFlush) strip_drain(q, qn, job, dp, out);
}

// GATED: an octave-o centre (x, y) is examined only when bit o of the mask
// cell holding (x 2^o, y 2^o) / 4 is set, unless more than gate.fmax of the
// image's cells have bit o set, or o is beyond the gate's kCnnHeads bits
// (then the octave is examined densely).
// Returns how many strict extrema are left in the wave's queue.
template <bool GATED>
__device__ __forceinline__ int detect_strip(const float* __restrict__ pyr, const DetTile& job, int strip_h,
                                             const DetParams& dp,
                                             const GateParams& gate, float (*q)[kQCap], const DetOut& out) {
    static_assert(kDetStripH <= 64, "one activity bit per strip row");
    const int lane = threadIdx.x & 63;
    const int x0 = job.tx0, y0 = job.ty0;
    const int xend = min(x0 + kStripW, job.w - dp.border), yend = min(y0 + strip_h, job.h - dp.border);
    const int gx = x0 - 2 + lane;
    const bool col_ok = lane >= 2 && gx < xend;
    // bit i: this lane's centre on row y0 + i is examined
    uint64_t rows_on = ~0ull;
    if constexpr (GATED) {
        const CnnImage cg = gate.cells[job.image];
        const bool dense =
            job.octave >= kCnnHeads ||
            (float)gate.active[job.image * kMaxOctaves + job.octave] > gate.fmax * (float)(cg.H4 * cg.W4);
        if (!dense) {
            rows_on = 0ull;
            if (col_ok) {
                const uint8_t* m = gate.mask + cg.cell0 + min((gx << job.octave) >> 2, cg.W4 - 1);
                // rows of one cell row share its byte: one load for the 4, 2
                // or 1 rows of a cell, several on the way at a time (against
                // a load per row: 128 gated images 836 -> 824 us, 40 of them
                // 344 -> 337)
                const int per = job.octave < 2 ? 4 >> job.octave : 1;
                const uint32_t run = (1u << per) - 1u;
#pragma unroll 4
                for (int y = y0 - y0 % per; y < yend; y += per) {
                    const int cy = min((y << job.octave) >> 2, cg.H4 - 1);
                    const uint32_t bit = (m[(int64_t)cy * cg.W4] >> job.octave) & 1u;
                    const uint64_t rows = bit ? run : 0u;
                    rows_on |= y < y0 ? rows >> (y0 - y) : rows << (y - y0);
                }
                rows_on &= (1ull << (yend - y0)) - 1ull;   // (the last cell's rows past the strip; at most 48 rows)
            }
            if (!__ballot(rows_on != 0ull)) return 0;   // nothing active: the strip is not even loaded
        }
    }
    const StripPlanes col = strip_planes(pyr, job, gx);
    // Plane rows live in a ring of kRing slots, row y in slot (y - y0 + 2) %
    // kRing, and coefficient rows in a ring of three, row y in slot
    // (y - y0 + 1) % 3.  Centre row y computes the coefficients of row y+1,
    // which frees plane row y's slot for row y + kRing, loaded right away and
    // first needed four rows later.  Loads past the strip's last plane row
    // re-read that row (clamped; every load is unconditional, so the waits
    // for them are exact).
    constexpr int kRing = 6;
    const int last = yend + 1;
    StripRow g[kRing], t0, t1;
    load_row(col, job, y0 - 2, t0);
    load_row(col, job, y0 - 1, t1);
#pragma unroll
    for (int r = 2; r < kRing + 2; ++r) load_row(col, job, min(y0 - 2 + r, last), g[r % kRing]);
    float4 a[3];
    a[0] = strip_alpha(t0, t1, g[2], dp);     // row y0-1
    a[1] = strip_alpha(t1, g[2], g[3], dp);   // row y0
    int qn = 0;
    for (int y = y0; y < yend; y += kRing) {
#pragma unroll
        for (int r = 0; r < kRing; ++r) {
            a[(r + 2) % 3] = strip_alpha(g[(r + 2) % kRing], g[(r + 3) % kRing], g[(r + 4) % kRing], dp);
            load_row(col, job, min(y + r + kRing, last), g[(r + 2) % kRing]);
            if (y + r < yend)   // uniform over the wave
                strip_centres(a[r % 3], a[(r + 1) % 3], a[(r + 2) % 3], col_ok && ((rows_on >> (y + r - y0)) & 1ull),
                              gx, y + r, q, qn, job, dp, out);
        }
    }
    return qn;
}

// Requests one strip index from this XCD's work counter; the value arrives
// in lane 0 and is read (made uniform) only when it is needed.  (An
// increment rather than an add: the compiler rewrites a single-lane add into
// a wave-wide one whose result it consumes at once, stalling on the round
// trip; the counter never comes near the wrap limit.)
__device__ __forceinline__ int fetch_strip(int32_t* __restrict__ ctr) {
    unsigned t = 0u;
    if ((threadIdx.x & 63) == 0) t = atomicInc(reinterpret_cast<unsigned*>(ctr), 0xffffffffu);
    return (int)t;
}

// Two launch forms (picked by the autotuner):
// PERSISTENT = false: one wave per strip, the hardware dispatching the
//   workgroups (xcd_remap gives each XCD one contiguous range of strips).
// PERSISTENT = true: the grid (a multiple of 8, sized to the waves the chip
//   holds) is split evenly over the XCDs, and every XCD owns one contiguous
//   range of strips with a work counter in `work` (zeroed before the
//   launch); each wave pulls its next strip from the counter until the range
//   is used up, so uneven strips (octaves, ragged images, skipped gated
//   strips) balance by themselves.  The next index is requested when a
//   strip starts and read when it ends, so the atomic's round trip overlaps
//   the strip's work.
// Either way neighbouring strips run close together in time on one XCD and
// share their halo rows through its L2.
template <bool GATED, bool PERSISTENT>
__global__ __launch_bounds__(256) void k_detect_strip(const float* __restrict__ pyr, const DetTile* __restrict__ strips,
                                                      int nstrips, int strip_h, DetParams dp, GateParams gate,
                                                      int32_t* __restrict__ work, DetOut out) {
    __shared__ float queue[4][kQFields][kQCap];
    const int wave = threadIdx.x >> 6;
    if constexpr (!PERSISTENT) {
        const int sidx = __builtin_amdgcn_readfirstlane(xcd_remap(blockIdx.x, gridDim.x) * 4 + wave);
        const DetTile job = strips[min(sidx, nstrips - 1)];
        const int qn = sidx < nstrips ? detect_strip<GATED>(pyr, job, strip_h, dp, gate, queue[wave], out) : 0;
        workgroup_drain(queue[wave], qn, job, dp, out);   // (the only barriers)
    } else {
        const int x = blockIdx.x % kXcds;
        const int per = nstrips / kXcds, rem = nstrips % kXcds;
        const int base = x * per + min(x, rem), cnt = per + (x < rem ? 1 : 0);
        int32_t* ctr = work + x * kCntStride;
        int pending = fetch_strip(ctr);
        for (;;) {
            const int t = __builtin_amdgcn_readfirstlane(pending);
            if (t >= cnt) break;   // uniform over the wave; there are no barriers
            pending = fetch_strip(ctr);
            const DetTile job = strips[base + t];
            int qn = detect_strip<GATED>(pyr, job, strip_h, dp, gate, queue[wave], out);
            strip_drain(queue[wave], qn, job, dp, out);
        }
    }
}

__global__ void k_clear(int32_t* p, int n, int stride) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[(int64_t)i * stride] = 0;
}

constexpr int FIN_THREADS = 1024;
constexpr int FIN_PER = kCandCap / FIN_THREADS;  // candidates per thread

// One compare-exchange of a bitonic stage of block size `size` at distance
// S < 64 for the (key, payload) of element i held by this lane, whose
// partner (i ^ S) is in lane ^ S: the lower index keeps the smaller key in
// an ascending block, the larger in a descending one (equal keys stay where
// they are).  Both comparisons are made and one is selected, so no lane
// branches.
template <int S>
__device__ __forceinline__ void bitonic_lane_step(unsigned long long& k, int& p, int i, int size) {
    const unsigned long long o = lane_xor64<S>(k);
    const int op = (int)lane_xor<S>((uint32_t)p);
    const bool want_min = ((i & size) == 0) == ((i & S) == 0);
    const bool lt = o < k, gt = k < o;
    const bool take = (want_min & lt) | (!want_min & gt);
    k = take ? o : k;
    p = take ? op : p;
}

// The distances 32, 16, .., 1 (those below `size`) of one bitonic stage
// for both of the lane's elements.
__device__ __forceinline__ void bitonic_lane_steps(unsigned long long& k0, int& p0, int i0, unsigned long long& k1,
                                                   int& p1, int i1, int size) {
#define CDVS_STEP(S)                                   \
    if (size > S) {                                    \
        bitonic_lane_step<S>(k0, p0, i0, size);        \
        bitonic_lane_step<S>(k1, p1, i1, size);        \
    }
    CDVS_STEP(32) CDVS_STEP(16) CDVS_STEP(8) CDVS_STEP(4) CDVS_STEP(2) CDVS_STEP(1)
#undef CDVS_STEP
}

// The steps at distances below 128 of bitonic block sizes first..last on
// the 128-entry chunks of [0, npow): each wave takes whole chunks, two
// entries per lane (c*128 + lane and c*128 + 64 + lane) in registers.
__device__ __forceinline__ void bitonic_chunk_steps(unsigned long long* key, unsigned short* idx, int npow, int first,
                                                    int last) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int c = wave; c < npow / 128; c += nw) {
        const int i0 = 128 * c + lane, i1 = i0 + 64;
        unsigned long long k0 = key[i0], k1 = key[i1];
        int p0 = idx[i0], p1 = idx[i1];
        for (int size = first; size <= last; size <<= 1) {
            if (size >= 128) {   // distance 64: the lane's own pair, one direction for both
                const bool asc = (i0 & size) == 0;
                if (asc ? (k0 > k1) : (k0 < k1)) {
                    const unsigned long long tk = k0;
                    k0 = k1;
                    k1 = tk;
                    const int tp = p0;
                    p0 = p1;
                    p1 = tp;
                }
            }
            bitonic_lane_steps(k0, p0, i0, k1, p1, i1, size);
        }
        key[i0] = k0;
        key[i1] = k1;
        idx[i0] = (unsigned short)p0;
        idx[i1] = (unsigned short)p1;
    }
}

// Ascending bitonic sort of npow (a power of two, at least 128) 64-bit keys
// with 16-bit payloads in LDS by the whole workgroup: block sizes up to 128
// entirely in registers (lane shuffles), then for each larger size its
// distances of 128 and more through LDS with a barrier each, the rest in
// registers.
__device__ void bitonic_sort(unsigned long long* key, unsigned short* idx, int npow) {
    bitonic_chunk_steps(key, idx, npow, 2, 128);
    __syncthreads();
    for (int size = 256; size <= npow; size <<= 1) {
        for (int stride = size >> 1; stride >= 128; stride >>= 1) {
            for (int t = threadIdx.x; t < npow / 2; t += blockDim.x) {
                const int lo = 2 * t - (t & (stride - 1));
                const int hi = lo + stride;
                const bool asc = (lo & size) == 0;
                const unsigned long long kl = key[lo], kh = key[hi];
                if ((kl > kh) == asc) {
                    key[lo] = kh;
                    key[hi] = kl;
                    const unsigned short il = idx[lo];
                    idx[lo] = idx[hi];
                    idx[hi] = il;
                }
            }
            __syncthreads();
        }
        bitonic_chunk_steps(key, idx, npow, size, size);
        __syncthreads();
    }
}

// Exclusive prefix sums of v[0 .. 4 * FIN_THREADS) in place, and the total,
// by the whole workgroup.
__device__ __forceinline__ int scan4(int* v, int* wsum) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int4 q = reinterpret_cast<int4*>(v)[tid];
    const int sum = q.x + q.y + q.z + q.w;
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(incl, off);
        if (lane >= off) incl += u;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < FIN_THREADS / 64; ++w) {
        const int u = wsum[w];
        before += w < wave ? u : 0;
        total += u;
    }
    const int e = before + incl - sum;
    reinterpret_cast<int4*>(v)[tid] = make_int4(e, e + q.x, e + q.x + q.y, e + q.x + q.y + q.z);
    __syncthreads();
    return total;
}

// Where the count of keys, taken from the highest bin of hist[0 .. 4096)
// down, reaches `need` (1 <= need <= the keys in hist): that bin, and how
// many of its keys the count still needs.
__device__ __forceinline__ void nth_from_top(int* hist, int* wsum, int need, int* bin, int* rest) {
    const int tid = threadIdx.x;
    const int4 q = reinterpret_cast<int4*>(hist)[tid];
    const int total = scan4(hist, wsum);
    const int4 e = reinterpret_cast<int4*>(hist)[tid];
    const int cnt[4] = {q.x, q.y, q.z, q.w}, ex[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int above = total - ex[k] - cnt[k];   // keys in higher bins
        if (above < need && above + cnt[k] >= need) {   // one bin of all
            *bin = 4 * tid + k;
            *rest = need - above;
        }
    }
    __syncthreads();
}

// Minimum and maximum over the wave of unsigned values, in every lane.
__device__ __forceinline__ void wave_min_max(uint32_t& lo, uint32_t& hi) {
#define CDVS_STEP(S)                 \
    lo = min(lo, lane_xor<S>(lo));   \
    hi = max(hi, lane_xor<S>(hi));
    CDVS_STEP(1) CDVS_STEP(2) CDVS_STEP(4) CDVS_STEP(8) CDVS_STEP(16) CDVS_STEP(32)
#undef CDVS_STEP
}

// The kCandCap strongest by |p| of an image's n > kCandCap candidates, as
// indices in list[] (in no particular order): the kCandCap-th largest |p| by
// a radix select on its float bits (non-negative floats order like their
// bits), over the range they span so that the first round's counts spread,
// then every candidate above it and enough of those equal to it.
__device__ __forceinline__ void strongest(const float* __restrict__ absp, int n, int* hist, int* wsum, int* tmp,
                                          uint32_t* lohi, uint32_t* __restrict__ list) {
    const int tid = threadIdx.x;
    // four keys at a time (an image's candidates start on, and its capacity
    // is, a multiple of 256; what lies past n is skipped)
    auto each = [&](auto&& f) {
#pragma unroll 4
        for (int i = 4 * tid; i < n; i += 4 * FIN_THREADS) {
            const uint4 k = *reinterpret_cast<const uint4*>(absp + i);
            f(i, k.x, true);
            f(i + 1, k.y, i + 1 < n);
            f(i + 2, k.z, i + 2 < n);
            f(i + 3, k.w, i + 3 < n);
        }
    };
    uint32_t lo = 0xffffffffu, hi = 0u;
    each([&](int, uint32_t key, bool in) {
        lo = in ? min(lo, key) : lo;
        hi = in ? max(hi, key) : hi;
    });
    wave_min_max(lo, hi);
    if ((tid & 63) == 0) {
        atomicMin(&lohi[0], lo);
        atomicMax(&lohi[1], hi);
    }
    __syncthreads();
    lo = lohi[0];
    // keys are taken from lo; the top bits found so far are prefix, at shift sh
    const uint32_t range = lohi[1] - lo;
    int need = kCandCap, sh = 32 - __clz((int)range | 1), width = 0;
    uint32_t prefix = 0u;
#pragma unroll 1
    do {
        reinterpret_cast<int4*>(hist)[tid] = make_int4(0, 0, 0, 0);
        __syncthreads();
        width = min(sh, 12);
        const int up = sh;
        sh -= width;
        each([&](int, uint32_t bits, bool in) {
            const uint32_t key = bits - lo;
            if (in && (up > 31 || key >> up == prefix)) atomicAdd(&hist[(key >> sh) & ((1u << width) - 1u)], 1);
        });
        __syncthreads();
        nth_from_top(hist, wsum, need, &tmp[0], &tmp[1]);
        prefix = (prefix << width) | (uint32_t)tmp[0];
        need = tmp[1];   // keys still needed from the threshold's bin
        __syncthreads();
    } while (sh > 0);
    prefix += lo;
    if (tid < 2) tmp[tid] = 0;
    __syncthreads();
    const int lane = tid & 63;
    for (int i0 = 0; i0 < n; i0 += 4 * FIN_THREADS) {   // the same for every lane: they count together
        const int i = i0 + 4 * tid;
        uint4 k = make_uint4(0u, 0u, 0u, 0u);
        if (i < n) k = *reinterpret_cast<const uint4*>(absp + i);
        const uint32_t key[4] = {k.x, k.y, k.z, k.w};
        bool take[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            take[q] = i + q < n && key[q] > prefix;
            if (i + q < n && key[q] == prefix) take[q] = atomicAdd(&tmp[1], 1) < need;
        }
        int before = 0, all = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint64_t m = __ballot(take[q]);
            before += __popcll(m & ((1ull << lane) - 1ull));
            all += __popcll(m);
        }
        int base = 0;
        if (lane == 0 && all) base = atomicAdd(&tmp[0], all);
        base = __shfl(base, 0) + before;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (take[q]) list[base++] = (uint32_t)(i + q);
    }
    __threadfence_block();
    __syncthreads();
}

// Stage C + canonical order + top-k for one image per workgroup.
//
// The candidates of every octave but the first are binned into square cells
// (a counting sort in LDS over at most kFinCells cells; of 8 octave pixels, in
// large images more in the finer octaves), so that each candidate meets only
// the few of the next octave in the cells around it; the decisions are those
// of all pairs, as only pairs farther apart than the distance limit are
// skipped.  The
// survivors are put in canonical order by a counting sort as well, over 4096
// bins of their range of |p|, which leaves few in any one bin; an image with
// more than kFinCrowd in one that it keeps from is sorted in full.
//
// One workgroup per image is latency-bound whatever the image: the kernel is
// a chain of passes with a barrier each.  With two bitonic sorts of every
// candidate (the first to find the neighbours by binary search, in both
// adjacent octaves) it took 47 us for one 640x480 image (1262 candidates) and
// 199 us for 8192 candidates, beside 231 us of a kernel of its own that cut
// 38,600 candidates to their 8192 strongest (its threshold found by one lane
// walking the bins); now 13 us, and 63 us with the cut.
constexpr int kFinCells = 4 * FIN_THREADS;
constexpr int kFinCrowd = 32;
static_assert(kFinCells <= 1 << 12 && kCandCap <= 1 << 19, "a cell and a place in one word");
static_assert(kCandCap == 8 * FIN_THREADS, "8 flags per lane");

__global__ __launch_bounds__(FIN_THREADS) void k_finalize(const cdvs_keypoint* __restrict__ cand,
                                                          const float* __restrict__ absp,
                                                          int32_t* __restrict__ cand_cnt,
                                                          const int64_t* __restrict__ cand_off,
                                                          const int32_t* __restrict__ cand_capv,
                                                          int32_t* __restrict__ active, uint32_t* __restrict__ lists,
                                                          const int32_t* __restrict__ wh, float ratio_lim, int topk,
                                                          int kp_cap, cdvs_keypoint* __restrict__ kp,
                                                          int32_t* __restrict__ count,
                                                          int32_t* __restrict__ flags) {
    // 128 KB: the records (x, y, sigma, p) by cell, then the keys and
    // payloads of the sort
    __shared__ float4 rec[kCandCap];
    __shared__ __align__(16) int cell[kFinCells + 4];   // counts, then first positions; then the |p| histogram
    __shared__ int wsum[FIN_THREADS / 64];
    // an octave's first cell, cells per row and cell side (log2)
    __shared__ int obase[kMaxOctaves], ocx[kMaxOctaves], oshift[kMaxOctaves];
    __shared__ int tmp[4];
    __shared__ uint32_t min_all, lohi[2];               // smallest |p| of a reduced image; range of |p| of the survivors
    __shared__ int n_alive, crowded;
    __shared__ __align__(16) uint8_t dead[kCandCap];   // by position: lost to a finer candidate
    unsigned long long* key = reinterpret_cast<unsigned long long*>(rec);
    unsigned short* idx = reinterpret_cast<unsigned short*>(key + kCandCap);

    const int img = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int n_all = min(cand_cnt[img * kCntStride], cand_capv[img]);
    const cdvs_keypoint* c = cand + cand_off[img];
    const int W = wh[2 * img], H = wh[2 * img + 1];
    const int n = min(n_all, kCandCap);
    // an image with more candidates than the LDS holds is reduced to its
    // kCandCap strongest (exactly the ones stage C and the top-k can keep: a
    // candidate only ever loses to a stronger one)
    const uint32_t* list = nullptr;
    if (n_all > kCandCap) {   // uniform over the workgroup
        uint32_t* l = lists + (int64_t)img * kCandCap;
        if (tid == 0) {
            lohi[0] = 0xffffffffu;
            lohi[1] = 0u;
        }
        __syncthreads();
        strongest(absp + cand_off[img], n_all, cell, wsum, tmp, lohi, l);
        list = l;
    }
    reinterpret_cast<int4*>(cell)[tid] = make_int4(0, 0, 0, 0);
    reinterpret_cast<uint2*>(dead)[tid] = make_uint2(0u, 0u);
    if (tid == 0) {
        min_all = lohi[0] = 0xffffffffu;
        lohi[1] = 0u;
        n_alive = crowded = 0;
    }
    if (tid < 64) {
        // lane o: octave o's size (halved rounding up), and the smallest cells
        // with which all octaves' fit
        const int o = min(lane, kMaxOctaves - 1);
        const int w = (W + (1 << o) - 1) >> o, h = (H + (1 << o) - 1) >> o;
        int s = 3, sh, total, incl, cells;
        do {
            ++s;
            sh = max(3, s - o);
            cells = lane > 0 && lane < kMaxOctaves ? (((w - 1) >> sh) + 1) * (((h - 1) >> sh) + 1) : 0;
            incl = cells;
#pragma unroll
            for (int off = 1; off < kMaxOctaves; off <<= 1) {
                const int u = __shfl_up(incl, off);
                if (lane >= off) incl += u;
            }
            total = __shfl(incl, kMaxOctaves - 1);
        } while (total > kFinCells);
        if (lane < kMaxOctaves) {
            obase[lane] = incl - cells;
            ocx[lane] = ((w - 1) >> sh) + 1;
            oshift[lane] = sh;
        }
    }
    // this thread's candidates: position, scale and response, and the low
    // word of the canonical key (octave, iy, ix)
    float4 a[FIN_PER];
    uint32_t low[FIN_PER], src[FIN_PER];
    // (all indices first, then all records, so that each is one round trip;
    // lanes past the end read the last one again)
#pragma unroll
    for (int j = 0; j < FIN_PER; ++j)
        if (j * FIN_THREADS < n) {
            const int i = min(tid + j * FIN_THREADS, n - 1);
            src[j] = list ? list[i] : (uint32_t)i;
        }
#pragma unroll
    for (int j = 0; j < FIN_PER; ++j)
        if (j * FIN_THREADS < n) {
            const uint4* r = reinterpret_cast<const uint4*>(c + src[j]);
            const uint4 q = r[0], t = r[2];
            a[j] = make_float4(__uint_as_float(q.x), __uint_as_float(q.y), __uint_as_float(q.z), __uint_as_float(q.w));
            low[j] = (t.y << 28) | (t.w << 14) | t.z;
        }
    __syncthreads();
    // the cell, along one axis, of base-image coordinate v in an octave of
    // the given side (beyond the image: the outermost)
    auto cell_of = [&](float v, int o, int side) {
        return min(max((int)floorf(__builtin_amdgcn_ldexpf(v, -o)), 0), ((side + (1 << o) - 1) >> o) - 1) >> oshift[o];
    };
    int at[FIN_PER];   // the cell, and the place in it
    uint32_t my_min = 0xffffffffu;
#pragma unroll
    for (int j = 0; j < FIN_PER; ++j) {
        if (tid + j * FIN_THREADS < n) {
            const int o = (int)(low[j] >> 28);
            if (o > 0) {
                at[j] = obase[o] + cell_of(a[j].y, o, H) * ocx[o] + cell_of(a[j].x, o, W);
                at[j] |= atomicAdd(&cell[at[j]], 1) << 12;
            }
            my_min = min(my_min, __float_as_uint(fabsf(a[j].w)));
        }
    }
    if (list) {
        uint32_t hi = 0u;
        wave_min_max(my_min, hi);
        if (lane == 0) atomicMin(&min_all, my_min);
    }
    __syncthreads();
    const int binned = scan4(cell, wsum);
    if (tid == 0) cell[kFinCells] = binned;
#pragma unroll
    for (int j = 0; j < FIN_PER; ++j)
        if (tid + j * FIN_THREADS < n && low[j] >> 28 != 0u) rec[cell[at[j] & (kFinCells - 1)] + (at[j] >> 12)] = a[j];
    __syncthreads();

    // Stage C: each candidate meets those of the next coarser octave, and of
    // two that are duplicates the weaker one is out (equal: the coarser)
    uint32_t out = 0u;   // bit j: candidate j is
#pragma unroll
    for (int j = 0; j < FIN_PER; ++j) {
        const int ao = (int)(low[j] >> 28), o2 = ao + 1;
        if (tid + j * FIN_THREADS < n && o2 < kMaxOctaves) {
            const float aa = fabsf(a[j].w);
            const float lim = (float)(1 << o2);
            const float lim2 = lim * lim;
            // the cells searched are those of a square one pixel wider than
            // the limit, so rounding here cannot drop a pair the exact test
            // keeps
            const float reach = lim + 1.f;
            const int x0 = cell_of(a[j].x - reach, o2, W), x1 = cell_of(a[j].x + reach, o2, W);
            const int y0 = cell_of(a[j].y - reach, o2, H), y1 = cell_of(a[j].y + reach, o2, H);
            for (int y = y0; y <= y1; ++y) {
                const int row = obase[o2] + y * ocx[o2];
                const int end = cell[row + x1 + 1];
                for (int q = cell[row + x0]; q < end; ++q) {
                    const float4 b = rec[q];
                    const float dx = a[j].x - b.x, dy = a[j].y - b.y;
                    const float shi = fmaxf(a[j].z, b.z), slo = fminf(a[j].z, b.z);
                    if (((a[j].w > 0.f) == (b.w > 0.f)) & (dx * dx + dy * dy <= lim2) & (shi <= ratio_lim * slo)) {
                        if (fabsf(b.w) > aa) out |= 1u << j;
                        else dead[q] = 1;
                    }
                }
            }
        }
    }
    __syncthreads();
    uint32_t alive = 0u;
    {
        uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
        for (int j = 0; j < FIN_PER; ++j)
            if (tid + j * FIN_THREADS < n && !(out >> j & 1u) &&
                (low[j] >> 28 == 0u || !dead[cell[at[j] & (kFinCells - 1)] + (at[j] >> 12)])) {
                alive |= 1u << j;
                lo = min(lo, __float_as_uint(fabsf(a[j].w)));
                hi = max(hi, __float_as_uint(fabsf(a[j].w)));
            }
        wave_min_max(lo, hi);
        int na = __popc(alive);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) na += __shfl_xor(na, off);
        if (lane == 0 && na) {   // (one atomic of each kind per wave: a lane's own would queue up 1024 deep)
            atomicAdd(&n_alive, na);
            atomicMin(&lohi[0], lo);
            atomicMax(&lohi[1], hi);
        }
    }
    __syncthreads();   // every lane is done with the records and cells
    // Canonical order: a histogram of |p| over the survivors' own range,
    // strongest bin first, puts each one after all of the higher bins, and
    // the few of its own bin are compared with it by key
    const int total = n_alive, limit = min(topk > 0 ? topk : kp_cap, kp_cap), m = min(total, limit);
    const uint32_t top = lohi[1], range = top - lohi[0];
    const int sh = max(0, 32 - __clz((int)range | 1) - 12);   // range >> sh < kFinCells
    auto bin_of = [&](int j) { return (int)((top - __float_as_uint(fabsf(a[j].w))) >> sh); };
    reinterpret_cast<int4*>(cell)[tid] = make_int4(0, 0, 0, 0);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < FIN_PER; ++j)
        if (alive >> j & 1u) {
            const int b = bin_of(j), place = atomicAdd(&cell[b], 1);
            at[j] = b | place << 12;
        }
    __syncthreads();
    scan4(cell, wsum);
    if (tid == 0) cell[kFinCells] = total;
#pragma unroll
    for (int j = 0; j < FIN_PER; ++j)   // a crowded bin among those that are kept from
        if ((alive >> j & 1u) && (at[j] >> 12) >= kFinCrowd && cell[at[j] & (kFinCells - 1)] < m) crowded = 1;
    __syncthreads();
    auto key_of = [&](int j) { return ((unsigned long long)(~__float_as_uint(fabsf(a[j].w))) << 32) | low[j]; };
    if (!crowded) {   // uniform over the workgroup
#pragma unroll
        for (int j = 0; j < FIN_PER; ++j)
            if (alive >> j & 1u) key[cell[at[j] & (kFinCells - 1)] + (at[j] >> 12)] = key_of(j);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < FIN_PER; ++j)
            if (alive >> j & 1u) {
                const int b = at[j] & (kFinCells - 1), beg = cell[b];
                if (beg < m) {
                    const unsigned long long k = key_of(j);
                    int r = beg;
                    for (int q = beg; q < cell[b + 1]; ++q) r += key[q] < k;
                    if (r < m) idx[r] = (unsigned short)(tid + j * FIN_THREADS);
                    if (r == limit - 1) tmp[2] = (int)__float_as_uint(fabsf(a[j].w));   // the last one kept
                }
            }
        __syncthreads();
    } else {
        // many responses alike: a bitonic sort of all survivors
#pragma unroll
        for (int j = 0; j < FIN_PER; ++j)
            if (alive >> j & 1u) {
                const int q = cell[at[j] & (kFinCells - 1)] + (at[j] >> 12);
                key[q] = key_of(j);
                idx[q] = (unsigned short)(tid + j * FIN_THREADS);
            }
        int npow = 128;   // the sort works on whole 128-entry chunks (padding sorts last)
        while (npow < total) npow <<= 1;
        for (int i = total + tid; i < npow; i += FIN_THREADS) {
            key[i] = ~0ull;
            idx[i] = 0;
        }
        __syncthreads();
        bitonic_sort(key, idx, npow);
        if (tid == 0 && total >= limit) tmp[2] = (int)~(uint32_t)(key[limit - 1] >> 32);
    }
    for (int r = tid; r < m; r += FIN_THREADS) {
        const int i = idx[r];
        kp[(int64_t)img * kp_cap + r] = c[list ? list[i] : (uint32_t)i];
    }
    // the counters are left at zero for the next detection (every lane has read
    // this image's), which saves it a launch of its own for that
    if (active && tid < kMaxOctaves) active[img * kMaxOctaves + tid] = 0;
    if (img == 0 && tid < kXcds) cand_cnt[(gridDim.x + tid) * kCntStride] = 0;
    if (tid == 0) {
        cand_cnt[img * kCntStride] = 0;
        count[img] = m;
        // A reduced image's output is exact when its last kept keypoint is
        // stronger than every candidate that was dropped: each kept one was
        // judged against all candidates at least as strong, and no dropped
        // candidate could rank among them.  Otherwise the image is flagged.
        if (list && limit > 0) {
            const bool exact = total >= limit && (uint32_t)tmp[2] > min_all;
            if (!exact) atomicOr(flags, kFlagSelectInexact);
        }
    }
}

}  // namespace

hipError_t launch_clear(int32_t* p, int n, int stride, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_clear, dim3((n + 255) / 256), dim3(256), 0, stream, p, n, stride);
    return hipGetLastError();
}

hipError_t launch_detect_strips(const float* pyr, const DetTile* strips, int nstrips, int strip_h, int variant, int grid,
                                const DetParams& dp, const GateParams& gate, int32_t* work, const DetOut& out,
                                hipStream_t stream) {
    if (nstrips <= 0) return hipSuccess;
#define DETECT_LAUNCH(G, P, NB)                                                                                    \
    hipLaunchKernelGGL((k_detect_strip<G, P>), dim3(NB), dim3(256), 0, stream, pyr, strips, nstrips, strip_h, dp, gate, \
                       work, out)
    if (variant == kDetectPersistent) {
        // a multiple of the XCD count, no larger than one wave per strip
        int g = std::min(grid, (nstrips + 4 * kXcds - 1) / (4 * kXcds) * kXcds);
        g = std::max(kXcds, g / kXcds * kXcds);
        if (gate.mask)
            DETECT_LAUNCH(true, true, g);
        else
            DETECT_LAUNCH(false, true, g);
    } else {
        const int nb = (nstrips + 3) / 4;
        if (gate.mask)
            DETECT_LAUNCH(true, false, nb);
        else
            DETECT_LAUNCH(false, false, nb);
    }
#undef DETECT_LAUNCH
    return hipGetLastError();
}

hipError_t launch_finalize(const cdvs_keypoint* cand, const float* absp, int32_t* cand_cnt, const int64_t* cand_off,
                           const int32_t* cand_capv, int32_t* active, uint32_t* lists, const int32_t* wh, int n_images,
                           float dedup_ratio, int topk, int kp_cap, cdvs_keypoint* kp, int32_t* count, int32_t* flags,
                           hipStream_t stream) {
    if (n_images <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_finalize, dim3(n_images), dim3(FIN_THREADS), 0, stream, cand, absp, cand_cnt, cand_off,
                       cand_capv, active, lists, wh, dedup_ratio, topk, kp_cap, kp, count, flags);
    return hipGetLastError();
}

}  // namespace cdvs
