// Keypoint relevance and selection on gfx950 (Sec. III-B, Eqs. (4)-(5)):
// r = f1(sigma) f2(|p|) f3(d) f4(rho) f5(p_ss), each f a table over
// quantised values of one characteristic (bin = number of table edges at
// or below the value), and per image the keypoints of highest r are kept,
// equal r in their input order.  d is the distance to the image centre over
// the centre's distance to a corner.  Single precision, the products left
// to right, the distance without fused operations.
//
// One 1024-lane workgroup per image: every record's score is computed once
// and the records are ordered by the complement of r's bits (r >= 0, so its
// bits order like its value), equal ones by input index, and the first n_keep
// are copied out.  Up to 1024 records, one per lane, are sorted by four stable
// counting passes of 8 bits; more, and few of them in many images, by a bitonic
// sort on (r, index) pairs in LDS.  The bitonic sort's exchanges at distances below 128 stay inside one
// 128-key chunk, which one wave holds in registers (two keys per lane) and
// exchanges by lane shuffles; only the longer distances go through LDS with a
// workgroup barrier each.  Either is a chain of exchanges in a single
// workgroup per compute unit, bound by their latencies: for 1000 records the
// bitonic sort's 55 steps took 9 us of the kernel's 15, the four passes take
// 7.
#include "cdvs_internal.h"

namespace cdvs {

namespace {

constexpr int kRelThreads = 1024;
// Images of at most kRelFew records in a batch of more than kRelFewImages
// take the bitonic sort: its few stages leave most of their workgroup's waves
// idle, which then stand in nobody's way, while every wave counts in all four
// passes (for 64, 256 and 300 records, bitonic and counting: 256 images 8.5 and
// 7.4, 8.4 and 7.8, 8.7 and 8.0 us; 512 images 9.0 and 13.0, 11.4 and 13.7, 15.2 and
// 14.7; 4096 images 59 and 93, 87 and 104, 114 and 112).
constexpr int kRelFew = 256, kRelFewImages = 256;

__device__ __forceinline__ float centre_distance(float x, float y, float hx, float hy) {
#pragma clang fp contract(off)
    const float dx = x - hx, dy = y - hy;
    return sqrtf(dx * dx + dy * dy) / sqrtf(hx * hx + hy * hy);
}

__device__ __forceinline__ int bin_of(const float* edges, float v) {
    int b = 0;
#pragma unroll
    for (int e = 0; e < kRelEdges; ++e) b += edges[e] <= v ? 1 : 0;
    return b;
}

// One compare-exchange of a bitonic stage of block size `size` at distance
// S < 64, for the key k of element i held by this lane, whose partner
// (i ^ S) is in lane ^ S: the lower index keeps the smaller key in an
// ascending block, the larger in a descending one (by selects, no branch).
template <int S>
__device__ __forceinline__ unsigned long long bitonic_lane_step(unsigned long long k, int i, int size) {
    const unsigned long long o = lane_xor64<S>(k);
    const bool want_min = ((i & size) == 0) == ((i & S) == 0);
    const unsigned long long mn = o < k ? o : k, mx = o < k ? k : o;
    return want_min ? mn : mx;
}

// The steps at distances below 128 of bitonic block sizes first..last, on
// the 128-key chunks of key[0 .. npow): each wave takes whole chunks, two
// keys per lane (elements c*128 + lane and c*128 + 64 + lane).
__device__ __forceinline__ void bitonic_chunk_steps(unsigned long long* key, int npow, int first, int last) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int c = wave; c < npow / 128; c += nw) {
        const int i0 = 128 * c + lane, i1 = i0 + 64;
        unsigned long long k0 = key[i0], k1 = key[i1];
        for (int size = first; size <= last; size <<= 1) {
            if (size >= 128) {   // distance 64: the lane's own pair, one direction for both
                const bool asc = (i0 & size) == 0;
                const unsigned long long lo = k0 < k1 ? k0 : k1, hi = k0 < k1 ? k1 : k0;
                k0 = asc ? lo : hi;
                k1 = asc ? hi : lo;
            }
#define CDVS_STEP(S)                                 \
    if (size > S) {                                  \
        k0 = bitonic_lane_step<S>(k0, i0, size);     \
        k1 = bitonic_lane_step<S>(k1, i1, size);     \
    }
            CDVS_STEP(32) CDVS_STEP(16) CDVS_STEP(8) CDVS_STEP(4) CDVS_STEP(2) CDVS_STEP(1)
#undef CDVS_STEP
        }
        key[i0] = k0;
        key[i1] = k1;
    }
}

// Ascending bitonic sort of key[0 .. npow) (npow a power of two, at least
// 128) by the whole workgroup: block sizes up to 128 entirely in
// registers, then for each larger size its distances of 128 and more
// through LDS (a barrier each) and the rest in registers.
__device__ void bitonic_sort_keys(unsigned long long* key, int npow) {
    bitonic_chunk_steps(key, npow, 2, 128);
    __syncthreads();
    for (int size = 256; size <= npow; size <<= 1) {
        for (int stride = size >> 1; stride >= 128; stride >>= 1) {
            for (int t = threadIdx.x; t < npow / 2; t += blockDim.x) {
                const int lo = 2 * t - (t & (stride - 1)), hi = lo + stride;
                const unsigned long long a = key[lo], b = key[hi];
                if ((a > b) == ((lo & size) == 0)) {
                    key[lo] = b;
                    key[hi] = a;
                }
            }
            __syncthreads();
        }
        bitonic_chunk_steps(key, npow, size, size);
        __syncthreads();
    }
}

// The lane's rank among 1024 keys k, one per lane of the workgroup, in
// ascending order, equal keys in lane order: the keys sorted, and where each
// was.  Every pass splits the keys by 8 bits, stably: a wave's lanes of equal
// digit find each other by ballots, the digit's counts per wave are summed up
// over digits and waves, and keys and lanes move to their places.
struct RadixShared {
    uint32_t key[kRelThreads];
    uint16_t idx[kRelThreads];
    uint16_t hist[256][kRelThreads / 64];   // [digit][wave]: counts, then places
    int total[kRelThreads / 64];
};

__device__ __forceinline__ int wave_inclusive_sum(int s) {
    s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xf, 0xf, true);    // from 1, 2, 4 and 8 lanes below in the row of 16
    s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xf, 0xf, true);
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xf, 0xf, true);
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xf, 0xf, true);
    s += __builtin_amdgcn_update_dpp(0, s, 0x142, 0xa, 0xf, false);   // the rows of 16 before it
    s += __builtin_amdgcn_update_dpp(0, s, 0x143, 0xc, 0xf, false);
    return s;
}

__device__ __forceinline__ void radix_sort_lanes(RadixShared& sh, uint32_t& k, int& idx) {
    static_assert(kRelThreads == 1024, "four counters per lane, 16 waves");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint2* counters = reinterpret_cast<uint2*>(sh.hist);   // four per lane: waves 4 (tid % 4) .. of digit tid / 4
    idx = tid;
#pragma unroll 1
    for (int bit = 0; bit < 32; bit += 8) {
        counters[tid] = make_uint2(0u, 0u);
        const uint32_t d = (k >> bit) & 255u;
        uint32_t mlo = ~0u, mhi = ~0u;   // the wave's lanes with this digit
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool on = (d >> b) & 1u;
            const uint64_t bal = __builtin_amdgcn_ballot_w64(on);
            const uint32_t flip = on ? 0u : ~0u;
            mlo &= (uint32_t)bal ^ flip;
            mhi &= (uint32_t)(bal >> 32) ^ flip;
        }
        const int rank = __builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0));
        __syncthreads();
        if (rank == 0) sh.hist[d][wave] = (uint16_t)(__popc(mlo) + __popc(mhi));
        __syncthreads();
        const uint2 c = counters[tid];
        const int c0 = c.x & 0xffffu, c1 = c.x >> 16, c2 = c.y & 0xffffu, c3 = c.y >> 16;
        const int sum = c0 + c1 + c2 + c3, incl = wave_inclusive_sum(sum);
        if (lane == 63) sh.total[wave] = incl;
        __syncthreads();
        const int before =
            __builtin_amdgcn_readlane(wave_inclusive_sum(lane < wave ? sh.total[lane & 15] : 0), 15);   // (wave <= 15)
        const uint32_t p0 = (uint32_t)(before + incl - sum), p1 = p0 + c0, p2 = p1 + c1, p3 = p2 + c2;
        counters[tid] = make_uint2(p0 | (p1 << 16), p2 | (p3 << 16));
        __syncthreads();
        const int to = sh.hist[d][wave] + rank;
        sh.key[to] = k;
        sh.idx[to] = (uint16_t)idx;
        __syncthreads();
        k = sh.key[tid];
        idx = sh.idx[tid];
    }
}

__global__ __launch_bounds__(kRelThreads) void k_relevance(const cdvs_keypoint* __restrict__ kp_in,
                                                           const int32_t* __restrict__ count_in,
                                                           const int32_t* __restrict__ wh, int kp_cap,
                                                           const float* __restrict__ edges,
                                                           const float* __restrict__ values, int n_keep,
                                                           cdvs_keypoint* __restrict__ kp_out,
                                                           int32_t* __restrict__ count_out,
                                                           float* __restrict__ score_out) {
    __shared__ union {
        unsigned long long key[CDVS_MAX_KP_CAPACITY];
        RadixShared radix;
    } sm;
    unsigned long long* key = sm.key;
    __shared__ float se[kRelFeatures * kRelEdges], sv[kRelFeatures * kRelBins];
    const int img = blockIdx.x, tid = threadIdx.x;
    if (tid < kRelFeatures * kRelEdges) se[tid] = edges[tid];
    if (tid < kRelFeatures * kRelBins) sv[tid] = values[tid];
    __syncthreads();
    const int n = min(max(count_in[img], 0), kp_cap);
    int npow = 128;   // the sort works on whole 128-key chunks (padding sorts last)
    while (npow < n) npow <<= 1;
    const float hx = 0.5f * (float)(wh[2 * img] - 1), hy = 0.5f * (float)(wh[2 * img + 1] - 1);
    const cdvs_keypoint* in = kp_in + (int64_t)img * kp_cap;
    // record i's sort key
    auto score = [&](int i) {
        const cdvs_keypoint p = in[i];
        const float f[kRelFeatures] = {p.sigma, fabsf(p.p), centre_distance(p.x, p.y, hx, hy), p.rho, p.p_ss};
        float r = sv[bin_of(se, f[0])];
#pragma unroll
        for (int c = 1; c < kRelFeatures; ++c) r = r * sv[c * kRelBins + bin_of(se + c * kRelEdges, f[c])];
        return 0xFFFFFFFFu - __float_as_uint(r);
    };
    if (n <= kRelThreads && (n > kRelFew || gridDim.x <= kRelFewImages)) {   // uniform
        uint32_t k = tid < n ? score(tid) : 0xFFFFFFFFu;   // padding sorts last: no key is higher, and the index is
        int idx;
        radix_sort_lanes(sm.radix, k, idx);
        const int m = min(n, n_keep);
        if (tid < m) {
            kp_out[(int64_t)img * kp_cap + tid] = in[idx];
            if (score_out) score_out[(int64_t)img * kp_cap + tid] = __uint_as_float(0xFFFFFFFFu - k);
        }
        if (tid == 0) count_out[img] = m;
        return;
    }
    for (int i = tid; i < npow; i += kRelThreads)
        key[i] = i < n ? ((unsigned long long)score(i) << 32) | (unsigned)i : ~0ull;   // padding sorts last
    __syncthreads();
    bitonic_sort_keys(key, npow);
    const int m = min(n, n_keep);
    for (int i = tid; i < m; i += kRelThreads) {
        const unsigned long long k = key[i];
        kp_out[(int64_t)img * kp_cap + i] = in[(unsigned)k];
        if (score_out) score_out[(int64_t)img * kp_cap + i] = __uint_as_float(0xFFFFFFFFu - (unsigned)(k >> 32));
    }
    if (tid == 0) count_out[img] = m;
}

}  // namespace

hipError_t launch_relevance(const cdvs_keypoint* kp_in, const int32_t* count_in, const int32_t* wh, int n_images,
                            int kp_cap, const float* edges, const float* values, int n_keep, cdvs_keypoint* kp_out,
                            int32_t* count_out, float* score_out, hipStream_t s) {
    if (n_images <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_relevance, dim3(n_images), dim3(kRelThreads), 0, s, kp_in, count_in, wh, kp_cap, edges, values,
                       n_keep, kp_out, count_out, score_out);
    return hipGetLastError();
}

}  // namespace cdvs
