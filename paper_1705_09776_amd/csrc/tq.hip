// Transform coding and ternary quantisation of local descriptors on gfx950
// (Sec. III-C): each 8-bin cell histogram goes through one of two order-8
// transforms of additions, subtractions and power-of-two scalings (cells
// with row + col even take set A, the others set B, so that neighbouring
// cells differ), and each transformed element is coded as -1, 0 or +1 by
// two thresholds of its own.  The first n elements of a priority order are
// packed at two bits each (01 = +1, 10 = -1, 00 = 0; position p in word
// p / 16, bits 2 (p % 16) and up) into eight 32-bit words per descriptor,
// so the code is 2n bits instead of the 512-byte float descriptor.
//
// One lane per (descriptor, cell), four descriptors per wave and step; a wave
// takes up to four steps, with its cell's thresholds and its eight positions of
// the priority order in registers and the next step's descriptors on the way.
// Lanes exchange symbols through a few bytes of LDS per wave, without a
// barrier, and every lane gathers eight positions, half a code word.  (With a
// workgroup of 16 descriptors that staged the tables in LDS, met at two
// barriers and had half its lanes gather a word each, 256,000 descriptors from
// memory took 37 us; now 25 for 139 MB, near what a copy reaches.  One, two
// and eight steps: 29, 26 and 26; a run of steps per wave instead of the
// workgroup's waves side by side: 33.)
// Every transformed value is evaluated left to right as the
// transforms are written (parentheses first), in single precision, with no
// fused operations (there is no product to fuse; the scalings are exact),
// so the thresholds see exactly the values a plain single-precision
// evaluation gives.
#include <algorithm>

#include "cdvs_internal.h"

namespace cdvs {

namespace {

// Orders one wave's own LDS accesses.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

constexpr int kTqWaves = 4;     // per workgroup
constexpr int kTqDesc = 4;      // descriptors per wave and step
constexpr int kTqMaxSteps = 4;

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct Half {   // a cell's eight bins
    f32x4 a, b;
};

// The cell's bins of descriptor slot g.
__device__ __forceinline__ void load_cell(const float* __restrict__ desc, uint32_t g, int cell, Half& h) {
    const f32x4* p = reinterpret_cast<const f32x4*>(desc + (int64_t)g * kDescDim + cell * 8);
    h.a = __builtin_nontemporal_load(p);   // (read once)
    h.b = __builtin_nontemporal_load(p + 1);
}

// BY_IMAGE: a workgroup's descriptors are one image's, all images' first ones
// come first, and a workgroup beyond its image's count ends at once.  So the
// work lies at the front of the grid and spreads over all compute units
// however few of the slots are in use (in slot order, a capacity that is many
// workgroups puts the used ones of every image on the same XCDs and units).
// For capacities of at least four workgroups, where the one that the end of a
// capacity leaves partly empty costs less; below, workgroups divide the slots of
// the whole batch.  By images, capacity and descriptors in use, in slot order
// and by image: 128 of 4096: 100: 25 and 5 us, 1000: 31 and 15, all: 58 and 58;
// 1024 of 1000: 100: 33 and 15; 256 of 1000: 300: 15 and 9, all: 27.9 and 27.4; 16 of
// 8192: 1000: 8.3 and 5.3, all: 15.5 and 18.
template <bool BY_IMAGE>
__global__ __launch_bounds__(64 * kTqWaves) void k_tq_encode(const float* __restrict__ desc,
                                                             const int32_t* __restrict__ count, uint32_t slots, KpDiv kd,
                                                             const float* __restrict__ lo, const float* __restrict__ hi,
                                                             const int32_t* __restrict__ order, int n_elem, int steps,
                                                             uint32_t* __restrict__ codes) {
    // symbol rows padded to 136 bytes: a cell's eight symbols go out as one
    // 8-byte store, and the four descriptors of a wave start on different banks
    constexpr int kSymStride = kDescDim + 8;
    __shared__ __align__(8) uint8_t sym[kTqWaves][kTqDesc][kSymStride];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, cell = lane & 15, dl = lane >> 4;
    constexpr uint32_t kStep = kTqWaves * kTqDesc;   // (the workgroup's waves side by side)
    uint32_t g = wave * kTqDesc + dl, end;           // the lane's slot of the first step; past the last in use of its image
    if constexpr (BY_IMAGE) {
        const uint32_t n = slots / kd.d, img = blockIdx.x % n, first = blockIdx.x / n * steps * kStep;   // uniform
        const uint32_t K = min(max(count[img], 0), (int)kd.d);
        if (first >= K) return;
        g += img * kd.d + first;
        end = img * kd.d + K;
    } else {
        g += blockIdx.x * steps * kStep;
    }
    auto in_use = [&](uint32_t slot) {
        if constexpr (BY_IMAGE) return slot < end;
        if (slot >= slots) return false;
        const uint32_t img = kp_div_q(slot, kd);
        return (int)(slot - img * kd.d) < min(max(count[img], 0), (int)kd.d);
    };
    Half h;
    bool active = in_use(g);
    if (active) load_cell(desc, g, cell, h);
    float tlo[8], thi[8];
    int ord[8];
    uint32_t used = 0u;   // the lane's 16 bits of positions below n_elem
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        tlo[k] = lo[cell * 8 + k];
        thi[k] = hi[cell * 8 + k];
        ord[k] = order[cell * 8 + k] & (kDescDim - 1);   // a position in the symbol row, whatever the caller passed
        if (cell * 8 + k < n_elem) used |= 3u << (2 * k);
    }
    const bool set_a = (((cell >> 2) + (cell & 3)) & 1) == 0;
    uint8_t* row = sym[wave][dl];
    for (int st = 0; st < steps; ++st) {
        Half nh;
        const bool next = st + 1 < steps && in_use(g + kStep);
        if (next) load_cell(desc, g + kStep, cell, nh);
        if (active) {
            const float h0 = h.a.x, h1 = h.a.y, h2 = h.a.z, h3 = h.a.w, h4 = h.b.x, h5 = h.b.y, h6 = h.b.z, h7 = h.b.w;
            float v[8];
            if (set_a) {
                v[0] = (h2 - h6) / 2.f;
                v[1] = (h3 - h7) / 2.f;
                v[2] = (h0 - h1) / 2.f;
                v[3] = (h2 - h3) / 2.f;
                v[4] = (h4 - h5) / 2.f;
                v[5] = (h6 - h7) / 2.f;
                v[6] = ((h0 + h4) - (h2 + h6)) / 4.f;
                v[7] = ((h0 + h2 + h4 + h6) - (h1 + h3 + h5 + h7)) / 8.f;
            } else {   // set B
                v[0] = (h0 - h4) / 2.f;
                v[1] = (h1 - h5) / 2.f;
                v[2] = (h7 - h0) / 2.f;
                v[3] = (h1 - h2) / 2.f;
                v[4] = (h3 - h4) / 2.f;
                v[5] = (h5 - h6) / 2.f;
                v[6] = ((h1 + h5) - (h3 + h7)) / 4.f;
                v[7] = ((h0 + h1 + h2 + h3) - (h4 + h5 + h6 + h7)) / 8.f;
            }
            uint32_t s0 = 0u, s1 = 0u;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t c = v[k] > thi[k] ? 1u : (v[k] < tlo[k] ? 2u : 0u);
                if (k < 4) s0 |= c << (8 * k);
                else s1 |= c << (8 * (k - 4));
            }
            *reinterpret_cast<uint2*>(row + cell * 8) = make_uint2(s0, s1);
        }
        wave_sync();
        uint32_t w = 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j) w |= (uint32_t)row[ord[j]] << (2 * j);
        wave_sync();   // (before the next step's symbols)
        w &= used;
        // the odd lane beside it has the word's upper half
        w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xf, 0xf, false) << 16;
        if (active && (cell & 1) == 0) codes[(int64_t)g * kTqWords + (cell >> 1)] = w;
        h = nh;
        active = next;
        g += kStep;
    }
}

}  // namespace

hipError_t launch_tq_encode(const float* desc, const int32_t* count, int n_images, int kp_cap, const float* lo,
                            const float* hi, const int32_t* order, int n_elem, uint32_t* codes, hipStream_t s) {
    const int64_t slots = (int64_t)n_images * kp_cap;
    if (slots <= 0) return hipSuccess;
    // several steps only where there are still waves for the whole chip (8192)
    const int64_t wave_steps = (slots + kTqDesc - 1) / kTqDesc;
    const int steps = (int)std::min<int64_t>(std::max<int64_t>(wave_steps / 8192, 1), kTqMaxSteps);
    const int per_wg = steps * kTqWaves * kTqDesc;   // descriptors
    const KpDiv kd = make_kp_div((uint32_t)kp_cap);
    if (kp_cap >= 4 * per_wg)
        hipLaunchKernelGGL(k_tq_encode<true>, dim3((unsigned)(n_images * ((kp_cap + per_wg - 1) / per_wg))),
                           dim3(64 * kTqWaves), 0, s, desc, count, (uint32_t)slots, kd, lo, hi, order, n_elem, steps, codes);
    else
        hipLaunchKernelGGL(k_tq_encode<false>, dim3((unsigned)((slots + per_wg - 1) / per_wg)), dim3(64 * kTqWaves), 0, s,
                           desc, count, (uint32_t)slots, kd, lo, hi, order, n_elem, steps, codes);
    return hipGetLastError();
}

}  // namespace cdvs
