// Offline pre-processing of the GQS layer on the GPU (gfx950): the same steps as the host packer
// -- group the weights along K in runs of G, score every group (Sec. 3.1 Eq. 4 with a caller-supplied
// diag(H^-1), or the group's sum of squares), prune the least salient groups of every row
// (Sec. 3.2, Fig. 3), quantise the kept ones (Eq. 1-2) -- producing the BSR arrays of the Sec. 3.2
// listing plus scales and zeros, and, in the same pass, the blocks of the device image that the
// GEMV kernel streams.  The arithmetic is the host packer's operation for operation (float64
// saliency sums in index order, single IEEE fp32 operations in the quantiser, round-half-even),
// so the results are the same bits.
//
// One wavefront per output row.  The saliencies of the row lie in LDS as 64-bit keys (a sum of
// squares is not negative, so its bit pattern orders like the number); the pruned count-th smallest
// is found by bisection over the keys' bits, one ballot per 64 columns and step, and the columns
// that stay are listed in order.  Lane by lane the listed groups are then quantised and written,
// neighbouring lanes to neighbouring places.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "gqsa_internal.hpp"

namespace gqsa {
namespace {

constexpr int kThreads = 256;          // of the small kernels
constexpr int kMaxColumns = 4096;      // group-columns of a row (the format's limit): 40 KB of LDS

struct PackArgs {
    const float* W;            // [N][K]
    const float* hinv;         // [K] or nullptr
    const int32_t* rowIndex;   // [N+1]
    const int64_t* row_pos;    // [N] first stream position of every row
    int32_t* groups;           // canonical arrays (outputs)
    uint8_t* values;
    uint16_t* scales;
    uint16_t* zeros;
    uint8_t* blocks;           // device image, blocks region (zeroed beforehand)
    int* status;               // bit 0: a non-finite saliency; bit 1: a bad entry of hinv; bit 2: a scale beyond fp16
    long long K;
    int kg, bits, cb, U, L, bb, slots_per_group;     // (U blocks per tile, L lanes in use per block)
};

__device__ __forceinline__ uint16_t half_bits(float f) { return __builtin_bit_cast(uint16_t, static_cast<_Float16>(f)); }
__device__ __forceinline__ float half_value(uint16_t b) { return static_cast<float>(__builtin_bit_cast(_Float16, b)); }

// Eight weights.  WIDE: the address is a multiple of 16 bytes (two loads); else any float's.
template <bool WIDE>
__device__ __forceinline__ void load8(const float* p, float* w)
{
    if constexpr (WIDE) {
        const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
        w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
        w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = p[e];
    }
}

// A workgroup is one wavefront: its LDS accesses complete in order, this only keeps the compiler
// from moving them across.
__device__ __forceinline__ void wavefront_fence() { __syncthreads(); }

// W is read twice (the second time, by the kept groups, mostly from the caches); the 64 MB of 4096x4096 take 11 us
// at the rate of a plain read, the kernel 36 us: the rest is the bisection's chain of LDS reads and ballots
// (about 25 steps: a step per leading bit until the pruned count is met exactly) and 17 divisions per kept
// group.  A workgroup of 256 threads per row that compared every key with every other one, its threads
// each reading and writing groups of their own, took 101 us, and its time grew with the square of the columns: S = 50 %,
// W4 G = 16 4096x4096 101 -> 36 us, 2441x16384 595 -> 94 us; W8 G = 8 4096x4096 219 -> 46 us, 4883x8192 at
// S = 30 % 927 -> 145 us; W4 G = 128 4096x8192 186 -> 65 us; W4 G = 32 40000x1024 at S = 70 % 454 -> 98 us.
template <int G, bool WIDE>
__global__ __launch_bounds__(kLanes) void pack_rows_kernel(PackArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int kg = a.kg;
    unsigned long long* keys = reinterpret_cast<unsigned long long*>(lds);      // [kg]
    uint16_t* list = reinterpret_cast<uint16_t*>(lds + static_cast<size_t>(kg) * 8);    // [kept groups] their columns

    const int lane = threadIdx.x;
    const long long n = blockIdx.x;
    const float* wrow = a.W + n * a.K;
    const int g0 = a.rowIndex[n];
    const int keep = a.rowIndex[n + 1] - g0;
    if (keep == 0) return;                                  // (uniform: the whole wavefront leaves)
    const int drop = kg - keep;

    // saliency of a weight: w^2 / d_k^2; of a group: the sum over its members, float64, index order
    bool bad = false;
    for (int c = lane; c < kg; c += kLanes) {
        const float* p = wrow + static_cast<long long>(c) * G;
        double acc = 0.0;
#pragma unroll
        for (int h = 0; h < G / 8; ++h) {
            float w[8];
            load8<WIDE>(p + 8 * h, w);
            if (a.hinv) {
                const float* d = a.hinv + static_cast<long long>(c) * G + 8 * h;
                for (int e = 0; e < 8; ++e) {
                    const double t = static_cast<double>(w[e]) / static_cast<double>(d[e]);
                    acc += t * t;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) acc += static_cast<double>(w[e]) * static_cast<double>(w[e]);
            }
        }
        keys[c] = __builtin_bit_cast(unsigned long long, acc);
        bad = bad || !(fabs(acc) <= 1.79769313486231570815e+308);     // NaN or infinite
    }
    if (__ballot(bad) != 0) {
        if (lane == 0) atomicOr(a.status, 1);
        return;
    }
    wavefront_fence();

    // The pruned groups are the `drop` first ones in the order (saliency, column).  Bisection from the
    // top bit down (bit 63, the sign, is clear): `low` = the largest number found so far with at most `drop`
    // keys below it, bit by bit; once exactly `drop` keys lie below it, no tie is left to decide.
    unsigned long long low = 0;
    int below = 0;             // keys less than low
    if (drop > 0) {
        for (int bit = 62; bit >= 0 && below != drop; --bit) {
            const unsigned long long candidate = low | (1ull << bit);
            int count = 0;
            for (int c = lane; c - lane < kg; c += kLanes)
                count += __popcll(__ballot(c < kg && keys[c] < candidate));
            if (count <= drop) {
                low = candidate;
                below = count;
            }
        }
    }
    // pruned: the keys below `low`, and of those equal to it the first drop - below by column
    int ties_left = drop - below, kept_before = 0;
    for (int base = 0; base < kg; base += kLanes) {
        const int c = base + lane;
        const unsigned long long key = c < kg ? keys[c] : 0;
        const unsigned long long lanes_below = (1ull << lane) - 1ull;
        const unsigned long long equal = __ballot(c < kg && key == low);
        const bool tie_goes = ((equal >> lane) & 1ull) != 0 && static_cast<int>(__popcll(equal & lanes_below)) < ties_left;
        const bool stays = c < kg && key >= low && !tie_goes;
        const unsigned long long staying = __ballot(stays);
        if (stays) list[kept_before + __popcll(staying & lanes_below)] = static_cast<uint16_t>(c);
        kept_before += __popcll(staying);
        ties_left -= min(ties_left, static_cast<int>(__popcll(equal)));
    }
    wavefront_fence();

    // where the row begins in the image: tiles of U blocks of L groups, lane l owns U consecutive positions
    const int tile_groups = a.L * a.U;
    const long long tile0 = a.row_pos[n] / tile_groups;
    const int first = static_cast<int>(a.row_pos[n] % tile_groups);
    constexpr float kMinScale = 0x1p-14f;
    const float levels = static_cast<float>((1 << a.bits) - 1);
    const int cb = a.cb, pb = cb < 16 ? cb : 16;
    for (int i = lane; i < keep; i += kLanes) {         // i = the group's number inside its row
        const int c = list[i];
        const long long g = static_cast<long long>(g0) + i;
        const float* p = wrow + static_cast<long long>(c) * G;
        float w[G];
#pragma unroll
        for (int h = 0; h < G / 8; ++h) load8<WIDE>(p + 8 * h, w + 8 * h);
        // Eq. 1: the first smallest and the last largest element, as the host's scan finds them
        float lo = w[0], hi = w[0];
#pragma unroll
        for (int j = 1; j < G; ++j) {
            if (w[j] < lo) lo = w[j];
            if (!(w[j] < hi)) hi = w[j];
        }
        float s = (hi - lo) / levels;
        uint16_t sb = half_bits(s);
        if ((sb & 0x7FFFu) >= 0x7C00u) atomicOr(a.status, 4);      // the group's range is beyond what an fp16 scale holds
        s = half_value(sb);
        if (!(s >= kMinScale)) {
            s = kMinScale;
            sb = half_bits(s);
        }
        float z = __builtin_rintf(-lo / s);         // round-half-even
        z = (z < -2048.0f) ? -2048.0f : z;
        z = (2048.0f < z) ? 2048.0f : z;
        const uint16_t zb = half_bits(z);
        a.groups[g] = c;
        a.scales[g] = sb;
        a.zeros[g] = zb;
        const int place = first + i;                // of the group, counted from the start of the row's first tile
        const int position = place % tile_groups;
        const long long block = (tile0 + place / tile_groups) * a.U + position % a.U;
        const int slot = position / a.U;
        uint8_t* base = a.blocks + block * a.bb;
        uint8_t* vout = a.values + g * cb;
        // Eq. 2, eight codes at a time: a canonical word (two codes per byte, even element low; or
        // one byte per code) and the image's word (4-bit: element 2m at bits 4m, 2m+1 at 16+4m)
#pragma unroll
        for (int h = 0; h < G / 8; ++h) {
            uint32_t q8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float q = __builtin_rintf(w[8 * h + e] / s) + z;
                q = (0.0f < q) ? q : 0.0f;
                q = (q < levels) ? q : levels;
                q8[e] = static_cast<uint32_t>(q);
            }
            if (a.bits == 4) {
                uint32_t canon = 0, image = 0;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    canon |= q8[e] << (4 * e);
                    image |= q8[e] << ((e & 1) ? 16 + 4 * (e >> 1) : 4 * (e >> 1));
                }
                *reinterpret_cast<uint32_t*>(vout + 4 * h) = canon;
                const int byte = 4 * h;             // of the lane's code string
                *reinterpret_cast<uint32_t*>(base + (byte / pb) * a.L * pb + slot * pb + byte % pb) = image;
            } else {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const uint32_t word = q8[4 * half] | (q8[4 * half + 1] << 8) | (q8[4 * half + 2] << 16) | (q8[4 * half + 3] << 24);
                    const int byte = 8 * h + 4 * half;
                    *reinterpret_cast<uint32_t*>(vout + byte) = word;
                    *reinterpret_cast<uint32_t*>(base + (byte / pb) * a.L * pb + slot * pb + byte % pb) = word;
                }
            }
        }
        *reinterpret_cast<uint32_t*>(base + a.L * cb + slot * 4) = static_cast<uint32_t>(sb) | (static_cast<uint32_t>(zb) << 16);
        *reinterpret_cast<uint16_t*>(base + a.L * (cb + 4) + slot * 2) =
            static_cast<uint16_t>(((c * a.slots_per_group) << 4) | (i == 0 ? 1 : 0));
    }
}

template <int G>
void launch_pack_rows(const PackArgs& a, int64_t n_rows, hipStream_t s)
{
    const size_t lds = static_cast<size_t>(a.kg) * 10;
    const dim3 grid(static_cast<unsigned>(n_rows)), block(kLanes);
    // (K is a multiple of 16: with an aligned W every group of every row is aligned)
    if ((reinterpret_cast<uintptr_t>(a.W) & 15u) == 0)
        hipLaunchKernelGGL((pack_rows_kernel<G, true>), grid, block, lds, s, a);
    else
        hipLaunchKernelGGL((pack_rows_kernel<G, false>), grid, block, lds, s, a);
}

__global__ __launch_bounds__(kThreads) void check_hinv_kernel(const float* d, long long K, int* status)
{
    const long long k = static_cast<long long>(blockIdx.x) * kThreads + threadIdx.x;
    if (k < K && !(d[k] > 0.0f && d[k] <= 3.40282346638528859812e+38f)) atomicOr(status, 2);
}

struct DeviceBuffers {        // temporaries of one pack, freed whatever happens
    void* p[8] = {};
    ~DeviceBuffers() { for (void* q : p) if (q) (void)hipFree(q); }
};

#define GQSA_HIP(call)                                                                   \
    do {                                                                                 \
        const hipError_t e_ = (call);                                                    \
        if (e_ != hipSuccess) {                                                          \
            std::fprintf(stderr, "libgqsa: %s: %s\n", #call, hipGetErrorString(e_));    \
            return GQSA_ERR_HIP;                                                         \
        }                                                                                \
    } while (0)

}  // namespace

// W_dev [N][K] fp32 and hinv_dev [K] (or nullptr) on the current GPU; m has N, K, G, bits and its
// row pointers (the kept count of every row is known beforehand).  Fills the canonical arrays and
// the device image of m -- on the GPU, then copied to the host side of the handle -- and leaves
// the handle uploaded.  Synchronises `stream`.
gqsa_status_t pack_on_device(const float* W_dev, const float* hinv_dev, gqsa_matrix* m, void* stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t nnz = m->nnzg();
    const int cb = m->code_bytes();
    if (m->K / m->G > kMaxColumns) return GQSA_ERR_SHAPE;
    // the layout of the image follows from the row pointers alone: partition, row positions,
    // per-worker records, row tables (host), with the blocks left empty
    std::vector<int64_t> row_pos;
    if (gqsa_status_t st = build_image(m, default_partition(*m), /*fill_blocks=*/false, &row_pos)) return st;
    m->groups.assign(static_cast<size_t>(nnz), 0);
    m->values.assign(static_cast<size_t>(nnz) * cb, 0);
    m->scales.assign(static_cast<size_t>(nnz), 0);
    m->zeros.assign(static_cast<size_t>(nnz), 0);

    DeviceBuffers tmp;
    void* img = nullptr;
    GQSA_HIP(hipMalloc(&img, m->image.size()));
    struct ImageGuard { void* p; ~ImageGuard() { if (p) (void)hipFree(p); } } guard{img};
    const size_t blocks_bytes = m->map.wave_info;          // the blocks region comes first
    GQSA_HIP(hipMemsetAsync(img, 0, blocks_bytes, s));
    GQSA_HIP(hipMemcpyAsync(static_cast<uint8_t*>(img) + blocks_bytes, m->image.data() + blocks_bytes,
                            m->image.size() - blocks_bytes, hipMemcpyHostToDevice, s));
    const size_t sizes[7] = {(static_cast<size_t>(m->N) + 1) * 4, static_cast<size_t>(m->N) * 8,
                             static_cast<size_t>(nnz) * 4, static_cast<size_t>(nnz) * cb,
                             static_cast<size_t>(nnz) * 2, static_cast<size_t>(nnz) * 2, 4};
    for (int i = 0; i < 7; ++i) GQSA_HIP(hipMalloc(&tmp.p[i], sizes[i] ? sizes[i] : 4));
    GQSA_HIP(hipMemcpyAsync(tmp.p[0], m->rowIndex.data(), sizes[0], hipMemcpyHostToDevice, s));
    GQSA_HIP(hipMemcpyAsync(tmp.p[1], row_pos.data(), sizes[1], hipMemcpyHostToDevice, s));
    GQSA_HIP(hipMemsetAsync(tmp.p[6], 0, 4, s));

    PackArgs a{};
    a.W = W_dev;
    a.hinv = hinv_dev;
    a.rowIndex = static_cast<const int32_t*>(tmp.p[0]);
    a.row_pos = static_cast<const int64_t*>(tmp.p[1]);
    a.groups = static_cast<int32_t*>(tmp.p[2]);
    a.values = static_cast<uint8_t*>(tmp.p[3]);
    a.scales = static_cast<uint16_t*>(tmp.p[4]);
    a.zeros = static_cast<uint16_t*>(tmp.p[5]);
    a.blocks = static_cast<uint8_t*>(img);
    a.status = static_cast<int*>(tmp.p[6]);
    a.K = m->K;
    a.kg = static_cast<int>(m->K / m->G);
    a.bits = m->bits;
    a.cb = cb;
    a.U = m->tile_blocks;
    a.L = m->tile_lanes;
    a.bb = m->block_bytes();
    a.slots_per_group = m->G >= 16 ? m->G / 16 : 1;
    if (hinv_dev)
        hipLaunchKernelGGL(check_hinv_kernel, dim3(static_cast<unsigned>((m->K + kThreads - 1) / kThreads)), dim3(kThreads), 0, s,
                           hinv_dev, static_cast<long long>(m->K), a.status);
    switch (m->G) {
        case 8: launch_pack_rows<8>(a, m->N, s); break;
        case 16: launch_pack_rows<16>(a, m->N, s); break;
        case 32: launch_pack_rows<32>(a, m->N, s); break;
        case 64: launch_pack_rows<64>(a, m->N, s); break;
        case 128: launch_pack_rows<128>(a, m->N, s); break;
        default: return GQSA_ERR_UNSUPPORTED;
    }
    GQSA_HIP(hipGetLastError());
    int status = 0;
    GQSA_HIP(hipMemcpyAsync(&status, tmp.p[6], 4, hipMemcpyDeviceToHost, s));
    if (nnz > 0) {
        GQSA_HIP(hipMemcpyAsync(m->groups.data(), tmp.p[2], sizes[2], hipMemcpyDeviceToHost, s));
        GQSA_HIP(hipMemcpyAsync(m->values.data(), tmp.p[3], sizes[3], hipMemcpyDeviceToHost, s));
        GQSA_HIP(hipMemcpyAsync(m->scales.data(), tmp.p[4], sizes[4], hipMemcpyDeviceToHost, s));
        GQSA_HIP(hipMemcpyAsync(m->zeros.data(), tmp.p[5], sizes[5], hipMemcpyDeviceToHost, s));
    }
    GQSA_HIP(hipMemcpyAsync(m->image.data(), img, blocks_bytes, hipMemcpyDeviceToHost, s));
    GQSA_HIP(hipStreamSynchronize(s));
    if (status != 0) return GQSA_ERR_RANGE;                // non-finite weights, a bad diag(H^-1), or a scale beyond fp16
    // the image is where the GEMV wants it already: the handle takes it over
    if (gqsa_status_t st = device_upload(m, img)) return st;
    guard.p = nullptr;
    return GQSA_OK;
}

}  // namespace gqsa
