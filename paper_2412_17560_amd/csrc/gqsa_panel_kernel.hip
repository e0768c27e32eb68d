// y[b, n] = sum_k W^[n, k] x[b, k] for up to 16 activation rows at once on the matrix cores, from
// the panel image (gqsa_panels.cpp): a panel's groups of one group-column, 16 rows x 16 weights
// with the pruned ones zero, times the 16 x 16 activations under them, is one 16x16x16 product.
// The dequantisation of Eq. 3 stays exact -- no weight is ever rounded to fp16 -- in both forms
// of the kernel (INTZ, chosen per matrix when the image is built):
//   - every stored zero is an integer of at most 1024 in magnitude (what Eq. 1 yields): the zero
//     is taken off the codes in fp16 before the product (q - z is an exact small integer there),
//     the matrix cores multiply it by x with fp32 accumulation, the scale is applied to the sum:
//         sum_j (q_j - z) s x_j  =  s * sum_j (q_j - z) x_j;
//   - any other zero (Sec. 3.4 trains scale and zero freely): the matrix cores multiply the codes
//     q themselves (exact in fp16) by x, a second product with a matrix of ones gives the sum of
//     the 16 activations, and scale and zero are applied to the two fp32 results per group:
//         sum_j (q_j - z) s x_j  =  s * (sum_j q_j x_j  -  z * sum_j x_j).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <type_traits>
#include <utility>

#include "gqsa_internal.hpp"

namespace gqsa {
namespace {

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kPanelsPerQuad = 4;      // panels whose records are staged, and whose headers are held, together
constexpr int kInFlight = 4;          // group-columns whose products are under way together
constexpr int kPanelWaves = 16;      // wavefronts of a workgroup (or 8, see WAVES): each takes every 16th (8th) unit (a run of group-columns) of the panel
constexpr uint32_t kDirectArea = 9216;    // bytes of LDS a wavefront stages records in (16 x 9 KB = 144 of the 160 KB)
constexpr uint32_t kTurnedArea = 8944;    // ... where it turns the activations' loads round as well,
constexpr uint32_t kTurnArea = 1296;      // and in which it does that (together all of the 160 KB)
constexpr int kMaxUnitBytes = 3072;   // records of one panel in one unit, at most (16 rows x the unit's columns)

__device__ __forceinline__ float half_bits_to_float(uint32_t h)
{
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(h)));
}

__device__ __forceinline__ uint16_t float_to_half_bits(float v)
{
    return __builtin_bit_cast(uint16_t, static_cast<_Float16>(v));     // round to nearest even
}

// Four codes -> four fp16 numbers in units of 2^-9, exactly: a code in the low bits of an empty 16-bit half is the fp16 subnormal
// q 2^-24, at bits 4..7 it is q 2^-20, and one fused multiply-add by 2^15 or 2^11 turns either into (q - z) 2^-9 (`off` = -z 2^-9, twice;
// an integer z of at most 1024 in magnitude: every intermediate and the result are integers below 2048 in that unit, so each
// step is exact) -- or, without a zero, into q 2^-9.  The unit travels with the sums and comes off the results, a power of two: the same bits as
// with the plain integers.  (A splice with 1024 in front of the codes, taken off again, took one instruction more for the zero and an AND-OR
// -- 5.3 cycles -- where an AND -- 3 -- is enough.)
// 4-bit: `pair` holds the two bytes (e0 | e2 << 4), (e1 | e3 << 4) in bits 0..7 and 16..23.
constexpr float kUnitInverse = 512.0f;
struct DecodeConstants {
    uint32_t nib_lo, nib_hi;      // 0x000F000F and << 4
    half2_t low, high;            // 2^15 for codes in the low bits, 2^11 at bits 4..7
};
template <bool INTZ>
__device__ __forceinline__ half2_t to_unit(uint32_t codes, half2_t times, half2_t off)
{
    const half2_t q = __builtin_bit_cast(half2_t, codes);
    return INTZ ? __builtin_elementwise_fma(q, times, off) : q * times;
}
template <bool INTZ>
__device__ __forceinline__ half4_t decode4_w4(uint32_t pair, const DecodeConstants& k, half2_t off)
{
    const half2_t a = to_unit<INTZ>(pair & k.nib_lo, k.low, off);
    const half2_t b = to_unit<INTZ>(pair & k.nib_hi, k.high, off);
    return half4_t{a.x, a.y, b.x, b.y};
}
// 8-bit: four bytes, one per element, in the word of the pair (upper, lower) that `sel` names:
// sel = 0x0c010c00 for the lower word, 0x0c050c04 for the upper one.
template <bool INTZ>
__device__ __forceinline__ half4_t decode4_w8(uint32_t upper, uint32_t lower, uint32_t sel, const DecodeConstants& k, half2_t off)
{
    const half2_t a = to_unit<INTZ>(__builtin_amdgcn_perm(upper, lower, sel), k.low, off);                  // bytes 0, 1
    const half2_t b = to_unit<INTZ>(__builtin_amdgcn_perm(upper, lower, sel + 0x00020002u), k.low, off);    // bytes 2, 3
    return half4_t{a.x, a.y, b.x, b.y};
}

// The matrices of a launch: up to four that are multiplied with the same activations (q/k/v,
// gate/up: same K, group size and code width; N may differ).  Their panels are numbered through,
// matrix after matrix, so the panels of a workgroup (blockIdx.x, + gridDim.x, ...) may belong to
// different matrices and still share the activations they load.
// (The images themselves come as separate read-only kernel arguments: the compiler reads a
// block's header with scalar loads only from memory it knows nothing writes to.)
template <int N, typename F, int... I>
__device__ __forceinline__ void for_each_index_of(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
// f(0), f(1), .. f(N - 1), the numbers as compile-time constants
template <int N, typename F>
__device__ __forceinline__ void for_each_index(F&& f)
{
    for_each_index_of<N>(f, std::make_integer_sequence<int, N>{});
}

// How a wavefront gets the activations (see the kernel).
enum class Rows { direct, turned, few };

// few and turned: the records of a unit's panels come in panel by panel, each panel with `pieces` loads (1 to 3), into slots of the staging area
// in turn.  Loads return in the order of issue, so once all but the newest `newer_loads` have, panel pp's are there: those of the panels issued behind
// it.  Two waits serve all cases: for all but three loads, and for all.  (With one for every count that occurs, chosen by comparisons,
// 6318x1024 W8 at 8 rows took 3 % longer, 5916x2048 2 %.)
constexpr int slots_for(int pieces) { return pieces == 1 ? 8 : pieces == 2 ? 4 : 2; }
constexpr int newer_loads(int pp, int n_live, int n_slots, int pieces) { return ((n_live < n_slots + pp ? n_live : n_slots + pp) - 1 - pp) * pieces; }
constexpr int kStillOut = 3;
constexpr int may_be_out(int newer) { return newer < kStillOut ? 0 : kStillOut; }
// The schedule played through: the first panels' loads, then for every panel the wait, its records read, its slot passed on.
constexpr bool records_there_when_read(int panels)
{
    for (int n_live = 1; n_live <= panels; ++n_live) {
        for (int pieces = 1; pieces <= 3; ++pieces) {
            const int n_slots = slots_for(pieces);
            int requested = n_live < n_slots ? n_live : n_slots;        // panels
            for (int pp = 0; pp < n_live; ++pp) {
                const int returned = requested * pieces - may_be_out(newer_loads(pp, n_live, n_slots, pieces));
                if (requested <= pp || returned < (pp + 1) * pieces) return false;
                if (requested < n_live) ++requested;                    // into the slot of panel pp
            }
            if (requested != n_live) return false;
        }
    }
    return true;
}
static_assert(records_there_when_read(8), "a panel's records would be read before they are there");

struct PanelTargets {
    uint16_t* y[kMaxMatricesPerLaunch];
    int N[kMaxMatricesPerLaunch];
    int first[kMaxMatricesPerLaunch];       // panels of the matrices before this one (entries past the last matrix: `total`)
    int total;                  // panels of all matrices
};

// A workgroup takes up to four panels (eight: QUADS) of 16 output rows (blockIdx.x, + gridDim.x, ...); wavefront
// w takes the units w, w + 16, ... (a unit = a run of group-columns, half a slice or less) of
// every one of them, so the activations under a unit are loaded once for all of the workgroup's
// panels.  A block's header is the same for all lanes and is read with scalar loads (turned: the words of the columns; what staging asks of
// all panels comes with one vector load there, and few reads all words that way, see load_ends).  The records
// of a panel in a unit are contiguous in the image; the wavefront copies them from global memory
// straight into its own part of LDS, 1 KiB per instruction with nothing passing through
// registers (direct: all of its panels at once when they fit, else two and two; turned and few: panel after panel, a few ahead), and every lane then
// reads its group's codes, scale and zero from there: which group is a lane's (its row's, in the
// column at hand) follows from the header with a masked population count.  Fetching 8 bytes per
// lane from global memory instead kept 1.5 KB per wavefront under way where this keeps 6 KB.
// No lane reads conditionally: one whose row has no group in a column reads a neighbouring
// record.  More than 8 rows, or G > 16: the next one or the bytes behind the last; whatever it computes from them stays
// in its own column of the product, which it then leaves out.  Two columns a product (few): the record before, or the
// zeros ahead of the first one.  What it decodes from that also enters the sums that another lane of the same output row
// keeps, times the zeros that the activations hold there -- so it has to be finite, which decoded codes always are and
// the zeros are.  The activation rows beyond `batch` are copies of the last one: they only reach result rows
// that are never stored.
// Operands of v_mfma_f32_16x16x16_f16 in a wavefront: lane l holds A[l % 16][4 (l / 16) .. + 3],
// B[4 (l / 16) .. + 3][l % 16] and receives D[4 (l / 16) .. + 3][l % 16].  Here A = the
// activations (row = activation row, 16 elements of one group-column), B = the codes (column =
// output row of the panel), so a lane ends up with the sums of output row l % 16 for the
// activation rows 4 (l / 16) .. + 3 -- and the scale and zero it loaded with its codes are the
// ones those sums need.
// M = 16-element chunks per group (G = 16 M): a group-column then takes M products, chained
// through the accumulator input since they share scale and zero, and a wavefront's unit of work
// is 16 / M group-columns with 4-bit codes, 8 / M with 8-bit codes (so that 16 rows x the unit's
// columns are at most 3 KiB of records).
// INTZ: every zero of the matrix is an integer of at most 1024 in magnitude (what Eq. 1 produces,
// short of extreme groups): the zero is then taken off the codes before the product, exactly, so
// sum_j (q_j - z) x_j comes out of one product and only the scale is left to apply; otherwise the
// zero is an arbitrary fp16 number and multiplies the second product's sum of activations.
// MULTI: more than one matrix in the launch (the lookups of a panel's matrix cost scalar
// registers, which the headers of four panels already fill: one matrix keeps its own code).
// WAVES: 16 wavefronts per workgroup and one workgroup per compute unit, or -- for one matrix of more
// panels than four per compute unit -- 8 and two: the loads of one then run under the products
// of the other (workgroups of 16 wavefronts can only follow one another, each loading, then
// computing).  Either way four wavefronts per SIMD unit, 128 vector registers each.
// QUADS: a workgroup has up to four panels, or eight (direct takes them four at a time -- a quad: their headers share the scalar registers,
// their records the staging area -- turned and few one by one), under the activations of a unit, which are loaded
// once for all of them: every compute unit pulls all of x through its L1 (128 KB at 16 rows and K = 4096, direct at
// about 16 bytes per cycle: 3.4 us, see Rows), so a second workgroup or launch for the panels beyond the fourth
// pays that again.  Two quads against one when they came (direct), at 16 rows, K = 4096, W4 S = 50 %: gate/up of 2 x 11008 in one launch
// instead of two 24.3 -> 22.6 us, 2 x 14336 29.0 -> 25.1 us (W8 33.5 -> 29.4), one matrix of 60000 rows 46.5 -> 43.4 us, 32000 rows
// the same.  (One matrix of 1025 to 2048 panels has at most four for each of its 512 workgroups and never reaches a second quad; what
// it gained, 20000 rows 25.0 -> 18.5 us, 28672x8192 45.4 -> 40.2, came from there being 512 of them where there were 313 and 448.)
template <int BITS, int M, bool INTZ, bool MULTI, int WAVES, int QUADS, Rows ROWS>
__device__ __forceinline__ void panel_products(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ headers0, const uint8_t* __restrict__ data0,
    int K, int n_slices, int batch, int stride, int total,
    const uint8_t* __restrict__ headers1, const uint8_t* __restrict__ headers2, const uint8_t* __restrict__ headers3,
    const uint8_t* __restrict__ data1, const uint8_t* __restrict__ data2, const uint8_t* __restrict__ data3,
    const PanelTargets tgt)
{
    constexpr int CB = 2 * BITS * M;                // code bytes per group
    constexpr bool PAIRED8 = BITS == 8 && M == 1;   // 8-bit, G = 16: quarter 0, word, quarter 1, quarter 2, word, quarter 3
    constexpr int RB = CB + (PAIRED8 ? 8 : 4);      // record: codes of quarters 0, 1 | scale, zero | codes of quarters 2, 3
    constexpr int QB = (BITS / 2) * M;              // code bytes of a lane (one quarter of every chunk)
    constexpr int QW = (QB + 3) / 4;                // ... in registers
    constexpr bool PAIRED = QB == 2;                // 4-bit, G = 16: a 12-byte record, read whole
    // (turned with one matrix: launches of at most as many panels as workgroups, see panels_gemm)
    constexpr bool kOnePanel = !MULTI && ROWS == Rows::turned;
    constexpr int kPanelsPerWorkgroup = kOnePanel ? 1 : QUADS * kPanelsPerQuad;     // at most
    static_assert(!kOnePanel || QUADS == 1, "one panel is less than a quad");
    constexpr int HC = (BITS == 4 ? 16 : 8) / M;    // group-columns of a unit: 16 rows x HC columns x RB bytes <= kMaxUnitBytes
    static_assert(HC >= 1 && HC <= 16 && kPanelRows * HC * RB <= kMaxUnitBytes, "a unit's records must fit their staging area");
    constexpr int XCH = HC * M;                     // 16-element chunks of activations under a unit
    constexpr bool FEW = ROWS == Rows::few, TURNED = ROWS != Rows::direct;
    constexpr int XL = FEW ? XCH / 4 : XCH / 2;     // loads that fetch them: 8 rows of 128 bytes or 16 of 64
    constexpr uint32_t kWaveLds = TURNED ? kTurnedArea : kDirectArea, kTurnLds = TURNED ? kTurnArea : 0;
    static_assert(!FEW || M == 1, "pairs of columns of 16 weights");
    constexpr int UPS = kSliceColumns / HC;         // units per slice
    constexpr int kFly = (INTZ || M > 1) ? kInFlight : 2;      // (two sums per column without INTZ: registers)
    constexpr int FLY = HC < kFly ? HC : kFly;
    constexpr uint32_t kSpare = (RB + 15u) & ~15u;
    static_assert(kSpare + 2 * (kMaxUnitBytes + kSpare) <= kWaveLds, "two panels' worth must fit a wavefront's staging area");
    __shared__ __attribute__((aligned(16))) uint8_t staged[WAVES * (kWaveLds + kTurnLds)];
    float* part = reinterpret_cast<float*>(staged);            // the same memory once the products are done
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wl = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = blockIdx.x;
    const int n_units = UPS * n_slices;

    // the workgroup's panels: wg, wg + stride, ... (stride = the grid's size), each in its matrix; one past the last
    // stands in as the last and is not computed
    const auto locate = [&](int pp, int& m, int& p) {
        const int v = min(wg + pp * stride, total - 1);
        if constexpr (MULTI) {
            // (selects among values at fixed places of the argument block: no load depends on another)
            static_assert(kMaxMatricesPerLaunch == 4, "written out for four matrices");
            const int f1 = tgt.first[1], f2 = tgt.first[2], f3 = tgt.first[3];
            m = (v >= f1 ? 1 : 0) + (v >= f2 ? 1 : 0) + (v >= f3 ? 1 : 0);
            p = v - (m == 0 ? 0 : m == 1 ? f1 : m == 2 ? f2 : f3);
        } else {
            m = 0;
            p = v;
        }
    };
    const auto is_live = [&](int pp) { return wg + pp * stride < total; };     // (the same for the whole workgroup)
    int n_live = 1;             // (the grid has no workgroup without a panel)
#pragma unroll
    for (int pp = 1; pp < kPanelsPerWorkgroup; ++pp) n_live = is_live(pp) ? pp + 1 : n_live;
    const uint32_t panel_headers = static_cast<uint32_t>(n_slices) * kPanelHeaderBytes;
    // What staging asks of a panel is worked out for all panels at once, lanes 4 pp .. 4 pp + 3 for panel pp (with scalar instructions, panel after
    // panel and with a branch at every choice of a matrix, it was 300 of the 500 instructions ahead of the first load), and read out of lane 4 pp.
    // The lanes of panels that the workgroup does not have follow its first one (all workgroups' on the launch's last panel are one line for everybody).
    static_assert(4 * kPanelsPerWorkgroup <= kLanes, "four lanes a panel");
    uint64_t headers_at = 0, data_at = 0;
    if constexpr (ROWS != Rows::direct) {
        int m, p;
        const int pp = (lane >> 2) & (kPanelsPerWorkgroup - 1);
        locate(pp < n_live ? pp : 0, m, p);
        uint64_t h = reinterpret_cast<uint64_t>(headers0), d = reinterpret_cast<uint64_t>(data0);
        if constexpr (MULTI) {
            uint64_t hs[3] = {reinterpret_cast<uint64_t>(headers1), reinterpret_cast<uint64_t>(headers2), reinterpret_cast<uint64_t>(headers3)};
            uint64_t ds[3] = {reinterpret_cast<uint64_t>(data1), reinterpret_cast<uint64_t>(data2), reinterpret_cast<uint64_t>(data3)};
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                asm volatile("" : "+s"(hs[i]), "+s"(ds[i]));       // (read with the first ones, not inside a branch)
                if (m > i) h = hs[i];
                if (m > i) d = ds[i];
            }
        }
        headers_at = h + static_cast<uint64_t>(static_cast<uint32_t>(p)) * panel_headers;
        data_at = d;
    }
    const auto of_lane = [&](uint64_t v, int at) {
        return static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), at))) |
               static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), at))) << 32;
    };
    typedef const __attribute__((address_space(1))) uint8_t* global_bytes;
    typedef const __attribute__((address_space(1))) uint32_t* global_words;
    const auto headers_of = [&](int pp) {         // (of a panel that the workgroup has)
        return MULTI ? of_lane(headers_at, 4 * pp)
                     : reinterpret_cast<uint64_t>(headers0) + static_cast<uint64_t>(static_cast<uint32_t>(wg + pp * stride)) * panel_headers;
    };
    const int r = lane & 15;                        // activation row (A), output row of the panel (B, D)
    const int j = lane >> 4;                        // which four of a group's 16 elements (FEW: which eight of two groups')
    // A unit's header words.  `ends`: of a panel's four lanes the first takes the word of the unit's first column, the second that of the last one,
    // the others the word that says where the block's data start.  Few: also the words of all columns, a vector load per panel (scalar
    // ones arrived up to 3500 cycles later with 16 wavefronts asking): of every 16 lanes lane i takes column 2 i (the lanes 0..31) or 2 i + 1 (32..63).
    const uint32_t ends_lane = (lane & 2) ? kSliceColumns * 4u : (lane & 1) * (HC * 4u - 4u), ends_columns = (lane & 2) ? 0u : ~0u;
    const uint32_t words_lane = 4u * (2 * min(r, HC / 2 - 1) + (j >> 1));
    const auto load_ends = [&](int unit) {
        const uint32_t at = static_cast<uint32_t>(unit / UPS) * kPanelHeaderBytes + ends_lane + ((unit % UPS) * (HC * 4u) & ends_columns);
        return *reinterpret_cast<global_words>(headers_at + at);
    };
    const auto load_words = [&](int pp, int unit) {
        const uint32_t columns = static_cast<uint32_t>(unit / UPS) * kPanelHeaderBytes + (unit % UPS) * (HC * 4u);
        return *reinterpret_cast<global_words>(reinterpret_cast<global_bytes>(headers_of(pp)) + (columns + words_lane));
    };

    // The activations under a unit, once for all panels of the workgroup.
    // direct: of two neighbouring chunks the lanes 0..31 load the first (elements 0-7 and 8-15 of row r), the lanes 32..63 the
    // second, and a swap between the two halves of the wavefront hands every lane the four elements it supplies to a product:
    // elements 0-3, 8-11, 4-7, 12-15 of the chunk for j = 0..3 (which element sits in which of the product's 16 slots does not
    // matter as long as the codes follow suit).  Neighbouring lanes are in different rows, so every lane's 16 bytes are a request
    // of their own, and x arrives at 16 bytes a cycle and compute unit: 3.5 us for 16 rows of 4096.
    // turned: a lane loads 16 bytes of row lane / 4, four lanes next to each other in memory -- 1.2 us for the same rows -- and
    // what it needs of them comes out of a turn through LDS, rows 80 bytes apart there so that the lanes' accesses spread
    // over the banks.  One matrix of one panel a workgroup from 9 to 12 rows on, and most joint launches with G = 16 (see panels_gemm).  (direct / turned, 16 rows,
    // W4 S = 50 %: 1024x4096 7.0 / 6.1 us, 4096x4096 7.9 / 7.2, 2048x8192 12.1 / 10.0, 4096x11008 15.6 / 13.7, G = 64 4096x4096 7.3 / 6.0; one matrix of
    // two panels a workgroup and more is ahead with direct, 8192x11008 19.4 / 20.1: there the wavefronts whose activations arrive first
    // multiply while the others' are on their way.)
    // few (at most 8 activation rows): likewise with eight lanes to a row; elements 8 (j & 1) .. + 7 of row r & 7, of the first column of a
    // pair for j < 2 and r < 8, of the second for j >= 2 and r >= 8, and nothing -- 16 zero bytes -- else.
    constexpr int kRowLanes = FEW ? 8 : 4, kRowStride = FEW ? 144 : 80;
    const int xr = TURNED ? lane / kRowLanes : r, xp = TURNED ? lane % kRowLanes : 2 * (j >> 1) + (j & 1);
    const uint32_t x_lane = static_cast<uint32_t>(min(xr, batch - 1)) * static_cast<uint32_t>(2 * K);      // (bytes: 16 rows of at most 65536)
    const int chunks = K >> 4;
    uint8_t* mine = staged + wl * kWaveLds;                     // this wavefront's staging area
    uint8_t* turn = staged + WAVES * kWaveLds + wl * kTurnLds;
    constexpr int kZeros = 8 * 144;                             // FEW: where the zero bytes are (read at 0 and 64 from here)
    static_assert(!TURNED || (FEW ? kZeros + 80 : 16 * 80) <= kTurnLds, "the turned load must fit its area");
    u32x4_t* turn_in = reinterpret_cast<u32x4_t*>(turn + xr * kRowStride + xp * 16);
    const uint8_t* turn_out = turn + (!FEW ? r * kRowStride + (2 * (j & 1) + (j >> 1)) * 8 : (r < 8) == (j < 2) ? (r & 7) * kRowStride + j * 16 : kZeros);
    if constexpr (FEW) {
        if (lane < 5) *reinterpret_cast<u32x4_t*>(turn + kZeros + 16 * lane) = u32x4_t{0, 0, 0, 0};
    }
    u32x4_t xw[XL];
    const auto load_x = [&](int unit) {
        const int chunk = unit * XCH;
        const uint8_t* xb = reinterpret_cast<const uint8_t*>(x);
        if (chunk + XCH <= chunks) {
            const uint8_t* from = xb + 32 * chunk;
            const uint32_t at = x_lane + 16u * xp;
#pragma unroll
            for (int i = 0; i < XL; ++i) xw[i] = *reinterpret_cast<const u32x4_t*>(from + at + 16 * kRowLanes * i);
        } else {        // the last slice may be short: chunks beyond K -- no groups there -- take the last one's
#pragma unroll
            for (int i = 0; i < XL; ++i) {
                const uint32_t g = min(chunk + (kRowLanes / 2) * i + (xp >> 1), chunks - 1);
                xw[i] = *reinterpret_cast<const u32x4_t*>(xb + (x_lane + (32 * g + 16 * (xp & 1))));
            }
        }
    };

    const uint32_t below = (1u << r) - 1u;
    DecodeConstants dk;
    dk.nib_lo = 0x000F000Fu;
    dk.nib_hi = 0x00F000F0u;
    dk.low = half2_t{(_Float16)32768.0f, (_Float16)32768.0f};
    dk.high = half2_t{(_Float16)2048.0f, (_Float16)2048.0f};
    constexpr _Float16 zero_unit = (_Float16)(-1.0f / kUnitInverse);
    const float4_t zero4 = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr _Float16 kOne = (_Float16)(1.0f / kUnitInverse);
    const half4_t ones = {kOne, kOne, kOne, kOne};
    // a lane supplies elements 0-3, 8-11, 4-7, 12-15 of every chunk for j = 0..3: quarters 0, 2, 1, 3
    const uint32_t quarter = 2u * (j & 1) + (j >> 1);
    const uint32_t code_lane = quarter * QB + (quarter >= 2 ? 4u : 0u);     // where its codes start in a record
    // PAIRED: a lane reads the whole 12-byte record (codes of quarters 0, 1 | scale, zero | codes of
    // quarters 2, 3); a byte permute with a selector that differs by lane puts the lane's two code
    // bytes, from the first or the third word, into bits 0..7 and 16..23
    // PAIRED8: a lane reads the 12 bytes (quarter, scale | zero, quarter) that hold its quarter; the
    // permutes of the decode take the code bytes from the first or the third word
    const uint32_t half_of_record = quarter >= 2 ? 12u : 0u;
    const uint32_t sel_codes = PAIRED8 ? 0x0c010c00u + (quarter & 1u) * 0x00040004u
                                       : 0x0c010c00u + (quarter & 1u) * 0x00020002u + (quarter >= 2 ? 0x00040004u : 0u);

    float acc[kPanelsPerWorkgroup][4];
#pragma unroll
    for (int pp = 0; pp < kPanelsPerWorkgroup; ++pp)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[pp][v] = 0.0f;

    const auto word_of = [&](uint32_t h, int at) { return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(h), at)); };
    // The records of a panel in a unit are contiguous (first group of the first column .. last group of the last column).  Every
    // lane copies 16 bytes per KiB of them, global memory -> LDS directly (lane l's bytes land at the given LDS address + 16 l), no
    // registers.  The panels' records have slots of the staging area in turn, each with room for one more record: few ahead of
    // the first (a lane without a group reads the one before, and before the first one there are zeros), else behind the last.
    // All panels of a unit take as many loads, `pieces` (see records_there_when_read).
    uint32_t span = 0;                  // lane 4 pp: bytes of panel pp's records | where they start in the block << 16,
    uint64_t records_from = 0;          // and where that is
    int pieces = 0, n_slots = 1;
    uint32_t slot_bytes = 0;
    const uint32_t mine_at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t*)mine));
    const auto slot_of = [&](int pp) { return static_cast<uint32_t>(pp & (n_slots - 1)) * slot_bytes + (FEW ? kSpare : 0u); };
    // Piece i of `bytes` bytes.  Lanes past the end are switched off (they would take their cycles) but the first, so that every piece is
    // a load that counts; its address stays inside (the image ends with 256 zero bytes).  The scalar registers of the address may come
    // straight from a v_readlane, and a vector-memory instruction may read those only five wait states later; the compiler sees to that for its
    // own loads but not inside a statement of assembly, so the statement brings the five itself: one a move, three the s_nop (m0 takes one).
    const auto copy = [&](uint32_t to, int i, uint32_t bytes, uint64_t from) {
        const uint32_t o = 16u * lane + 1024u * i;
        const unsigned long long lanes = __builtin_amdgcn_ballot_w64(o < bytes || o == 1024u * i);     // (__ballot takes an int: a select and a second comparison)
        unsigned long long all;
        asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, %4\n\ts_nop 2\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, %0"
                     : "=&s"(all) : "{m0}"(to + 1024u * i), "v"(min(o, (max(bytes, 1u) - 1u) & ~15u)), "s"(from), "s"(lanes) : "memory");
    };
    const auto issue = [&](int pp) {
        const uint64_t from = of_lane(records_from, 4 * pp);
        const uint32_t bytes = word_of(span, 4 * pp) & 0xFFFFu, to = mine_at + slot_of(pp);
#pragma unroll
        for (int i = 0; i < kMaxUnitBytes / 1024; ++i) {
            if (i >= pieces) break;
            copy(to, i, bytes, from);
        }
    };
    // what a unit's headers say, and the loads of its first panels
    const auto begin_unit = [&](uint32_t ends) {
        const auto of_quad = [&](auto ctrl) { return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(ends), decltype(ctrl)::value, 0xF, 0xF, true)); };
        const uint32_t first = (of_quad(std::integral_constant<int, 0x00>{}) >> 16) * RB, last = of_quad(std::integral_constant<int, 0x55>{});
        const uint32_t bytes = ((last >> 16) + __builtin_popcount(last & 0xFFFFu)) * RB - first;     // <= kMaxUnitBytes
        span = bytes | first << 16;
        records_from = data_at + (static_cast<uint64_t>(of_quad(std::integral_constant<int, 0xAA>{})) * 16u + first);
        pieces = __builtin_amdgcn_ballot_w64(bytes > 2048) ? 3 : __builtin_amdgcn_ballot_w64(bytes > 1024) ? 2 : 1;
        slot_bytes = static_cast<uint32_t>(pieces) * 1024u + kSpare;
        n_slots = slots_for(pieces);
        static_assert(8 * (1024 + kSpare) <= kWaveLds && 4 * (2048 + kSpare) <= kWaveLds && 2 * (3072 + kSpare) <= kWaveLds && kMaxUnitBytes == 3072,
                      "the slots must fit a wavefront's staging area");
        // The records go where others lay.  A lane's reads of those must be back first -- the loads into LDS are not
        // ordered against them.
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        for (int pp = 0; pp < min(n_live, n_slots); ++pp) issue(pp);
        if constexpr (FEW) {
            // What a lane without a group multiplies meets the zeros of the other column's activations, so it has to be finite:
            // the record before the first one is zero.
            if (lane < n_slots)
#pragma unroll
                for (uint32_t i = 0; i < kSpare / 16; ++i) *reinterpret_cast<u32x4_t*>(mine + lane * slot_bytes + 16 * i) = u32x4_t{0, 0, 0, 0};
        }
    };
    // waits until the records of panel pp are in LDS
    const auto wait_for = [&](int pp) {
        static_assert(kStillOut == 3, "the wait below");
        if (pp + 1 < kPanelsPerWorkgroup) {
            asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
            if (may_be_out(newer_loads(pp, n_live, n_slots, pieces)) > 0) return;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    // once all of panel pp's records have been read: its slot takes the next panel's
    const auto pass_on = [&](int pp) {
        if (pp + n_slots < n_live) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue(pp + n_slots);
        }
    };

    uint2 xa[HC][M];
    typedef const __attribute__((address_space(3))) uint32_t* lds_words;
    // The products of one panel of a step: its records in LDS, its header words in 16 lanes of h.
    const auto products = [&](float* sums, const uint32_t (&hh)[HC], uint32_t records, auto whole, auto&& all_read) {
        // (sums of eight panels leave registers for the records of eight columns at a time, of four where a column takes two sums)
        constexpr int HL = decltype(whole)::value || BITS == 8 ? HC : HC > 8 ? 8 : !INTZ && HC > 4 ? 4 : HC;
#pragma unroll
        for (int c0 = 0; c0 < HC; c0 += HL) {
        if (c0 > 0) asm volatile("" ::: "memory");
        uint32_t code[HL][(PAIRED || PAIRED8) ? 2 : QW], sz[HL];
        constexpr bool TRI = PAIRED || PAIRED8;     // three words, the middle one is scale | zero as it is: the whole 12-byte
                                                    // record, or the half of the 24-byte one that holds the lane's quarter
#pragma unroll
        for (int c = 0; c < HL; ++c) {
            const uint32_t h = hh[c0 + c];
            const uint32_t at = ((h >> 16) + __builtin_popcount(h & 0xFFFFu & below)) * RB + records;
            if constexpr (TRI) {
                const lds_words w = reinterpret_cast<lds_words>(at);
                code[c][0] = w[0];
                sz[c] = w[1];
                code[c][1] = w[2];
            } else {
                const lds_words w = reinterpret_cast<lds_words>(at + code_lane);
#pragma unroll
                for (int t = 0; t < QW; ++t) code[c][t] = w[t];
                sz[c] = *reinterpret_cast<lds_words>(at + CB / 2);
            }
        }
        // four columns at a time: the products of the later ones are under way while the
        // first one's sums are scaled.  Which lanes have a group in a column is a lane
        // mask made from the header word with scalar arithmetic (bit r -> lanes r, r + 16, ...)
#pragma unroll
        for (int c = 0; c < HL; c += FLY) {
            float4_t d[FLY], e[FLY];
            uint32_t sz_word[FLY];
#pragma unroll
            for (int i = 0; i < FLY; ++i) {
                sz_word[i] = sz[c + i];
                const half2_t both = __builtin_bit_cast(half2_t, sz_word[i]);
                const _Float16 minus_z = both.y * zero_unit;
                const half2_t off = {minus_z, minus_z};
                d[i] = zero4;
                e[i] = zero4;
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    const half4_t a = __builtin_bit_cast(half4_t, xa[c0 + c + i][k]);
                    half4_t q;
                    if constexpr (PAIRED8) {
                        q = decode4_w8<INTZ>(code[c + i][1], code[c + i][0], sel_codes, dk, off);
                    } else if constexpr (PAIRED) {
                        q = decode4_w4<INTZ>(__builtin_amdgcn_perm(code[c + i][1], code[c + i][0], sel_codes), dk, off);   // (same selectors: bytes 0..3 = word 0, 4..7 = word 2)
                    } else if constexpr (BITS == 4) {     // chunk k: two bytes, the lower or the upper half of a word
                        q = decode4_w4<INTZ>(__builtin_amdgcn_perm(0u, code[c + i][k / 2], (k & 1) ? 0x0c030c02u : 0x0c010c00u), dk, off);
                    } else {
                        q = decode4_w8<INTZ>(0u, code[c + i][k], 0x0c010c00u, dk, off);
                    }
                    d[i] = __builtin_amdgcn_mfma_f32_16x16x16f16(a, q, d[i], 0, 0, 0);      // sum_j q_j x_j, or sum_j (q_j - z) x_j
                    if constexpr (!INTZ) e[i] = __builtin_amdgcn_mfma_f32_16x16x16f16(a, ones, e[i], 0, 0, 0);   // sum_j x_j
                }
            }
#pragma unroll
            for (int i = 0; i < FLY; ++i) {
                const unsigned long long lanes = static_cast<unsigned long long>(hh[c0 + c + i] & 0xFFFFu) * 0x0001000100010001ull;
                float sc = half_bits_to_float(sz_word[i] & 0xFFFFu);
                asm volatile("" : "+v"(sc));        // (kept a conversion of its own: an fp32 multiply-add takes 3 cycles, one that converts 5.3: 32000x4096 24.6 -> 24.0 us)
                if (__builtin_amdgcn_inverse_ballot_w64(lanes)) {
                    if constexpr (INTZ) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) sums[v] = __builtin_fmaf(sc, d[i][v], sums[v]);
                    } else {
                        const float z = half_bits_to_float(sz_word[i] >> 16);
#pragma unroll
                        for (int v = 0; v < 4; ++v) sums[v] = __builtin_fmaf(sc, __builtin_fmaf(-z, e[i][v], d[i][v]), sums[v]);
                    }
                }
            }
            if (c == 0 && c0 + HL == HC) all_read();
        }
        }
    };

    // few: at most 8 activation rows, G = 16.  Half of a 16x16x16 product's rows would be copies; instead two columns share a
    // product of 32 elements: A holds the first column's activations in rows 0..7 (zeros where the second's elements are) and
    // the second's in rows 8..15, so the lanes j < 2 end up with the sums of the first column and the lanes j >= 2 with those of
    // the second -- and each lane has read, decoded and scaled the group of its own column only.  The launches are bound by
    // vector instructions (5.3 cycles each with four wavefronts on a SIMD unit, 3 for a plain fp32 multiply-add): per pair of
    // columns 6 for address and presence (the header words stay in a vector register, lane i's is broadcast by the instruction that
    // uses it), 10 (8-bit codes: 9) for the codes, four of them ANDs at 3 cycles, 5 for the scale, where two columns by themselves take 6, 12 and 10;
    // counted over a panel of the compiled joint forms, the passing on of its slot included, 23.6 (8-bit codes 24.2) a pair, and 15.2 (15.5) a column in turned.
    // At 8 rows, W4 S = 50 %, when the form came: 4096x4096 6.9 -> 5.7 us, 3 x 4096x4096 in one launch 13.3 -> 11.3, 2 x 11008x4096 21.2 -> 18.1,
    // 4096x11008 12.4 -> 9.9, 32000x4096 24.0 -> 21.3; W8 4096x4096 7.6 -> 6.1, 2 x 14336x4096 28.0 -> 22.8, 4096x14336 18.1 -> 13.5.
    u32x4_t xp8[FEW ? HC / 2 : 1];
    const auto products_few = [&](float* sums, uint32_t words, uint32_t records, auto whole, auto&& all_read) {
        constexpr int PAIRS = HC / 2;
        constexpr int STEP = INTZ && (QUADS == 1 || BITS == 8) ? 4 : 2;       // pairs under way together (registers)
        // (pairs whose records are held together: with the sums of eight panels there are registers for half of them, with two sums a pair on top for a
        // quarter.  W4, any zeros, 8 rows: all of them, 39 registers spilled among the products, took 3 to 17 % longer than half, and half, with the header words of the
        // last panels spilled, 0 to 5 % longer than a quarter: 20000x4096 S = 30 % 17.2 -> 16.6 us, 2 x 11008x4096 S = 50 % 19.8 -> 19.4, 2 x 16384x4096 23.8 -> 23.2)
        constexpr int HELD = decltype(whole)::value ? PAIRS : INTZ ? PAIRS / 2 : PAIRS / 4;
        const uint32_t upto = (2u << r) - 1u, own = 1u << r;
        const uint32_t before = (words >> 16) * RB + (records - RB + (PAIRED8 ? 12u * (j & 1) : 0u));
        const uint32_t to_codes = 8u * (j & 1);             // 4-bit: codes, scale | zero, codes
        for_each_index<PAIRS / HELD>([&](auto part) {
        constexpr int p0 = decltype(part)::value * HELD;
        if (p0 > 0) asm volatile("" ::: "memory");
        uint32_t code[HELD][BITS / 4], sz[HELD];
        bool present[HELD];
        for_each_index<HELD>([&](auto index) {
            constexpr int i = decltype(index)::value;
            // the header word and the byte offset of lane i of the lane's 16: its column's
            const uint32_t mask = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(words), 0x150 + p0 + i, 0xF, 0xF, true)) & upto;
            const uint32_t at = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(before), 0x150 + p0 + i, 0xF, 0xF, true)) +
                                static_cast<uint32_t>(__builtin_popcount(mask)) * RB;
            present[i] = mask >= own;
            if constexpr (PAIRED8) {
                const uint32_t* w = reinterpret_cast<const uint32_t*>(staged + at);
                code[i][0] = w[0];
                sz[i] = w[1];
                code[i][1] = w[2];
            } else {
                code[i][0] = *reinterpret_cast<const uint32_t*>(staged + (at + to_codes));
                sz[i] = *reinterpret_cast<const uint32_t*>(staged + (at + 4));
            }
        });
#pragma unroll
        for (int i0 = 0; i0 < HELD; i0 += STEP) {
            float4_t d[STEP], e[STEP];
#pragma unroll
            for (int i = 0; i < STEP; ++i) {
                const half2_t both = __builtin_bit_cast(half2_t, sz[i0 + i]);
                const _Float16 minus_z = both.y * zero_unit;
                const half2_t off = {minus_z, minus_z};
                half2_t q[4];
                if constexpr (BITS == 4) {
                    // (bytes e0 | e2 << 4, e1 | e3 << 4, e4 | e6 << 4, e5 | e7 << 4: pairs (e0, e4), (e2, e6), (e1, e5), (e3, e7); the activations follow suit)
                    const uint32_t w = code[i0 + i][0], v = w >> 8;
                    q[0] = to_unit<INTZ>(w & dk.nib_lo, dk.low, off);
                    q[1] = to_unit<INTZ>(w & dk.nib_hi, dk.high, off);
                    q[2] = to_unit<INTZ>(v & dk.nib_lo, dk.low, off);
                    q[3] = to_unit<INTZ>(v & dk.nib_hi, dk.high, off);
                } else {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        q[2 * t] = to_unit<INTZ>(__builtin_amdgcn_perm(0u, code[i0 + i][t * (BITS / 4 - 1)], 0x0c010c00u), dk.low, off);
                        q[2 * t + 1] = to_unit<INTZ>(__builtin_amdgcn_perm(0u, code[i0 + i][t * (BITS / 4 - 1)], 0x0c030c02u), dk.low, off);
                    }
                }
                const half8_t a = __builtin_bit_cast(half8_t, xp8[FEW ? p0 + i0 + i : 0]);
                const half8_t b = {q[0].x, q[0].y, q[1].x, q[1].y, q[2].x, q[2].y, q[3].x, q[3].y};
                d[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, zero4, 0, 0, 0);
                if constexpr (!INTZ) {
                    const half8_t ones8 = {ones.x, ones.x, ones.x, ones.x, ones.x, ones.x, ones.x, ones.x};
                    e[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, ones8, zero4, 0, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < STEP; ++i) {
                float sc = half_bits_to_float(sz[i0 + i] & 0xFFFFu);
                asm volatile("" : "+v"(sc));
                if (present[i0 + i]) {
                    if constexpr (INTZ) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) sums[v] = __builtin_fmaf(sc, d[i][v], sums[v]);
                    } else {
                        const float z = half_bits_to_float(sz[i0 + i] >> 16);
#pragma unroll
                        for (int v = 0; v < 4; ++v) sums[v] = __builtin_fmaf(sc, __builtin_fmaf(-z, e[i][v], d[i][v]), sums[v]);
                    }
                }
            }
            if (i0 == 0 && p0 + HELD == PAIRS) all_read();
        }
        });
    };

    const auto turn_x = [&]() {
        uint2* flat = &xa[0][0];
        if constexpr (!TURNED) {
#pragma unroll
            for (int i = 0; i < XL; ++i) {
                const auto s0 = __builtin_amdgcn_permlane32_swap(xw[i].x, xw[i].z, false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(xw[i].y, xw[i].w, false, false);
                flat[2 * i] = uint2{s0[0], s1[0]};
                flat[2 * i + 1] = uint2{s0[1], s1[1]};
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            // (a wavefront's LDS accesses complete in order: one area serves all of its loads)
            *turn_in = xw[i];
            asm volatile("" ::: "memory");
            if constexpr (FEW) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const u32x4_t w = *reinterpret_cast<const u32x4_t*>(turn_out + 64 * t);
                    if constexpr (BITS == 4)
                        xp8[2 * i + t] = u32x4_t{__builtin_amdgcn_perm(w.z, w.x, 0x05040100u), __builtin_amdgcn_perm(w.w, w.y, 0x05040100u),
                                                 __builtin_amdgcn_perm(w.z, w.x, 0x07060302u), __builtin_amdgcn_perm(w.w, w.y, 0x07060302u)};
                    else
                        xp8[2 * i + t] = w;
                }
            } else {
                flat[2 * i] = *reinterpret_cast<const uint2*>(turn_out);
                flat[2 * i + 1] = *reinterpret_cast<const uint2*>(turn_out + 32);
            }
            asm volatile("" ::: "memory");
        }
    };
    // turned: the header words of the panels' columns, scalar loads -- of a quad's panels at once where they fit the scalar
    // registers (8-bit codes, G > 16), else a panel's when its products start (one latency a panel; asked for ahead of that they are slower yet: while a
    // scalar load is under way every wait for LDS waits for it as well).
    constexpr bool kQuadWords = !FEW && kPanelsPerQuad * HC <= 32;
    uint32_t hh[kQuadWords ? kPanelsPerQuad : 1][FEW ? 1 : HC] = {};
    const auto load_columns = [&](int at, int pp, int unit) {
        const auto from = reinterpret_cast<const __attribute__((address_space(4))) uint32_t*>(
            headers_of(pp) + (static_cast<uint32_t>(unit / UPS) * kPanelHeaderBytes + (unit % UPS) * (HC * 4u)));
#pragma unroll
        for (int c = 0; c < HC; ++c) hh[at][c] = from[c];
    };
    const auto load_quad = [&](int quad, int unit) {
        if constexpr (kQuadWords) {
#pragma unroll
            for (int pp = 0; pp < kPanelsPerQuad; ++pp) {
                if (quad * kPanelsPerQuad + pp >= n_live) break;
                load_columns(pp, quad * kPanelsPerQuad + pp, unit);
            }
        }
    };
    // the products of a panel whose records are in LDS, `records` past the place of the block's first one
    const auto multiply = [&](int pp, int unit, uint32_t words, uint32_t records, auto whole, auto&& arrived, auto&& all_read) {
        if constexpr (FEW) {
            arrived();
            products_few(acc[pp], words, wl * kWaveLds + records, whole, all_read);
        } else {
            if constexpr (!kQuadWords) load_columns(0, pp, unit);
            else if (pp > 0 && pp % kPanelsPerQuad == 0) load_quad(pp / kPanelsPerQuad, unit);
            arrived();
            products(acc[pp], hh[kQuadWords ? pp % kPanelsPerQuad : 0], mine_at + records + (PAIRED8 ? half_of_record : 0u), whole, all_read);
        }
    };
    if constexpr (ROWS == Rows::direct) {
        // direct: the records of a quad (or of two of its panels) are requested and awaited together.  Panel by panel, as below, took up to
        // 14 % longer in this form (4822x4096 G = 128 7.4 -> 8.5 us, 32000x4096 at 16 rows 23.1 -> 23.9).
        for (int unit = wl; unit < n_units; unit += WAVES) {
            const int s = unit / UPS;
            const int sub = unit % UPS;
            load_x(unit);       // (ahead of everything; turned once the records' loads have been issued too)
#pragma unroll
            for (int quad = 0; quad < QUADS; ++quad) {
                int mat[kPanelsPerQuad], pan[kPanelsPerQuad];
                bool live[kPanelsPerQuad];
#pragma unroll
                for (int pp = 0; pp < kPanelsPerQuad; ++pp) {
                    live[pp] = is_live(quad * kPanelsPerQuad + pp);
                    locate(quad * kPanelsPerQuad + pp, mat[pp], pan[pp]);
                }
                if (quad > 0 && !live[0]) break;                // (the same for the whole workgroup)
                // the headers of four panels at once (scalar loads; a panel beyond the
                // last one stands in as the last one and is not computed)
                // (where 4 x HC words do not fit the scalar registers -- AGAIN -- only the first and the
                // last column's word of each panel are read here, and all of a panel's words a second
                // time, from the scalar cache, when its products start)
                constexpr bool AGAIN = kPanelsPerQuad * HC > 32;
                uint32_t hh_all[AGAIN ? 1 : kPanelsPerQuad][AGAIN ? 1 : HC];
                uint32_t header_at[kPanelsPerQuad];        // byte offset of the unit's first word in the panel's matrix's headers
                uint32_t h_first[kPanelsPerQuad], h_last[kPanelsPerQuad], where[kPanelsPerQuad];
#pragma unroll
                for (int pp = 0; pp < kPanelsPerQuad; ++pp) {
                    // (the choice is made here, at the load: a header is read with scalar loads only if the
                    // compiler can trace its address to a read-only argument)
                    const uint8_t* headers = !MULTI || mat[pp] == 0 ? headers0 : mat[pp] == 1 ? headers1 : mat[pp] == 2 ? headers2 : headers3;
                    const uint32_t* header = reinterpret_cast<const uint32_t*>(
                        headers + static_cast<size_t>(pan[pp] * n_slices + s) * kPanelHeaderBytes);
                    header_at[pp] = static_cast<uint32_t>((pan[pp] * n_slices + s) * kPanelHeaderBytes + sub * HC * 4);
                    if constexpr (!AGAIN) {
#pragma unroll
                        for (int c = 0; c < HC; ++c) hh_all[pp][c] = header[sub * HC + c];
                    }
                    h_first[pp] = header[sub * HC];
                    h_last[pp] = header[sub * HC + HC - 1];
                    where[pp] = header[32];
                }
                // Where each panel's records of this unit lie (they are contiguous: first group of the
                // first column .. last group of the last column) and where they go in the wavefront's
                // staging area: one after the other, each rounded up to 16 bytes plus room for one more
                // record (a lane without a group may read the one behind the last).  All four panels are
                // staged at once when they fit, else two and two.
                uint32_t first[kPanelsPerQuad], bytes[kPanelsPerQuad], room[kPanelsPerQuad], slot[kPanelsPerQuad];
#pragma unroll
                for (int pp = 0; pp < kPanelsPerQuad; ++pp) {
                    const uint32_t last = h_last[pp];
                    first[pp] = h_first[pp] >> 16;
                    bytes[pp] = ((last >> 16) + __builtin_popcount(last & 0xFFFFu) - first[pp]) * RB;     // <= kMaxUnitBytes
                    room[pp] = ((bytes[pp] + 15u) & ~15u) + kSpare;
                }
                const bool two_and_two = room[0] + room[1] + room[2] + room[3] > kWaveLds;
                slot[0] = 0;
                slot[1] = room[0];
                slot[2] = two_and_two ? 0 : room[0] + room[1];
                slot[3] = slot[2] + room[2];
#pragma unroll
                for (int pp = 0; pp < kPanelsPerQuad; ++pp) {
                    if (pp == 0 || (pp == 2 && two_and_two)) {
                        // The records go where others lay: panels 0 and 1, the quad before, the unit before.  A lane's
                        // reads of those must be back first -- the loads into LDS are not ordered against
                        // them, and the compiler waits for a value where it is used, which may be further down
                        // (and is, in some of the compiled forms).
                        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                        // stage: every lane copies 16 bytes per KiB of a panel's records, global memory ->
                        // LDS directly (lane l's bytes land at the given LDS address + 16 l), no registers
#pragma unroll
                        for (int q = pp; q < kPanelsPerQuad; ++q) {
                            if (live[q] && (q < pp + 2 || !two_and_two)) {
                                const uint8_t* data = !MULTI || mat[q] == 0 ? data0 : mat[q] == 1 ? data1 : mat[q] == 2 ? data2 : data3;
                                const uint8_t* from = data + static_cast<size_t>(where[q]) * 16 + first[q] * RB;
#pragma unroll
                                for (int i = 0; i < kMaxUnitBytes / 1024; ++i) {
                                    const uint32_t o = 16u * lane + 1024u * i;
                                    if (o < bytes[q])
                                        __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t*>(from + o),
                                                                         (__attribute__((address_space(3))) void*)(mine + slot[q] + 1024u * i),
                                                                         16, 0, 0);
                                }
                            }
                        }
                        if (pp == 0 && quad == 0) turn_x();
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the records are in LDS before any lane reads them
                    }
                    if (live[pp]) {                             // (the same for the whole workgroup)
                        uint32_t hh[HC];
                        if constexpr (!AGAIN) {
#pragma unroll
                            for (int c = 0; c < HC; ++c) hh[c] = hh_all[pp][c];
                        } else {
                            uint32_t at = header_at[pp];
                            asm volatile("" : "+s"(at));            // (a read of its own, not the values kept from above)
                            const uint8_t* headers = !MULTI || mat[pp] == 0 ? headers0 : mat[pp] == 1 ? headers1 : mat[pp] == 2 ? headers2 : headers3;
                            const uint32_t* again = reinterpret_cast<const uint32_t*>(headers + at);
#pragma unroll
                            for (int c = 0; c < HC; ++c) hh[c] = again[c];
                        }
                        products(acc[quad * kPanelsPerQuad + pp], hh, mine_at + slot[pp] - first[pp] * RB + (PAIRED8 ? half_of_record : 0u),
                                 std::bool_constant<QUADS == 1>{}, []() {});
                    }
                }
            }
        }
    } else {
        bool single = kOnePanel;
        if constexpr (!kOnePanel && QUADS == 1) single = n_live == 1;
        if (single) {
            // One panel: while a unit's products are computed, the next one's records and (where there are registers for them) activations
            // are on their way, and the headers of the one behind it, which say where its records are.
            constexpr bool kXAhead = XL <= 4;
            if constexpr (FEW) {        // (the zeros ahead of the first record, see begin_unit)
                if (lane < static_cast<int>(kSpare / 16)) *reinterpret_cast<u32x4_t*>(mine + 16 * lane) = u32x4_t{0, 0, 0, 0};
            }
            constexpr uint32_t kSlot = FEW ? kSpare : 0u;
            const uint64_t data_from = MULTI ? of_lane(data_at, 0) : reinterpret_cast<uint64_t>(data0);
            uint32_t first = 0;
            const auto begin = [&](uint32_t ends) {
                const uint32_t last = word_of(ends, 1);
                first = (word_of(ends, 0) >> 16) * RB;
                const uint32_t bytes = ((last >> 16) + __builtin_popcount(last & 0xFFFFu)) * RB - first;
                const uint64_t from = data_from + (static_cast<uint64_t>(word_of(ends, 2)) * 16u + first);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (as in begin_unit)
#pragma unroll
                for (int i = 0; i < kMaxUnitBytes / 1024; ++i) {
                    if (bytes <= 1024u * i) break;
                    copy(mine_at + kSlot, i, bytes, from);
                }
            };
            int unit = wl;
            uint32_t words = 0, ends_next = 0, words_next = 0;
            const auto of_unit = [&](int u) { return min(u, n_units - 1); };
            if (unit < n_units) {
                const uint32_t ends = load_ends(unit);
                if constexpr (FEW) words = load_words(0, unit);
                load_quad(0, unit);
                __builtin_amdgcn_sched_barrier(0);
                load_x(unit);
                __builtin_amdgcn_sched_barrier(0);
                ends_next = load_ends(of_unit(unit + WAVES));
                if constexpr (FEW) words_next = load_words(0, of_unit(unit + WAVES));
                begin(ends);
                turn_x();
            }
            while (unit < n_units) {
                const bool more = unit + WAVES < n_units;
                uint32_t ends_after = 0, words_after = 0;
                multiply(0, unit, words, kSlot - first, std::bool_constant<!FEW || BITS == 8>{}, [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }, [&]() {
                    if (!more) return;
                    ends_after = load_ends(of_unit(unit + 2 * WAVES));
                    if constexpr (FEW) words_after = load_words(0, of_unit(unit + 2 * WAVES));
                    if (kXAhead) load_x(unit + WAVES);
                    begin(ends_next);
                });
                if (!more) break;
                unit += WAVES;
                load_quad(0, unit);
                if (!kXAhead) load_x(unit);
                words = words_next;
                ends_next = ends_after;
                words_next = words_after;
                turn_x();
            }
        } else {
            // Several: the records of the first panels are on their way while the activations are turned, and those of the later ones while
            // the first ones' products are computed.  The activations are requested ahead of the headers, so they are there when the
            // headers are, and the records' loads, which the headers place, come next: a wait for the activations behind those would be one for the
            // records of all panels.  (For two panels the headers went first for a while, in a copy of their own: shorter by itself, but with both
            // copies in the kernel W4 at 9 to 16 rows kept sums of the eighth panel in memory.)  Before, all of a quad's panels were awaited together: at 16 rows the products of 2 x 11008x4096 began when three
            // quarters of the image had arrived.
            constexpr bool kEndsAhead = INTZ || QUADS == 1;
            int unit = wl;
            uint32_t words[FEW ? kPanelsPerWorkgroup : 1] = {}, ends_next = 0;
            const auto load_all_words = [&](int u) {
                if constexpr (FEW) {
#pragma unroll
                    for (int pp = 0; pp < kPanelsPerWorkgroup; ++pp) {
                        if (pp >= n_live) break;
                        words[pp] = load_words(pp, u);
                    }
                }
            };
            if (unit < n_units) {
                load_x(unit);
                __builtin_amdgcn_sched_barrier(0);
                const uint32_t ends = load_ends(unit);
                if (kEndsAhead) ends_next = load_ends(min(unit + WAVES, n_units - 1));
                load_all_words(unit);
                load_quad(0, unit);
                begin_unit(ends);
                turn_x();
            }
            while (unit < n_units) {
#pragma unroll
                for (int pp = 0; pp < kPanelsPerWorkgroup; ++pp) {
                    if (pp >= n_live) break;
                    multiply(pp, unit, words[FEW ? pp : 0], slot_of(pp) - (word_of(span, 4 * pp) >> 16), std::bool_constant<FEW ? BITS == 8 || QUADS == 1 : BITS == 8>{}, [&]() { wait_for(pp); }, [&]() { pass_on(pp); });
                }
                unit += WAVES;
                if (unit >= n_units) break;
                load_quad(0, unit);
                load_x(unit);
                load_all_words(unit);
                const uint32_t ends = kEndsAhead ? ends_next : load_ends(unit);
                if (kEndsAhead) ends_next = load_ends(min(unit + WAVES, n_units - 1));
                begin_unit(ends);
                turn_x();
            }
        }
    }

    // few: the sums of the first columns are in the lanes j < 2, of the second ones in the lanes 32 further on, for the
    // activation rows 4 (j & 1) .. + 3: added up, both have the rows' sums
    if constexpr (FEW) {
#pragma unroll
        for (int pp = 0; pp < kPanelsPerWorkgroup; ++pp)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint32_t sum = __builtin_bit_cast(uint32_t, acc[pp][v]);
                const auto both = __builtin_amdgcn_permlane32_swap(sum, sum, false, false);
                const uint32_t first = both[0], second = both[1];
                acc[pp][v] = __builtin_bit_cast(float, first) + __builtin_bit_cast(float, second);
            }
    }

    // The wavefronts' sums meet in LDS (the staging areas, once every wavefront is done with its
    // own): all panels' at once, then the wavefronts share out the (panel, accumulator register)
    // pairs: pair t = the activation rows 4 j + (t % 4) of panel t / 4, whose contributions are
    // added in wavefront order and stored.
    static_assert(kPanelsPerWorkgroup * WAVES * 4u * kLanes * sizeof(float) <= sizeof(staged), "the sums must fit the staging areas");
    __syncthreads();
#pragma unroll
    for (int pp = 0; pp < kPanelsPerWorkgroup; ++pp) {
        if (!is_live(pp)) break;
#pragma unroll
        for (int v = 0; v < 4; ++v) part[((pp * 4 + v) * WAVES + wl) * kLanes + lane] = acc[pp][v];
    }
    __syncthreads();
    for (int t = wl; t < 4 * kPanelsPerWorkgroup; t += WAVES) {      // t = (panel, accumulator register)
        const int pp = t >> 2, v = t & 3;
        int m, p;
        if (is_live(pp)) {
            locate(pp, m, p);
            float sum = 0.0f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) sum += part[(t * WAVES + w) * kLanes + lane];
            const int b = 4 * j + v;                    // activation row
            const int row = p * kPanelRows + r;         // output row
            const int n = !MULTI || m == 0 ? tgt.N[0] : m == 1 ? tgt.N[1] : m == 2 ? tgt.N[2] : tgt.N[3];
            uint16_t* y = !MULTI || m == 0 ? tgt.y[0] : m == 1 ? tgt.y[1] : m == 2 ? tgt.y[2] : tgt.y[3];
            if (b < batch && row < n) y[static_cast<size_t>(b) * n + row] = float_to_half_bits(sum * kUnitInverse);
        }
    }
}

// One matrix: the leading parameters, which its first loads depend on, are in scalar registers when a wavefront starts (the file is
// compiled with kernel-argument preloading: 4096x4096 at 8 and 16 rows 6.15 / 7.55 -> 5.9 / 7.3 us).
template <int BITS, int M, bool INTZ, int WAVES, int QUADS, Rows ROWS>
__global__ __launch_bounds__(WAVES * kLanes, 4) void gqsa_panel_kernel(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ headers, const uint8_t* __restrict__ data,
    int K, int n_slices, int batch, int stride, int total, const PanelTargets tgt)
{
    panel_products<BITS, M, INTZ, false, WAVES, QUADS, ROWS>(x, headers, data, K, n_slices, batch, stride, total, nullptr, nullptr, nullptr,
                                                            nullptr, nullptr, nullptr, tgt);
}

// Several: the scalar registers are short, so nothing is preloaded (the structure comes first).
template <int BITS, int M, bool INTZ, int WAVES, int QUADS, Rows ROWS>
__global__ __launch_bounds__(WAVES * kLanes, 4) void gqsa_panel_multi_kernel(
    const PanelTargets tgt, const uint16_t* __restrict__ x,
    const uint8_t* __restrict__ headers0, const uint8_t* __restrict__ headers1,
    const uint8_t* __restrict__ headers2, const uint8_t* __restrict__ headers3,
    const uint8_t* __restrict__ data0, const uint8_t* __restrict__ data1,
    const uint8_t* __restrict__ data2, const uint8_t* __restrict__ data3, int K, int n_slices, int batch, int stride)
{
    panel_products<BITS, M, INTZ, true, WAVES, QUADS, ROWS>(x, headers0, data0, K, n_slices, batch, stride, tgt.total, headers1, headers2, headers3,
                                                           data1, data2, data3, tgt);
}

}  // namespace

#define GQSA_HIP(call)                                                                   \
    do {                                                                                 \
        const hipError_t e_ = (call);                                                    \
        if (e_ != hipSuccess) {                                                          \
            std::fprintf(stderr, "libgqsa: %s: %s\n", #call, hipGetErrorString(e_));    \
            return GQSA_ERR_HIP;                                                         \
        }                                                                                \
    } while (0)

gqsa_status_t panels_upload(gqsa_matrix* m)
{
    if (m->panel_image.empty() || m->d_panels) return GQSA_OK;
    void* img = nullptr;
    GQSA_HIP(hipMalloc(&img, m->panel_image.size()));
    const hipError_t e = hipMemcpy(img, m->panel_image.data(), m->panel_image.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        std::fprintf(stderr, "libgqsa: upload failed: %s\n", hipGetErrorString(e));
        (void)hipFree(img);
        return GQSA_ERR_HIP;
    }
    m->d_panels = img;
    return GQSA_OK;
}

void panels_release(gqsa_matrix* m)
{
    if (m->d_panels) (void)hipFree(m->d_panels);
    m->d_panels = nullptr;
}

// Up to 16 activation rows in one launch, for up to four matrices that share them (same K, group
// size, code width and handling of the zero; the caller checks).  x [batch, K], ys[i] [batch, N_i],
// fp16, on the device.
gqsa_status_t panels_gemm(const gqsa_matrix* const* ms, int n, const void* x, void* const* ys, int batch, void* stream)
{
    if (n < 1 || n > kMaxMatricesPerLaunch || batch < 1 || batch > kPanelRows) return GQSA_ERR_UNSUPPORTED;
    // the images belong to the GPU they were uploaded on
    int dev = -1;
    GQSA_HIP(hipGetDevice(&dev));
    for (int i = 0; i < n; ++i)
        if (ms[i]->device != dev) return GQSA_ERR_HIP;
    PanelTargets tgt{};
    const uint8_t* headers[kMaxMatricesPerLaunch];
    const uint8_t* data[kMaxMatricesPerLaunch];
    int64_t total = 0;
    for (int i = 0; i < n; ++i) {
        const gqsa_matrix* m = ms[i];
        if (!m->d_panels) return GQSA_ERR_UNSUPPORTED;
        if (m->K != ms[0]->K || m->G != ms[0]->G || m->bits != ms[0]->bits || m->n_slices != ms[0]->n_slices ||
            m->panel_integer_zeros != ms[0]->panel_integer_zeros)
            return GQSA_ERR_SHAPE;
        const uint8_t* img = static_cast<const uint8_t*>(m->d_panels);
        headers[i] = img;
        data[i] = img + m->panel_blocks_offset;
        tgt.y[i] = static_cast<uint16_t*>(ys[i]);
        tgt.N[i] = static_cast<int>(m->N);
        tgt.first[i] = static_cast<int>(total);
        total += m->n_panels;
    }
    if (total > INT32_MAX) return GQSA_ERR_SHAPE;
    for (int i = n; i < kMaxMatricesPerLaunch; ++i) {
        tgt.first[i] = static_cast<int>(total);
        headers[i] = headers[0];
        data[i] = data[0];
    }
    tgt.total = static_cast<int>(total);
    const gqsa_matrix* m = ms[0];
    // Up to four panels per compute unit: one workgroup of 16 wavefronts on each.  More panels:
    // workgroups of up to eight (see QUADS) -- with several matrices still one per compute unit (the caller
    // sends no more than eight panels per compute unit this way), with one matrix smaller ones, two
    // to a compute unit (see WAVES; with 16 wavefronts and one per compute unit 20000 and 28672x8192
    // take 2 % longer, 60000 rows 13 %).
    const bool many = total > kPanelsPerQuad * kMaxDefaultWorkgroups;
    const bool halves = many && n == 1;
    const int64_t per_wg = many ? 2 * kPanelsPerQuad : kPanelsPerQuad;
    const int64_t wgs = std::min<int64_t>(total, std::max<int64_t>((halves ? 2 : 1) * kMaxDefaultWorkgroups,
                                                                   (total + per_wg - 1) / per_wg));
    // What the forms are for: see the kernel.  turned takes the same time whatever the rows, direct less with fewer of them (the copies of
    // the last one are one request), so it is the rows that decide.  direct against turned, one matrix of at most 256 panels, S = 50 %, 4096x4096,
    // 4096x11008, 1024x4096 and 2000x8192 (us of 4096x11008, mean of direct / turned over the four):
    //   4-bit codes, G > 16: 3 and 8 rows of G = 64 9.5 / 11.0 and 11.5 / 11.0 (G = 32 9.4 / 11.0 and 11.0 / 11.1, G = 128 8.8 / 10.6 and 11.4 / 10.6); 9 rows
    //     11.4 / 11.0 and 10.9 / 10.7 (G = 64, 32), 1.04 and 1.02; 10 and 11 rows 1.00;
    //   8-bit codes, G > 16: 9, 10, 11 rows of G = 32 11.5 / 12.1, 11.8 / 12.0, 12.0 / 12.1; G = 32 and 64 0.97, 1.00, 1.04;
    //   G = 16, 4-bit codes: 11.7 / 12.1, 11.8 / 12.3, 12.2 / 12.3; 0.97, 0.985, 1.025; 8-bit codes: 13.3 / 13.2, 13.4 / 13.2, 13.4 / 13.2; 0.98, 0.99, 1.00
    //     (1024x4096 5.9 / 6.15, 5.95 / 6.1, 6.0 / 6.1).
    // (The figures of 9 to 11 rows are from when turned was compiled for four panels.  With one it is 2 % faster, and the lines could come down: 8-bit codes of
    // G = 16 at 9, 10, 11 rows 1.02, 1.035, 1.05, 4-bit ones of G = 64 and 128 at 8 rows 1.04 to 1.08.  100 random launches of 9 to 16 rows, G = 16 to 128, S = 0 to
    // 80 %, against the lines of before, 10 and 12 rows: 1.06 times as fast, none slower.)
    // Several matrices of G = 16, 9 rows and more.  Up to one panel a workgroup, and with more than four (direct awaits the records of a whole quad),
    // turned is ahead whatever the rows, the codes and K; with two to four it is x that decides.  direct / turned at S = 50 %, by the units of 16 (8-bit codes:
    // 8) columns that K has, 9 and 16 rows (two matrices, the wavefronts' share of x grows with K up to 16 units, one each):
    //   panels a workgroup        0.3           1.5           3             6
    //   4-bit, 8 units       1.02, 1.13    0.94, 1.01    0.95, 0.99    1.06, 1.09
    //          16 units      1.06, 1.17    0.99, 1.05    1.01, 1.04    1.05, 1.06
    //          24 units      1.01, 1.29    0.94, 1.01    0.95, 1.00    1.04, 1.06
    //   8-bit, 8 units       1.08, 1.09    0.98, 0.99    0.98, 0.98    1.11, 1.09
    //          16 units      1.19, 1.19    1.01, 1.04    1.00, 1.00    1.03, 1.04
    //          24 units      1.16, 1.18    0.99, 1.04    1.04, 1.04    1.09, 1.07
    // (10 to 16 units of 4-bit codes at 12 rows 1.01 to 1.04, 32 and 43 units at 12 and 14 rows 0.95 to 0.99, at 16 rows 0.98 to 1.04; any zeros
    // alike.)  8-bit codes that are hardly pruned, where direct stages two and two because the records of a workgroup's panels do not all fit: 8, 12 and 16 units,
    // four panels, S = 30 % 1.04, 1.15, 1.07, S = 0 1.06, 1.03, 1.02 (4-bit ones 0.96 to 1.04: no rule of their own).
    // 848 launches of two to four panels a workgroup: by this rule 0.74 % faster than direct throughout, the worst 0.95 times as fast, turned throughout 0.17 % slower, the
    // worst 0.93.  Several matrices of larger groups: direct (not compiled in the other form).
    const int unit_columns = m->bits == 4 ? 16 : 8, units = static_cast<int>(m->n_slices) * (kSliceColumns / unit_columns);
    int64_t stored = 0;
    for (int i = 0; i < n; ++i) stored += ms[i]->nnzg();
    // (mean bytes of a panel's records in a unit, G = 16: 12 bytes a 4-bit group, 24 an 8-bit one; nine tenths, as the panels differ)
    const int64_t panel_bytes = stored * (m->bits * 3) * unit_columns / std::max<int64_t>(1, total * (m->K / m->G));
    const bool apart = (total + kMaxDefaultWorkgroups - 1) / kMaxDefaultWorkgroups * panel_bytes * 10 > int64_t{kDirectArea} * 9;
    const bool joint_turned = m->G == 16 && (total <= kMaxDefaultWorkgroups || many ||
                                             (m->bits == 4 ? units > 8 && batch >= (units <= kPanelWaves ? 12 : 15)
                                                           : units > kPanelWaves || (apart && units > 4)));
    const int turned_from = m->bits == 4 && m->G > 16 ? 9 : m->bits == 8 && m->G == 16 ? 12 : 11;
    const bool turns = n > 1 ? joint_turned : total <= kMaxDefaultWorkgroups && batch >= turned_from;
    const Rows rows = batch <= 8 && m->G == 16 ? Rows::few : turns ? Rows::turned : Rows::direct;
    const dim3 grid(static_cast<unsigned>(wgs)), block((halves ? kPanelWaves / 2 : kPanelWaves) * kLanes);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // run(bits, chunks per group, integer zeros) for the format at hand
    const auto pick = [&](auto run) {
        using std::integral_constant;
        const auto with = [&](auto bits, auto chunks) {
            if (m->panel_integer_zeros) run(bits, chunks, std::true_type{});
            else run(bits, chunks, std::false_type{});
        };
        const integral_constant<int, 4> four{};
        const integral_constant<int, 8> eight{};
        switch (m->bits * 1000 + m->G) {
            case 4016: with(four, integral_constant<int, 1>{}); break;
            case 4032: with(four, integral_constant<int, 2>{}); break;
            case 4064: with(four, integral_constant<int, 4>{}); break;
            case 4128: with(four, integral_constant<int, 8>{}); break;
            case 8016: with(eight, integral_constant<int, 1>{}); break;
            case 8032: with(eight, integral_constant<int, 2>{}); break;
            case 8064: with(eight, integral_constant<int, 4>{}); break;
            default: return false;
        }
        return true;
    };
    const auto launch = [&](auto multi, auto waves, auto quads) {
        constexpr int kWaves = decltype(waves)::value, kQuads = decltype(quads)::value;
        constexpr bool kMulti = decltype(multi)::value;
        return pick([&](auto bits, auto chunks, auto integer_zeros) {
            constexpr int kBits = decltype(bits)::value, kChunks = decltype(chunks)::value;
            constexpr bool kInteger = decltype(integer_zeros)::value;
            const auto go = [&](auto how) {
                constexpr Rows kRows = decltype(how)::value;
                if constexpr (kMulti)
                    hipLaunchKernelGGL((gqsa_panel_multi_kernel<kBits, kChunks, kInteger, kWaves, kQuads, kRows>), grid, block, 0, s, tgt,
                                       static_cast<const uint16_t*>(x), headers[0], headers[1], headers[2], headers[3], data[0], data[1],
                                       data[2], data[3], static_cast<int>(m->K), static_cast<int>(m->n_slices), batch, static_cast<int>(wgs));
                else
                    hipLaunchKernelGGL((gqsa_panel_kernel<kBits, kChunks, kInteger, kWaves, kQuads, kRows>), grid, block, 0, s,
                                       static_cast<const uint16_t*>(x), headers[0], data[0], static_cast<int>(m->K),
                                       static_cast<int>(m->n_slices), batch, static_cast<int>(wgs), tgt.total, tgt);
            };
            // (only the forms that `rows` can be are compiled)
            if constexpr (kChunks == 1) {
                if (rows == Rows::few) return go(std::integral_constant<Rows, Rows::few>{});
            }
            if constexpr (kMulti ? kChunks == 1 : kQuads == 1) {
                if (rows == Rows::turned) return go(std::integral_constant<Rows, Rows::turned>{});
            }
            if constexpr (!(kMulti && kChunks == 1 && kQuads == 2)) go(std::integral_constant<Rows, Rows::direct>{});
        });
    };
    using Whole = std::integral_constant<int, kPanelWaves>;
    using Half = std::integral_constant<int, kPanelWaves / 2>;
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    const bool ok = n > 1 ? (many ? launch(std::true_type{}, Whole{}, Two{}) : launch(std::true_type{}, Whole{}, One{}))
                          : (many ? launch(std::false_type{}, Half{}, Two{}) : launch(std::false_type{}, Whole{}, One{}));
    if (!ok) return GQSA_ERR_UNSUPPORTED;
    GQSA_HIP(hipGetLastError());
    return GQSA_OK;
}

}  // namespace gqsa
