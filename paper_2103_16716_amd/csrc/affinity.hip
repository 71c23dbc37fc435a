// Token-expert affinity S = H . W^T (Sec. 3.1, Eq. 2), S[t, e] = h_t . w_e.
//
// Both element types run on the CDNA4 matrix cores with fp32 accumulation:
// bf16 on v_mfma_f32_32x32x16_bf16 / 16x16x32_bf16, fp32 on
// v_mfma_f32_32x32x2_f32 / 16x16x4_f32 (full fp32 products and sums). The
// contraction dimension is the model dimension d, contiguous in both H and W.
// At every shape of interest the bf16 product is bound by reading H (about
// E / (1 + 2E/d) flop per byte), so H is streamed from HBM once, W (at most a few
// MiB) is re-read from L2, and the kernels are organised around keeping
// enough reads in flight.
//
// Two kernels, each for both types:
//   affinity_pipe_kernel   BM tokens x BN experts per block; chunks of 128
//                          bytes of a row of both operands go straight from
//                          global memory into a ring of LDS stages
//   affinity_small_kernel  32 x 32 or 32 x 64 outputs per block, whose waves split d:
//                          problems with too few outputs to give every
//                          compute unit a tile of the pipelined kernel
//
// Every kernel can read H through a row index (`rows`, null for the
// identity): output row i is then h_{rows[i]} . W^T. This is the random
// shuffle of tokens to workers (Sec. 3.2.1, Shuffling) folded into the GEMM's
// loads, so the shuffled copy of H is never written. An index outside
// [0, h_rows) gives a zero row (memory-safe; not a valid shuffle).
#include <mutex>

#include "common.hpp"
#include "internal.hpp"

namespace base {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

#define BASE_LDS __attribute__((address_space(3)))

// 16 bytes of a row per lane, the unit of every load and matrix operand.
// Contracting one unit of A and B per lane takes kMma instructions: bf16 one
// over the lanes' 8 elements; fp32 four, instruction i over the lanes' element
// i (the order of the contraction index is free as long as A and B agree).
// Callers run instruction i over all their tiles before i + 1, so that no
// instruction waits for the one before it.
struct Bf16 {
    using elem_t = uint16_t;
    using unit_t = bf16x8_t;
    static constexpr int kPer = 8;   // elements per unit
    static constexpr int kMma = 1;
    __device__ static f32x16_t mma32(unit_t a, unit_t b, f32x16_t c, int) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    __device__ static f32x4_t mma16(unit_t a, unit_t b, f32x4_t c, int) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
struct F32 {
    using elem_t = float;
    using unit_t = f32x4_t;
    static constexpr int kPer = 4;
    static constexpr int kMma = 4;
    __device__ static f32x16_t mma32(unit_t a, unit_t b, f32x16_t c, int i) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], c, 0, 0, 0);
    }
    __device__ static f32x4_t mma16(unit_t a, unit_t b, f32x4_t c, int i) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], c, 0, 0, 0);
    }
};

__device__ inline int64_t source_row(const int32_t *rows, int64_t h_rows, int i) {
    if (rows == nullptr) return i;
    const int64_t r = rows[i];
    return (r >= 0 && r < h_rows) ? r : -1;
}

// Whether S rows t0 + step(0), ..., t0 + step(N - 1) have a source row in range:
// bit i of the result. Rows past T repeat the last one, so that the N loads
// are issued together; a test at each store made every one wait for its own
// load or branch (a call in bf16, 6000 x 100 x 1000: 12.1 us, then 10.4; 40379 x
// 26 x 232 through an index: 9.9, then 9.1).
template <int N, class Step>
__device__ inline uint32_t rows_in_range(const int32_t *rows, int64_t h_rows, int t0, int T,
                                         Step step) {
    if (rows == nullptr) return ~0u;
    uint32_t ok = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int t = t0 + step(i);
        const int64_t r = rows[t < T ? t : T - 1];
        ok |= (uint32_t)(r >= 0 && r < h_rows) << i;
    }
    return ok;
}

// The grid is one-dimensional. Blocks go to the eight XCDs in turn (block L
// to XCD L % 8); the nn expert tiles of a token tile are placed on one XCD
// one after another (the same L % 8, consecutive L / 8), so that the token
// tile's rows of H come from memory once and from that XCD's L2 for the other
// expert tiles. With one expert tile this is the identity.
__device__ inline void tile_of(int L, int nn, int &mt, int &nt) {
    const int u = L >> 3;
    mt = (u / nn) * 8 + (L & 7);
    nt = u % nn;
}

// --------------------------------------------------------- pipelined GEMM --

// Waits until at most N vector-memory operations of this wave are in flight
// (the LDS-direct loads count until their data is in LDS) and its LDS reads
// are done: the stage they read is refilled after the barrier that follows.
template <int N>
__device__ inline void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt field");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

// Workgroup barrier with no memory wait of its own: each wave has already
// waited for the loads the barrier publishes. The empty asm statements keep
// the compiler from moving memory accesses across it.
__device__ inline void bare_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A block of BM tokens x BN experts, a wave for every TM x TN of its 32 x 32
// tiles, kSt stages of one 128-byte chunk of each row of both operands
// (64 bf16 or 32 fp32 elements), kSt - 1 chunks ahead of the one being
// multiplied. A 16-byte slot s of an LDS row r holds the row's unit
// s ^ (r % 8), so that the operand reads (eight rows per 128-byte row group)
// fall on distinct banks.
//
// Token tile mt starts at chunk mt % nk and goes round. Without that, all
// blocks read the same 128 bytes of every row at about the same time, and with
// row strides that are powers of two those fall on few memory channels. H is
// read once, so its loads are marked non-temporal where that pays (kNt, see
// kStreamFrom) and leave the L2 to W.
// T = 32768, E = 128, d = 2048: 39.8 us before, 36.2 with the rotation,
// 31.5 with both (4.8 TB/s); T = 65536, d = 4096, E = 32: 83 us, 118 without the
// rotation. The rotation gives a row's sum an order that depends on
// its tile. Sums of two or four parts, each always in the same order and added in
// the same order, would not: they need the parts' registers, and at the same
// sizes took 41-44 and 90-120 us.
constexpr int kChunk = 128;          // bytes of a row per stage
constexpr int kUnits = kChunk / 16;
constexpr int kNonTemporal = 2;      // cache policy bit of the LDS-direct load

__device__ const uint4 zero_unit = {0, 0, 0, 0};

template <class In, int BM, int BN, int TM, int TN, int kSt, bool kNt>
__global__ __launch_bounds__(64 * (BM / (32 * TM)) * (BN / (32 * TN))) void affinity_pipe_kernel(
    const typename In::elem_t *__restrict__ H, const int32_t *__restrict__ rows, int64_t h_rows,
    const typename In::elem_t *__restrict__ W, float *__restrict__ S, int T, int E, int d) {
    using unit_t = typename In::unit_t;
    constexpr int kWm = BM / (32 * TM), kWn = BN / (32 * TN);
    constexpr int kThreads = 64 * kWm * kWn;
    constexpr int kSa = BM * kUnits / kThreads, kSb = BN * kUnits / kThreads;
    constexpr int kStage = (BM + BN) * kChunk;
    constexpr int kPK = kUnits * In::kPer;   // elements of d per chunk
    static_assert(kThreads % 64 == 0 && (kThreads / 8) % 8 == 0 && kSa > 0 && kSb > 0, "tile");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    int mt, nt;
    tile_of(blockIdx.x, (E + BN - 1) / BN, mt, nt);
    if ((int64_t)mt * BM >= T) return;   // padding of the grid to whole groups of eight
    const int m0 = mt * BM;
    const int n0 = nt * BN;
    // This thread's 16-byte slots of each operand's chunk: slot q = i *
    // kThreads + tid is row q / 8, position q % 8, and holds the row's unit
    // (q % 8) ^ (row % 8), the same unit cu for every i. Rows past T or E, and
    // invalid source rows, read a valid row; their outputs are not stored
    // (or stored as zero).
    const int cu = (tid % kUnits) ^ ((tid / kUnits) & 7);
    const int wm = wave % kWm;
    const int wn = wave / kWm;
    const int lrow = lane & 31;
    const int lhalf = lane >> 5;
    // 32x32 accumulator layout: lane holds column lane % 32; register i holds
    // row 8 (i / 4) + 4 (lane / 32) + i % 4. The checks of a wave's 32 rows are
    // loaded here, beside the other indices, and not between the last product
    // and its store (64 x 64 tiles, 300000 x 8 x 16 through an index: 20.1 us, 17.0
    // this way; with 64 rows a wave it is 19.0 and 20.9).
    const auto step = [](int i) { return 8 * (i >> 2) + (i & 3); };
    const auto checks = [&](int x) {
        return rows_in_range<16>(rows, h_rows, m0 + 32 * (wm * TM + x) + 4 * lhalf, T, step);
    };
    const uint32_t early = TM == 1 ? checks(0) : 0u;
    const typename In::elem_t *ga[kSa], *gb[kSb];
#pragma unroll
    for (int i = 0; i < kSa; ++i) {
        const int r = (i * kThreads + tid) / kUnits;
        int64_t hr = m0 + r < T ? source_row(rows, h_rows, m0 + r) : 0;
        if (hr < 0) hr = 0;
        ga[i] = H + hr * d + cu * In::kPer;
    }
#pragma unroll
    for (int i = 0; i < kSb; ++i) {
        const int r = (i * kThreads + tid) / kUnits;
        const int er = n0 + r < E ? n0 + r : E - 1;
        gb[i] = W + (int64_t)er * d + cu * In::kPer;
    }
    const int nk = kSt == 1 ? 1 : (d + kPK - 1) / kPK;
    const int rot = mt % nk;
    auto chunk_of = [&](int kc) { return kc + rot < nk ? kc + rot : kc + rot - nk; };
    auto issue = [&](int kc, int st) {
        BASE_LDS unsigned char *base = (BASE_LDS unsigned char *)lds + st * kStage;
        const int64_t k = (int64_t)chunk_of(kc) * kPK;
        // Units past d (last chunk, d not a multiple of the chunk) are zero.
        const bool in = k + cu * In::kPer < d;
#pragma unroll
        for (int i = 0; i < kSa; ++i)
            __builtin_amdgcn_global_load_lds(
                in ? (const void *)(ga[i] + k) : (const void *)&zero_unit,
                (BASE_LDS void *)(base + (i * kThreads + wave * 64) * 16), 16, 0,
                kNt ? kNonTemporal : 0);
#pragma unroll
        for (int i = 0; i < kSb; ++i)
            __builtin_amdgcn_global_load_lds(
                in ? (const void *)(gb[i] + k) : (const void *)&zero_unit,
                (BASE_LDS void *)(base + BM * kChunk + (i * kThreads + wave * 64) * 16), 16, 0, 0);
    };
    f32x16_t acc[TM][TN];
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[x][j][i] = 0.0f;
    if (kSt == 1) issue(0, 0);
#pragma unroll
    for (int st = 0; st < kSt - 1; ++st)
        if (st < nk) issue(st, st);
    int st = 0;
    for (int kc = 0; kc < nk; ++kc) {
        // Chunk kc has landed once at most the later chunks' loads are in
        // flight; after the barrier every wave's part of it is in LDS and
        // every wave is done with the stage refilled next.
        if (kSt > 1 && kc + kSt - 2 < nk) wait_vmcnt<(kSa + kSb) * (kSt > 1 ? kSt - 2 : 0)>();
        else wait_vmcnt<0>();
        bare_barrier();
        if (kSt > 1 && kc + kSt - 1 < nk) issue(kc + kSt - 1, st == 0 ? kSt - 1 : st - 1);
        const unsigned char *A = lds + st * kStage;
        const unsigned char *B = A + BM * kChunk;
        st = st + 1 < kSt ? st + 1 : 0;
        // Two units of every row per step, one per half wave.
#pragma unroll
        for (int ks = 0; ks < kUnits / 2; ++ks) {
            if (kSt == 1 && 2 * ks * In::kPer >= d) break;   // (the rest holds zeros)
            const int c = 2 * ks + lhalf;
            unit_t a[TM];
#pragma unroll
            for (int x = 0; x < TM; ++x) {
                const int ra = 32 * (wm * TM + x) + lrow;
                a[x] = *reinterpret_cast<const unit_t *>(A + ra * kChunk + ((c ^ (ra & 7)) * 16));
            }
            unit_t b[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int rb = 32 * (wn * TN + j) + lrow;
                b[j] = *reinterpret_cast<const unit_t *>(B + rb * kChunk + ((c ^ (rb & 7)) * 16));
            }
#pragma unroll
            for (int i = 0; i < In::kMma; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int x = 0; x < TM; ++x) acc[x][j] = In::mma32(a[x], b[j], acc[x][j], i);
        }
    }
#pragma unroll
    for (int x = 0; x < TM; ++x) {
        const int t0 = m0 + 32 * (wm * TM + x) + 4 * lhalf;
        const uint32_t ok = TM == 1 ? early : checks(x);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int e = n0 + 32 * (wn * TN + j) + lrow;
            if (e >= E) continue;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int t = t0 + step(i);
                if (t < T) S[(int64_t)t * E + e] = (ok >> i & 1) != 0 ? acc[x][j][i] : 0.0f;
            }
        }
    }
}

// ---------------------------------------------------------- small problems --
//
// A block owns 32 tokens x 16 NJ experts (2 x NJ tiles of 16 x 16) and its
// kSWaves waves split d: wave w takes a contiguous run of the 64-byte steps
// of a row, loading its matrix operands straight from memory (a load
// instruction covers 16 rows x 64 bytes; two register sets of kSU steps in
// flight). The waves' partial tiles are added in LDS in wave order (a fixed
// order: the result does not depend on scheduling), NJ / 2 tiles per wave.
// Bound by the loads' latency, with two short register sets in flight (fp32,
// 8192 x 64 x 1024: a compute unit draws 9 bytes a clock from the L2, 62 TFLOP/s),
// so 64 experts a block where there are blocks enough, which load a quarter
// less per output: 17.6 us against 21.5 at 32 experts.
constexpr int kST = 32;
constexpr int kSWaves = 4;

template <class In, int NJ>
__global__ __launch_bounds__(64 * kSWaves) void affinity_small_kernel(
    const typename In::elem_t *__restrict__ H, const int32_t *__restrict__ rows, int64_t h_rows,
    const typename In::elem_t *__restrict__ W, float *__restrict__ S, int T, int E, int d) {
    using unit_t = typename In::unit_t;
    constexpr int kStep = 4 * In::kPer;   // elements of a row per step
    constexpr int kSU = NJ == 2 ? 4 : 2;  // steps per register set
    __shared__ f32x4_t red[kSWaves][2 * NJ][64];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int lrow = lane & 15;
    const int lq = lane >> 4;
    int mt, nt;
    tile_of(blockIdx.x, (E + 16 * NJ - 1) / (16 * NJ), mt, nt);
    if ((int64_t)mt * kST >= T) return;
    const int m0 = mt * kST;
    const int n0 = nt * 16 * NJ;
    // Operand rows: tokens m0 + 16 x + lane % 16, experts n0 + 16 j + lane %
    // 16; lane / 16 picks the unit of the step.
    const int steps = (d + kStep - 1) / kStep;
    const int q = (steps + kSWaves - 1) / kSWaves;   // steps per wave
    const int s0 = wave * q;
    const int s1 = s0 + q < steps ? s0 + q : steps;
    const typename In::elem_t *pa[2], *pb[NJ];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int t = m0 + 16 * x + lrow;
        int64_t hr = t < T ? source_row(rows, h_rows, t) : 0;
        if (hr < 0) hr = 0;
        pa[x] = H + hr * d + lq * In::kPer;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int e = n0 + 16 * j + lrow;
        pb[j] = W + (int64_t)(e < E ? e : E - 1) * d + lq * In::kPer;
    }
    f32x4_t acc[2][NJ];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[x][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    unit_t a[2][kSU][2], b[2][kSU][NJ];
    auto load = [&](int set, int s) {
#pragma unroll
        for (int u = 0; u < kSU; ++u) {
            if (s + u < s1) {   // (uniform)
                const int64_t k = (int64_t)(s + u) * kStep;
                // (units past d, in the last step only, are zero)
                const bool in = k + lq * In::kPer < d;
#pragma unroll
                for (int x = 0; x < 2; ++x)
                    a[set][u][x] = *reinterpret_cast<const unit_t *>(
                        in ? (const void *)(pa[x] + k) : (const void *)&zero_unit);
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    b[set][u][j] = *reinterpret_cast<const unit_t *>(
                        in ? (const void *)(pb[j] + k) : (const void *)&zero_unit);
            }
        }
    };
    auto mma = [&](int set, int s) {
#pragma unroll
        for (int u = 0; u < kSU; ++u)
            if (s + u < s1) {
#pragma unroll
                for (int i = 0; i < In::kMma; ++i)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            acc[x][j] = In::mma16(a[set][u][x], b[set][u][j], acc[x][j], i);
            }
    };
    load(0, s0);
    for (int s = s0; s < s1; s += 2 * kSU) {
        load(1, s + kSU);
        mma(0, s);
        load(0, s + 2 * kSU);
        mma(1, s + kSU);
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int j = 0; j < NJ; ++j) red[wave][NJ * x + j][lane] = acc[x][j];
    __syncthreads();
    static_assert(kSWaves == 4, "NJ / 2 tiles per wave below");
#pragma unroll
    for (int r = 0; r < NJ / 2; ++r) {
        const int tile = wave * (NJ / 2) + r;
        f32x4_t sum = red[0][tile][lane];
#pragma unroll
        for (int w = 1; w < kSWaves; ++w) sum += red[w][tile][lane];
        // 16x16 accumulator layout: lane holds column lane % 16; register i
        // holds row 4 (lane / 16) + i.
        const int e = n0 + 16 * (tile % NJ) + lrow;
        if (e >= E) continue;
        const int t0 = m0 + 16 * (tile / NJ) + 4 * lq;
        const uint32_t ok = rows_in_range<4>(rows, h_rows, t0, T, [](int i) { return i; });
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (t0 + i < T) S[(int64_t)(t0 + i) * E + e] = (ok >> i & 1) != 0 ? sum[i] : 0.0f;
    }
}

template <class In, int BM, int BN, int TM, int TN, int kSt, bool kNt>
hipError_t launch_pipe_as(const typename In::elem_t *H, const int32_t *rows, int64_t h_rows,
                       const typename In::elem_t *W, float *S, int64_t T, int64_t E, int64_t d,
                       hipStream_t stream) {
    constexpr size_t kLds = (size_t)kSt * (BM + BN) * kChunk;
    constexpr int kThreads = 64 * (BM / (32 * TM)) * (BN / (32 * TN));
    const auto kernel = &affinity_pipe_kernel<In, BM, BN, TM, TN, kSt, kNt>;
    // The LDS ring is above the default 64 KiB: opted in once per device.
    static std::mutex m;
    static bool granted[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    {
        std::lock_guard<std::mutex> lock(m);
        if (!granted[dev]) {
            const hipError_t err =
                hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
            if (err != hipSuccess) return err;
            granted[dev] = true;
        }
    }
    const int64_t nm8 = ((T + BM - 1) / BM + 7) / 8 * 8;   // token tiles, whole eights
    const int64_t nn = (E + BN - 1) / BN;
    // Rows of fewer chunks than the ring has stages fill only the first ones:
    // the LDS left lets more blocks share a compute unit (100000 x 128 x 64 in
    // bf16: 15.2 us with the whole ring, 12.3).
    constexpr int kPK = kUnits * In::kPer;
    const int64_t nk = (d + kPK - 1) / kPK;
    const size_t bytes = kLds / kSt * (size_t)(nk < kSt ? nk : kSt);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(nm8 * nn)), dim3(kThreads), bytes, stream, H, rows,
                       h_rows, W, S, (int)T, (int)E, (int)d);
    return hipGetLastError();
}

// H of so many bytes and more is loaded non-temporally; a smaller one stays in
// the last-level cache for the permute that reads it next. Affinity and then
// permute in us, H just written / other data written since, so marked and not
// (bf16, d = 2048; 512 MiB: E = 256, d = 4096): 32 MiB 37 / 37 and 34 / 34; 64 MiB 56 /
// 53 and 49 / 57; 128 MiB 94 / 83 and 81 / 100; 256 MiB 153 / 145 and 154 / 177; 512
// MiB 328 / 329 and 317 / 317, of which the affinity 149 and 157.
constexpr int64_t kStreamFrom = (int64_t)48 << 20;

template <class In, int BM, int BN, int TM, int TN, int kSt>
hipError_t launch_pipe(const typename In::elem_t *H, const int32_t *rows, int64_t h_rows,
                       const typename In::elem_t *W, float *S, int64_t T, int64_t E, int64_t d,
                       hipStream_t stream) {
    const int64_t bytes = T * d * (int64_t)sizeof(typename In::elem_t);
    if constexpr (kSt > 1)   // (not tiles of a single chunk)
        if (bytes >= kStreamFrom)
            return launch_pipe_as<In, BM, BN, TM, TN, kSt, true>(H, rows, h_rows, W, S, T, E, d,
                                                                 stream);
    return launch_pipe_as<In, BM, BN, TM, TN, kSt, false>(H, rows, h_rows, W, S, T, E, d, stream);
}

// The choice of tile. A product in BM x BN tiles takes about
// ceil(tiles / 256) turns of the 256 compute units, each as long as one tile's
// chunk of d times the chunks, so the rule takes the tile with the lowest
// turns * (time of a chunk); ties go to the earlier entry, the larger tile,
// which reads less. Measured microseconds per chunk with one tile on every
// compute unit (bf16: 64 elements a chunk; T x E x d in brackets):
//   256 x 256  2.4  (65536 x 256 x 4096: 155 us, 128 x 128 tiles 209)
//   256 x 128  1.55 (65536 x 128 x 2048: 52 us, 128 x 128 tiles 68)
//   256 x 64   1.07 (65536 x 64 x 1024: 29 us, 128 x 128 tiles 35)
//   128 x 128  1.05 (32768 x 128 x 2048: 33 us, 256 x 128 tiles 41)
//   128 x 64   0.66 (16384 x 128 x 2048: 21 us, 128 x 128 tiles 27)
//   64 x 64    0.46 (8192 x 128 x 2048: 17 us, 128 x 64 tiles 20)
//   32 x 64    0.42 (4096 x 128 x 2048: 14 us, 64 x 64 tiles 16, 32 x 32 17.5)
//   32 x 32    0.30 (2048 x 128 x 2048: 10 us, 64 x 64 tiles 16)
// Blocks of the small kernel share a compute unit, so turns after the first
// cost it a fifth less (bf16; 8192 x 128 x 2048 in 32 x 32: 31 us). Rows that
// are not whole 128-byte lines make the pipelined chunks span two (40379 x 26 x
// 232 in bf16: 256 x 64 tiles 9.9 us, 32 x 32 7.1), which costs the ones of one
// or two chunks less than the small kernel's turns (100003 x 33 x 40 in fp32: 32
// x 64 tiles 17.0 us, 256 x 64 16.0).
// fp32 is bound by the matrix cores at the larger tiles (32 elements a chunk;
// 65536 x 256 x 2048: 531 us, 130 TFLOP/s; 8192 x 64 x 1024: 17.6 us against 64
// on the vector units). Its 256 x 256 and 128 x 128 tiles are never the
// faster ones and not built.
struct TileCost {
    int bm, bn;
    double bf16, f32;
};
constexpr TileCost kTiles[] = {{256, 256, 2.4, 1e30}, {256, 128, 1.55, 4.1}, {256, 64, 1.07, 2.27},
                               {128, 128, 1.05, 1e30}, {128, 64, 0.66, 1.25}, {64, 64, 0.46, 0.75},
                               {kST, 64, 0.42, 0.44}, {kST, 32, 0.30, 0.32}};
constexpr int64_t kComputeUnits = 256;

constexpr int kOneChunk = 8;   // 64 x 64 tiles of a single chunk

template <class In>
int pick_tile(int64_t T, int64_t E, int64_t d) {
    constexpr bool kBf16 = In::kPer == 8;
    const int64_t bytes = d * (int64_t)sizeof(typename In::elem_t);
    const int64_t chunks = (bytes + kChunk - 1) / kChunk;
    const bool whole = bytes % kChunk == 0;
    // A launch of 2^32 threads and more is refused by the runtime.
    const auto fits = [&](int64_t bm, int64_t bn) {
        const int64_t blocks = ((T + bm - 1) / bm + 7) / 8 * 8 * ((E + bn - 1) / bn);
        return blocks * (bm >= 128 ? 512 : 256) < (int64_t)1 << 32;
    };
    // One chunk: no ring to fill, and each block is a chain of a few latencies.
    // The smallest tile puts most blocks on a compute unit (eight) and skips
    // the part of the chunk past d. 300000 x 8 x 16: bf16 18.9 us in 256 x 64 tiles,
    // 9.9 in these; fp32 23.6 in 32 x 32, 13.4; through an index 29.2 and 16.7,
    // 31.7 and 19.3.
    if (chunks == 1 && E <= 64 && fits(64, 64)) return kOneChunk;
    int best = -1;
    double low = 0.0;
    for (int i = 0; i < (int)(sizeof(kTiles) / sizeof(kTiles[0])); ++i) {
        const TileCost &t = kTiles[i];
        if (!fits(t.bm, t.bn)) continue;
        const int64_t tiles = ((T + t.bm - 1) / t.bm) * ((E + t.bn - 1) / t.bn);
        const double turns = (double)((tiles + kComputeUnits - 1) / kComputeUnits);
        double cost = turns * (kBf16 ? t.bf16 : t.f32);
        if (t.bm > kST) {
            if (!whole && chunks > 2) cost *= 1.4;
        } else if (kBf16) {
            cost *= 0.8 + 0.2 / turns;
        }
        if (best < 0 || cost < low) {
            best = i;
            low = cost;
        }
    }
    return best;   // (-1: none)
}

template <class In, int NJ>
hipError_t launch_small(const typename In::elem_t *H, const int32_t *rows, int64_t h_rows,
                        const typename In::elem_t *W, float *S, int64_t T, int64_t E, int64_t d,
                        hipStream_t stream) {
    const int64_t nm8 = ((T + kST - 1) / kST + 7) / 8 * 8;
    const int64_t nn = (E + 16 * NJ - 1) / (16 * NJ);
    hipLaunchKernelGGL((affinity_small_kernel<In, NJ>), dim3((unsigned)(nm8 * nn)),
                       dim3(64 * kSWaves), 0, stream, H, rows, h_rows, W, S, (int)T, (int)E, (int)d);
    return hipGetLastError();
}

template <class In>
hipError_t launch_affinity(const typename In::elem_t *H, const int32_t *rows, int64_t h_rows,
                           const typename In::elem_t *W, float *S, int64_t T, int64_t E, int64_t d,
                           hipStream_t stream) {
    constexpr bool kBf16 = In::kPer == 8;
    switch (pick_tile<In>(T, E, d)) {
        case -1: return hipErrorInvalidConfiguration;
        case 0:
            if constexpr (kBf16)
                return launch_pipe<In, 256, 256, 2, 4, 2>(H, rows, h_rows, W, S, T, E, d, stream);
            break;
        case 1: return launch_pipe<In, 256, 128, 2, 2, 3>(H, rows, h_rows, W, S, T, E, d, stream);
        case 2: return launch_pipe<In, 256, 64, 2, 1, 3>(H, rows, h_rows, W, S, T, E, d, stream);
        case 3:
            if constexpr (kBf16)
                return launch_pipe<In, 128, 128, 1, 2, 4>(H, rows, h_rows, W, S, T, E, d, stream);
            break;
        case 4: return launch_pipe<In, 128, 64, 1, 1, 4>(H, rows, h_rows, W, S, T, E, d, stream);
        case 5: return launch_pipe<In, 64, 64, 1, 1, 4>(H, rows, h_rows, W, S, T, E, d, stream);
        case kOneChunk:
            return launch_pipe<In, 64, 64, 1, 1, 1>(H, rows, h_rows, W, S, T, E, d, stream);
        case 6: return launch_small<In, 4>(H, rows, h_rows, W, S, T, E, d, stream);
        default: break;
    }
    return launch_small<In, 2>(H, rows, h_rows, W, S, T, E, d, stream);
}

}  // namespace

hipError_t launch_affinity_bf16(const uint16_t *H, const int32_t *rows, int64_t h_rows,
                                const uint16_t *W, float *S, int64_t T, int64_t E, int64_t d,
                                hipStream_t stream) {
    return launch_affinity<Bf16>(H, rows, h_rows, W, S, T, E, d, stream);
}

hipError_t launch_affinity_f32(const float *H, const int32_t *rows, int64_t h_rows,
                               const float *W, float *S, int64_t T, int64_t E, int64_t d,
                               hipStream_t stream) {
    return launch_affinity<F32>(H, rows, h_rows, W, S, T, E, d, stream);
}

}  // namespace base
