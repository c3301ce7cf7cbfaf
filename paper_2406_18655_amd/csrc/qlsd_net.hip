// Learned reliability refinement between BP and LSD (include/qlsd_net.h): a 3-layer
// message-passing network over the Tanner graph, hidden width 32.  Dense products run on
// bf16 MFMA with float32 accumulation; neighbour means in float32.  Training: one workgroup of 12
// wavefronts per shot at a time, node features in LDS, and the gradient of every parameter in
// registers across all shots a workgroup processes, added to the global gradient once per workgroup.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/qlsd_net.h"
#include "qlsd_internal.h"

namespace qlsd {
namespace {

constexpr int HID = 32;
constexpr int NL = 3;
constexpr int NPAR = QLSD_NET_PARAMS;
// parameter offsets (floats)
constexpr int P_W0 = 0, P_B0 = 64, P_LAYER = 96, P_LSTRIDE = 3136;
constexpr int P_A = 0, P_a = 1024, P_B = 1056, P_C = 2080, P_b = 3104;
constexpr int P_W = 96 + 3 * 3136, P_BO = P_W + 32;
// small float vectors kept in LDS: W0, b0, a1..3, b1..3, w, bo
constexpr int SV_W0 = 0, SV_B0 = 64, SV_A = 96, SV_BL = 192, SV_W = 288, SV_BO = 320, SV_N = 321;

typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));

// float -> bf16, round to nearest even (gfx950 converts in hardware: v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const float2v v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2v));
}


__host__ __device__ inline int pad16(int x) { return (x + 15) & ~15; }
__host__ __device__ inline size_t al16(size_t x) { return (x + 15) & ~size_t(15); }

struct NetArgs {
    DevGraph g;
    const float *lam;       // n
    const float *theta;     // NPAR
    const uint8_t *syn;     // B x m
    const float *llr;       // B x n
    const uint8_t *err;     // B x n (training)
    float *llr_out;         // B x n (inference)
    const int *list;        // inference: shots to process (nullable: 0..count-1)
    const int *list_count;  // device count when list != nullptr
    int count;
    float *grad;            // NPAR (training, accumulated)
    float *loss;            // 1 (training, accumulated)
    float inv_total;        // 1 / (shots * n) (training)
    unsigned char *act;     // activation workspace, one slice per workgroup (nullptr: in LDS)
    size_t act_stride;      // bytes per slice
    const uint32_t *nbc;    // large-graph inference: [MP][max_rw] byte offsets of fault rows (padded)
    const uint32_t *nbf;    // [NP][max_cw] byte offsets of check rows (padded)
    const float *rdc;       // [MP] 1 / check degree (0 on padding)
    const float *rdf;       // [NP] 1 / fault degree (of the fault in each row)
    const int32_t *perm;    // [NP] large-graph inference: fault held by each feature row (-1: padding)
    const int32_t *tdeg;    // [NP/16] largest fault degree of each 16-row tile
};

// Training: per-workgroup storage.  The shared part (bf16 weights, small vectors, u16 CSR/CSC tables)
// always sits in LDS; net_shared_layout is also the measure of the graphs a net accepts (limit: with a
// second copy of the vectors, which no kernel holds any more).  The activation part (the shot's inputs,
// features of every layer, aggregation and backward buffers) sits in LDS after it when both fit, else in a
// workgroup-private slice of a device workspace (large graphs such as the 936 x 8800 detector error model).
__host__ __device__ inline size_t net_shared_layout(int n, int m, int E, bool limit, size_t *o) {
    size_t off = 0;
    o[0] = off; off += al16(sizeof(uint16_t) * 9 * 1024);
    o[1] = off; off += al16(sizeof(float) * SV_N);
    o[2] = off; off += limit ? al16(sizeof(float) * SV_N) : 0;
    o[3] = off; off += al16(sizeof(uint16_t) * ((size_t)m + 1 + E + n + 1 + E));
    o[4] = off; off += al16(sizeof(float) * 4);
    return off;
}
// Inputs (posteriors, tanh, scaled priors, true errors, reciprocal degrees of faults; syndrome signs,
// reciprocal degrees of checks), features of every layer, the aggregation (one row per feature) and the
// masked gradient (bf16), the gradients of
// the fault features and of the products (float).  tight: the scaled priors are read from memory.
__host__ __device__ inline size_t net_act_layout(int n, int m, bool tight, size_t *o) {
    const int NP = pad16(n), MP = pad16(m), XP = NP > MP ? NP : MP;
    size_t off = 0;
    o[0] = off; off += al16(sizeof(float) * ((tight ? 4 : 5) * (size_t)n + 2 * (size_t)m));
    o[1] = off; off += al16(sizeof(uint16_t) * ((NL + 1) * (size_t)NP * HID + NL * (size_t)MP * HID));
    o[2] = off; off += al16(sizeof(uint16_t) * (size_t)(XP + 4) * HID);
    o[3] = off; off += al16(sizeof(uint16_t) * (size_t)XP * HID);
    o[4] = off; off += al16(sizeof(float) * ((size_t)NP + XP) * HID);
    return off;
}
constexpr int kTrainThreads = 768;
constexpr int kTrainWaves = kTrainThreads / 64;
constexpr int kTrainParts = 3;  // wavefronts that share a weight-gradient tile, each a third of the nodes
// Where the activations lie.  kTrainLds: in LDS, after the shared part and the transposed weights.
// kTrainTight: in LDS without transposed weights (operands gathered from the rows) and scaled priors, for
// graphs just too large for kTrainLds: every graph of the decoder's row weights whose features, gradients
// and tables fit in LDS trains there, so gradients on several streams do not meet in the net's workspace
// and the first call allocates nothing.  kTrainWorkspace: in the workspace.  At the end the LDS after the
// shared part makes room for every wavefront's gradients: kTrainParts copies of the matrices (kTrainTight:
// of one layer's at a time), then per wavefront the small vectors and the loss.
enum TrainPlace { kTrainWorkspace, kTrainTight, kTrainLds };
constexpr size_t kNetTransposed = sizeof(uint16_t) * 9 * 1024;
__host__ __device__ constexpr int train_flush_layers(TrainPlace p) { return p == kTrainLds ? NL : 1; }
constexpr size_t net_flush_bytes(TrainPlace p) {
    return sizeof(float) * (kTrainParts * 3 * train_flush_layers(p) * 1024 + kTrainWaves * (SV_N + 1));
}

// Feature rows of 32 bf16: the 8-byte group q4 (4 features) of row v sits at position
// q4 ^ ((v >> 1) & 7), so 16 consecutive rows' reads of one group, and reads and writes of whole rows,
// spread over the LDS banks.  Byte offsets of a group and of one feature.
__device__ __forceinline__ int row8(int v, int q4) { return v * 64 + ((q4 ^ ((v >> 1) & 7)) << 3); }
__device__ __forceinline__ int row2(int v, int f) { return row8(v, f >> 2) + (f & 3) * 2; }
// Rows of 32 floats: the 16-byte group q4 at the same position.  A row's offset with group 0's position
// (row8(v, 0), and twice it for floats) gives every group's by an exclusive or with q4 << 3 (<< 4).
__device__ __forceinline__ int frow(int v, int q4) { return 2 * row8(v, q4); }

__device__ __forceinline__ float4v unpack4(uint2 u) {
    return (float4v){__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                     __uint_as_float(u.y & 0xffff0000u)};
}
__device__ __forceinline__ uint2 pack4(float4v v) { return make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])); }

// Forward and backward of one shot at a time on one workgroup of 12 wavefronts; LDSACT: the activations
// sit in LDS (PLACE).  Dense products are pairs of v_mfma_f32_16x16x16_bf16 (features 0..15, then 16..31),
// formed transposed (D = W X^T) so a lane receives four consecutive features of one node and stores
// them as one word; a lane's operand, two groups of four features of one node, is gathered from the
// node's neighbours, averaged in float32 and rounded to bf16 in registers (forward), or read as two
// words.  Weight gradients sum over nodes: their operands are
// columns of the feature rows, and the tiles (one of B or C and one of A per wavefront and layer, the
// nodes split over three wavefronts) stay in registers across all shots of the workgroup.  The
// vectors' gradients stay in registers too: a thread always works on the same four features.
//
// A shot is bound by the latency of its phases (two per layer forward, four backward, of 1.6 to 4.4
// thousand cycles each with three wavefronts per SIMD; 12 wavefronts leave each 168 registers, enough
// for all gradients: 16 of 128 spilled and were slower), about 21 us; the prologue and the flush take
// 17 us a workgroup.  Gradient of 1,024 shots of [[144,12,12]]: 1.02 ms -> 0.113 ms (before: 4
// wavefronts, float atomics on LDS, four cycles a lane, for every element of the vectors' gradients,
// 2-byte operand reads and a tanh per feature).  256 shots of the 936 x 8800 detector error model with
// activations in the workspace: 28.1 -> 4.9 ms.

// DR, DC: every check has DR faults and every fault DC checks, so a node's neighbours are read
// together; 0: the degrees come from the tables.
template <TrainPlace PLACE, int DR, int DC>
__global__ __launch_bounds__(kTrainThreads) void net_train_kernel(NetArgs A) {
    constexpr bool LDSACT = PLACE != kTrainWorkspace, TIGHT = PLACE == kTrainTight, WCOL = PLACE == kTrainLds;
    extern __shared__ __align__(16) unsigned char smem[];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int n = A.g.n, m = A.g.m, E = A.g.nnz;
    const int NP = pad16(n), MP = pad16(m), XP = NP > MP ? NP : MP;
    size_t so[5], ao[5];
    const size_t shared_bytes = net_shared_layout(n, m, E, false, so);
    net_act_layout(n, m, TIGHT, ao);
    unsigned char *wrow = smem + so[0];  // [layer][A,B,C][out] rows of 32 inputs, as feature rows
    float *sv = (float *)(smem + so[1]);
    uint16_t *rp = (uint16_t *)(smem + so[3]), *ci = rp + (m + 1), *cp = ci + E, *ri = cp + (n + 1);
    float *loss = (float *)(smem + so[4]);
    unsigned char *wcol = smem + shared_bytes;  // WCOL: [layer][A,B,C][in] rows of 32 outputs
    unsigned char *act;
    if constexpr (LDSACT) act = smem + shared_bytes + (WCOL ? kNetTransposed : 0);
    else act = A.act + (size_t)blockIdx.x * A.act_stride;
    float *Lsh = (float *)(act + ao[0]), *x0 = Lsh + n, *ev = x0 + n, *rdf = ev + n, *sgn = rdf + n, *rdc = sgn + m, *x1 = rdc + m;
    auto scaled_prior = [&](int j) {
        if constexpr (TIGHT) return A.lam[j] * 0.125f;
        else return x1[j];
    };
    auto Hrow = [&](int l) { return act + ao[1] + (size_t)l * NP * 64; };
    auto Crow = [&](int l) { return act + ao[1] + (size_t)(NL + 1) * NP * 64 + (size_t)(l - 1) * MP * 64; };
    unsigned char *AGG = act + ao[2], *DUV = act + ao[3], *DH = act + ao[4], *DT = DH + (size_t)NP * 128;

    // every load of the prologue is issued before the first result is used
    constexpr int TH = 9 * 1024 / kTrainThreads;
    static_assert(TH * kTrainThreads == 9 * 1024 && kTrainThreads >= SV_N, "one pass over the parameters");
    auto matrix_offset = [](int mat) { return P_LAYER + (mat / 3) * P_LSTRIDE + (mat % 3 == 0 ? P_A : mat % 3 == 1 ? P_B : P_C); };
    float th[TH];
#pragma unroll
    for (int k = 0; k < TH; k++) {
        const int x = t + k * kTrainThreads;
        th[k] = A.theta[matrix_offset(x >> 10) + (x & 1023)];
    }
    auto offset_of = [](int x) {  // parameter offset of small-vector entry x
        if (x < SV_B0) return P_W0 + x;
        if (x < SV_A) return P_B0 + (x - SV_B0);
        if (x < SV_BL) return P_LAYER + ((x - SV_A) >> 5) * P_LSTRIDE + P_a + ((x - SV_A) & 31);
        if (x < SV_W) return P_LAYER + ((x - SV_BL) >> 5) * P_LSTRIDE + P_b + ((x - SV_BL) & 31);
        if (x < SV_BO) return P_W + (x - SV_W);
        return P_BO;
    };
    // LDSACT: the tables of neighbours hold their rows' offsets (row8(v, 0), below 2^16)
    auto entry = [](int v) { return (uint16_t)(LDSACT ? row8(v, 0) : v); };
    const float svt = t < SV_N ? A.theta[offset_of(t)] : 0.f;
    for (int x = t; x < E; x += kTrainThreads) {
        const int c = A.g.col_idx[x], r = A.g.row_idx[x];
        ci[x] = entry(c);
        ri[x] = entry(r);
    }
    for (int x = t; x <= m; x += kTrainThreads) rp[x] = (uint16_t)A.g.row_ptr[x];
    for (int x = t; x <= n; x += kTrainThreads) cp[x] = (uint16_t)A.g.col_ptr[x];
    if constexpr (!TIGHT)
        for (int j = t; j < n; j += kTrainThreads) x1[j] = A.lam[j] * 0.125f;
#pragma unroll
    for (int k = 0; k < TH; k++) {
        const int x = t + k * kTrainThreads, mat = x >> 10, o = (x >> 5) & 31, i = x & 31;
        const uint16_t w = f2bf(th[k]);
        *(uint16_t *)(wrow + row2(mat * 32 + o, i)) = w;
        if constexpr (WCOL) *(uint16_t *)(wcol + row2(mat * 32 + i, o)) = w;
    }
    if (t < SV_N) sv[t] = svt;
    __syncthreads();
    for (int j = t; j < n; j += kTrainThreads) rdf[j] = cp[j + 1] > cp[j] ? 1.0f / (float)(cp[j + 1] - cp[j]) : 0.f;
    for (int i = t; i < m; i += kTrainThreads) rdc[i] = rp[i + 1] > rp[i] ? 1.0f / (float)(rp[i + 1] - rp[i]) : 0.f;
    if (t == 0) loss[0] = 0.f;

    int tv = t;                 // the thread, opaque to the compiler from layer to layer: the offsets that
                                // depend on it only are cheaper to form again than to keep in registers
    int nl = lane & 15, kq = lane >> 4;  // products: node (or row) and group of the k range
    int q4 = t & 7;                      // elementwise phases: this thread's four features
    auto renew = [&]() {
        asm volatile("" : "+v"(tv));
        nl = tv & 15;
        kq = (tv >> 4) & 3;
        q4 = tv & 7;
    };
    const float4v zero4 = {0.f, 0.f, 0.f, 0.f};
    // operand: features 4 kq .. + 3 and 16 + 4 kq .. + 3 of one row
    struct Op { uint2 lo, hi; };
    const Op zero_op = {make_uint2(0u, 0u), make_uint2(0u, 0u)};
    auto load_op = [&](const unsigned char *rows, int v) {
        return Op{*(const uint2 *)(rows + row8(v, kq)), *(const uint2 *)(rows + row8(v, kq + 4))};
    };
    // operand rows of W^T (inputs ct 16 .. + 15, k = outputs)
    auto wt_op = [&](int mat, int ct) -> Op {
        if constexpr (WCOL) {
            return load_op(wcol, mat * 32 + ct * 16 + nl);
        } else {
            uint32_t h[8];
#pragma unroll
            for (int u = 0; u < 8; u++)
                h[u] = *(const uint16_t *)(wrow + row2(mat * 32 + (u >> 2) * 16 + kq * 4 + (u & 3), ct * 16 + nl));
            return Op{make_uint2(h[0] | h[1] << 16, h[2] | h[3] << 16), make_uint2(h[4] | h[5] << 16, h[6] | h[7] << 16)};
        }
    };
    auto product = [](const Op &w, const Op &x, float4v acc) {
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, w.lo), __builtin_bit_cast(short4v, x.lo), acc, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, w.hi), __builtin_bit_cast(short4v, x.hi), acc, 0, 0, 0);
    };
    // sum of f(neighbour's row offset) over a node's neighbours, in their order; ROWS: neighbours of a
    // check, else of a fault
    auto row_of = [](int v) { return LDSACT ? v : row8(v, 0); };  // offset of a table entry's row
    auto over = [&](auto Rows, int v, auto &&load, auto &&add) {
        constexpr bool ROWS = decltype(Rows)::value;
        constexpr int D = ROWS ? DR : DC;
        const uint16_t *idx = ROWS ? ci : ri;
        if constexpr (D > 0) {
            decltype(load(0)) x[D];
#pragma unroll
            for (int u = 0; u < D; u++) x[u] = load(row_of(idx[v * D + u]));
#pragma unroll
            for (int u = 0; u < D; u++) add(x[u]);
        } else {
            const int e1 = ROWS ? rp[v + 1] : cp[v + 1];
            for (int e = ROWS ? rp[v] : cp[v]; e < e1; e++) add(load(row_of(idx[e])));
        }
    };
    using Checks = std::true_type;   // over a check's faults
    using Faults = std::false_type;  // over a fault's checks
    // neighbour means: 4 features of one node (elementwise phases), an operand (products)
    auto mean4 = [&](auto Rows, const unsigned char *rows, int v, float rd) {
        float4v s = zero4;
        over(Rows, v, [&](int r) { return *(const uint2 *)(rows + (r ^ (q4 << 3))); }, [&](uint2 x) { s += unpack4(x); });
        return s * rd;
    };
    auto mean_op = [&](auto Rows, const unsigned char *rows, int v, float rd) {
        float4v a = zero4, b = zero4;
        over(Rows, v,
             [&](int r) { return Op{*(const uint2 *)(rows + (r ^ (kq << 3))), *(const uint2 *)(rows + (r ^ ((kq + 4) << 3)))}; },
             [&](const Op &x) {
                 a += unpack4(x.lo);
                 b += unpack4(x.hi);
             });
        return Op{pack4(a * rd), pack4(b * rd)};
    };
    // 16 x 16 tiles of weight gradients over the nodes of steps s0, s0 + kTrainParts, ...: rows from the
    // masked gradient's features, columns from the aggregation and, with a second accumulator, from
    // feature rows.
    const int gs = XP + 4;  // nodes per feature of the aggregation (the pad spreads it over the banks)
    auto wgrad = [&](int trow, int tcol, int steps, int s0, float4v &acc, auto Two, const unsigned char *rows, float4v &acc2) {
        constexpr bool TWO = decltype(Two)::value;
        for (int s = s0; s < steps; s += kTrainParts) {
            const int v = s * 16 + kq * 4;
            short4v a, c;
#pragma unroll
            for (int u = 0; u < 4; u++) a[u] = *(const short *)(DUV + row2(v + u, trow + nl));
            const short4v b = *(const short4v *)((const uint16_t *)AGG + (tcol + nl) * gs + v);
            if constexpr (TWO) {
#pragma unroll
                for (int u = 0; u < 4; u++) c[u] = *(const short *)(rows + row2(v + u, tcol + nl));
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
            if constexpr (TWO) acc2 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, c, acc2, 0, 0, 0);
        }
    };
    auto put_agg = [&](int v, float4v x) {
        const uint2 p = pack4(x);
        uint16_t *d = (uint16_t *)AGG + q4 * 4 * gs + v;
        d[0] = (uint16_t)p.x;
        d[gs] = (uint16_t)(p.x >> 16);
        d[2 * gs] = (uint16_t)p.y;
        d[3 * gs] = (uint16_t)(p.y >> 16);
    };
    // wavefront w's tiles: dB of tile w & 3 and dC of the same, dA likewise, part w >> 2
    static_assert(kTrainWaves == 4 * kTrainParts, "four tiles a matrix");
    const int g_row = ((wave >> 1) & 1) * 16, g_col = (wave & 1) * 16, g_part = wave >> 2;
    float4v gb[NL], gc[NL], ga[NL], accb[NL], acca[NL], accw = zero4, accb0 = zero4, accx0 = zero4, accx1 = zero4;
    float accbo = 0.f, accloss = 0.f;
#pragma unroll
    for (int l = 0; l < NL; l++) gb[l] = gc[l] = ga[l] = accb[l] = acca[l] = zero4;

    // LDSACT (no more faults or checks than threads): the next shot's inputs are in flight while this one runs
    float nx_llr = 0.f;
    int nx_err = 0, nx_syn = 0;
    auto fetch = [&](int shot) {
        if (shot >= A.count) return;
        if (t < n) {
            nx_llr = A.llr[(size_t)shot * n + t];
            nx_err = A.err[(size_t)shot * n + t];
        }
        if (t < m) nx_syn = A.syn[(size_t)shot * m + t];
    };
    if constexpr (LDSACT) fetch(blockIdx.x);
    for (int shot = blockIdx.x; shot < A.count; shot += gridDim.x) {
        __syncthreads();  // the previous shot's buffers, or the tables
        auto put_fault = [&](int j, float v, int e) {
            Lsh[j] = v;
            x0[j] = tanhf(v * 0.125f);
            ev[j] = (float)(e & 1);
        };
        if constexpr (LDSACT) {
            if (t < n) put_fault(t, nx_llr, nx_err);
            if (t < m) sgn[t] = (nx_syn & 1) ? -1.f : 1.f;
            fetch(shot + gridDim.x);
        } else {
            for (int j = t; j < n; j += kTrainThreads)
                put_fault(j, A.llr[(size_t)shot * n + j], A.err[(size_t)shot * n + j]);
            for (int i = t; i < m; i += kTrainThreads) sgn[i] = (A.syn[(size_t)shot * m + i] & 1) ? -1.f : 1.f;
        }
        __syncthreads();
        renew();
        // ---- forward: input layer
        for (int it = tv; it < NP * 8; it += kTrainThreads) {
            const int j = it >> 3;
            float4v h = zero4;
            if (j < n) {
                const float a = x0[j], b = scaled_prior(j);
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int f = q4 * 4 + u;
                    h[u] = fmaxf(sv[SV_W0 + f * 2] * a + sv[SV_W0 + f * 2 + 1] * b + sv[SV_B0 + f], 0.f);
                }
            }
            *(uint2 *)(Hrow(0) + row8(j, q4)) = pack4(h);
        }
        __syncthreads();
#pragma unroll
        for (int l = 1; l <= NL; l++) {
            const int mat = (l - 1) * 3;
            renew();
            // c = relu(A mean(h) + sigma a)
            for (int tile = wave; tile < MP / 16; tile += kTrainWaves) {
                const int i = tile * 16 + nl;
                Op x = zero_op;
                float sg = 0.f;
                if (i < m) {
                    x = mean_op(Checks{}, Hrow(l - 1), i, rdc[i]);
                    sg = sgn[i];
                }
#pragma unroll
                for (int ct = 0; ct < 2; ct++) {
                    const float4v d = product(load_op(wrow, mat * 32 + ct * 16 + nl), x, zero4);
                    const float4v a = *(const float4v *)(sv + SV_A + (l - 1) * HID + ct * 16 + kq * 4);
                    float4v c;
#pragma unroll
                    for (int u = 0; u < 4; u++) c[u] = i < m ? fmaxf(d[u] + sg * a[u], 0.f) : 0.f;
                    *(uint2 *)(Crow(l) + row8(i, ct * 4 + kq)) = pack4(c);
                }
            }
            __syncthreads();
            renew();
            // h = relu(B h + C mean(c) + b)
            for (int tile = wave; tile < NP / 16; tile += kTrainWaves) {
                const int j = tile * 16 + nl;
                Op x = zero_op;
                if (j < n) x = mean_op(Faults{}, Crow(l), j, rdf[j]);
                const Op h = load_op(Hrow(l - 1), j);
                float out = 0.f;
#pragma unroll
                for (int ct = 0; ct < 2; ct++) {
                    float4v d = product(load_op(wrow, (mat + 1) * 32 + ct * 16 + nl), h, zero4);
                    d = product(load_op(wrow, (mat + 2) * 32 + ct * 16 + nl), x, d);
                    const float4v b = *(const float4v *)(sv + SV_BL + (l - 1) * HID + ct * 16 + kq * 4);
                    float4v r;
#pragma unroll
                    for (int u = 0; u < 4; u++) r[u] = j < n ? fmaxf(d[u] + b[u], 0.f) : 0.f;
                    const uint2 p = pack4(r);
                    *(uint2 *)(Hrow(l) + row8(j, ct * 4 + kq)) = p;
                    if (l == NL) {
                        const float4v h4 = unpack4(p), w4 = *(const float4v *)(sv + SV_W + ct * 16 + kq * 4);
                        out += h4[0] * w4[0] + h4[1] * w4[1] + h4[2] * w4[2] + h4[3] * w4[3];
                    }
                }
                if (l == NL) {
                    // L' = L + w . h + b_out over the fault's four lanes; loss and its gradient
                    out += __shfl_xor(out, 16, 64);
                    out += __shfl_xor(out, 32, 64);
                    if (kq == 0 && j < n) {
                        const float Lp = Lsh[j] + (out + sv[SV_BO]), e = ev[j];
                        // softplus(-L') + e L'
                        accloss += (fmaxf(-Lp, 0.f) + log1pf(expf(-fabsf(Lp))) + e * Lp) * A.inv_total;
                        const float dD = (e - 1.f / (1.f + expf(Lp))) * A.inv_total;
                        accbo += dD;
                        Lsh[j] = dD;
                    }
                }
            }
            __syncthreads();
        }
        // ---- backward.  Per layer: the gradient of the fault features (from the output layer, or the
        // product with B plus the neighbour sum of the layer above), masked; g recomputed; then the
        // products, and the same on the checks' side.
        const float4v wv = *(const float4v *)(sv + SV_W + q4 * 4);
#pragma unroll
        for (int l = NL; l >= 0; l--) {
            renew();
            for (int it = tv; it < NP * 8; it += kTrainThreads) {
                const int j = it >> 3;
                float4v dh = zero4, h = unpack4(*(const uint2 *)(Hrow(l) + row8(j, q4)));
                if (l == NL) {
                    if (j < n) {
                        const float dD = Lsh[j];
                        accw += dD * h;
                        dh = dD * wv;
                    }
                } else if (j < n) {
                    float4v s = zero4;
                    over(Faults{}, j, [&](int r) { return *(const float4v *)(DT + ((2 * r) ^ (q4 << 4))); },
                         [&](float4v x) { s += x; });
                    dh = *(const float4v *)(DH + frow(j, q4)) + s;
                }
#pragma unroll
                for (int u = 0; u < 4; u++) dh[u] = h[u] > 0.f ? dh[u] : 0.f;
                if (l == 0) {
                    if (j < n) {
                        accx0 += dh * x0[j];
                        accx1 += dh * scaled_prior(j);
                        accb0 += dh;
                    }
                } else {
                    accb[l > 0 ? l - 1 : 0] += dh;
                    *(uint2 *)(DUV + row8(j, q4)) = pack4(dh);
                    float4v g = zero4;
                    if (j < n) g = mean4(Faults{}, Crow(l > 0 ? l : 1), j, rdf[j]);
                    put_agg(j, g);
                }
            }
            if (l == 0) break;
            const int li = l > 0 ? l - 1 : 0, mat = li * 3;
            __syncthreads();
            renew();
            // dB += du^T h_{l-1}, dC += du^T g; dg = du C -> DT, dh_{l-1} = du B -> DH
            wgrad(g_row, g_col, NP / 16, g_part, gc[li], std::true_type{}, Hrow(li), gb[li]);
            for (int tile = wave; tile < NP / 16; tile += kTrainWaves) {
                const int j = tile * 16 + nl;
                const Op du = load_op(DUV, j);
                const float rd = j < n ? rdf[j] : 0.f;  // dc_i sums dg_j / deg_j
#pragma unroll
                for (int ct = 0; ct < 2; ct++) {
                    *(float4v *)(DT + frow(j, ct * 4 + kq)) = product(wt_op(mat + 2, ct), du, zero4) * rd;
                    *(float4v *)(DH + frow(j, ct * 4 + kq)) = product(wt_op(mat + 1, ct), du, zero4);
                }
            }
            __syncthreads();
            renew();
            // dc_i = sum_{j in N(i)} dg_j / deg_j; dv = dc * [c > 0]; da; m_l recomputed into AGG
            for (int it = tv; it < MP * 8; it += kTrainThreads) {
                const int i = it >> 3;
                float4v dv = zero4, mean = zero4;
                if (i < m) {
                    over(Checks{}, i, [&](int r) { return *(const float4v *)(DT + ((2 * r) ^ (q4 << 4))); },
                         [&](float4v x) { dv += x; });
                    const float4v c = unpack4(*(const uint2 *)(Crow(li + 1) + row8(i, q4)));
#pragma unroll
                    for (int u = 0; u < 4; u++) dv[u] = c[u] > 0.f ? dv[u] : 0.f;
                    acca[li] += sgn[i] * dv;
                    mean = mean4(Checks{}, Hrow(li), i, rdc[i]);
                }
                *(uint2 *)(DUV + row8(i, q4)) = pack4(dv);
                put_agg(i, mean);
            }
            __syncthreads();
            renew();
            // dA += dv^T m; dm = dv A -> DT (summed over each fault's checks in the next phase)
            wgrad(g_row, g_col, MP / 16, g_part, ga[li], std::false_type{}, nullptr, ga[li]);
            for (int tile = wave; tile < MP / 16; tile += kTrainWaves) {
                const int i = tile * 16 + nl;
                const Op dv = load_op(DUV, i);
                const float rd = i < m ? rdc[i] : 0.f;  // dh_j sums dm_i / deg_i
#pragma unroll
                for (int ct = 0; ct < 2; ct++)
                    *(float4v *)(DT + frow(i, ct * 4 + kq)) = product(wt_op(mat, ct), dv, zero4) * rd;
            }
            __syncthreads();
        }
    }

    // ---- flush: tiles (rows: out features, columns: in features), vectors, loss.  LDSACT: every
    // wavefront stores its own, then the workgroup adds the copies and adds the sums to the global
    // gradient (float atomics on LDS would take four cycles a lane: 43 us here).
    constexpr int FL = train_flush_layers(PLACE), TILES = 3 * FL * 1024;  // layers, matrix entries at a time
    float *parts = (float *)wcol, *vec0 = parts + kTrainParts * TILES, *vecs = vec0 + wave * (SV_N + 1);
    if constexpr (LDSACT) __syncthreads();
    auto add_tile = [&](int mat, float4v g) {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int at = (g_row + kq * 4 + u) * HID + g_col + nl;
            if constexpr (LDSACT) parts[g_part * TILES + (mat % (3 * FL)) * 1024 + at] = g[u];
            else atomicAdd(&A.grad[matrix_offset(mat) + at], g[u]);
        }
    };
    auto add_vector = [&](int x, float v) {
        if constexpr (LDSACT) vecs[x] = v;
        else atomicAdd(&A.grad[offset_of(x)], v);
    };
    // the vectors: the wavefront's eight threads of each feature group, then one lane per group
    auto flush4 = [&](int base, int stride, float4v v) {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            v[u] += __shfl_xor(v[u], 8, 64);
            v[u] += __shfl_xor(v[u], 16, 64);
            v[u] += __shfl_xor(v[u], 32, 64);
        }
        if (lane < 8) {
#pragma unroll
            for (int u = 0; u < 4; u++) add_vector(base + (q4 * 4 + u) * stride, v[u]);
        }
    };
    flush4(SV_W0, 2, accx0);
    flush4(SV_W0 + 1, 2, accx1);
    flush4(SV_B0, 1, accb0);
    flush4(SV_W, 1, accw);
#pragma unroll
    for (int l = 0; l < NL; l++) {
        flush4(SV_A + l * HID, 1, acca[l]);
        flush4(SV_BL + l * HID, 1, accb[l]);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        accloss += __shfl_xor(accloss, off, 64);
        accbo += __shfl_xor(accbo, off, 64);
    }
    if (lane == 0) {
        add_vector(SV_BO, accbo);
        if constexpr (LDSACT) vecs[SV_N] = accloss;
        else atomicAdd(loss, accloss);
    }
#pragma unroll
    for (int l0 = 0; l0 < NL; l0 += FL) {
#pragma unroll
        for (int l = l0; l < l0 + FL; l++) {
            add_tile(l * 3, ga[l]);
            add_tile(l * 3 + 1, gb[l]);
            add_tile(l * 3 + 2, gc[l]);
        }
        if constexpr (LDSACT) {
            __syncthreads();
            // workgroups start at different places, so they do not queue on one address
            const int N = TILES + (l0 == 0 ? SV_N + 1 : 0);
            const int first = (int)((blockIdx.x * 64u * 37u) % (unsigned)N);
            for (int k = t; k < N; k += kTrainThreads) {
                const int x = k + first < N ? k + first : k + first - N;
                float s = 0.f;
                if (x < TILES) {
#pragma unroll
                    for (int c = 0; c < kTrainParts; c++) s += parts[c * TILES + x];
                    atomicAdd(&A.grad[matrix_offset(3 * l0 + (x >> 10)) + (x & 1023)], s);
                } else {
                    const int y = x - TILES;
#pragma unroll
                    for (int w = 0; w < kTrainWaves; w++) s += vec0[w * (SV_N + 1) + y];
                    atomicAdd(y < SV_N ? &A.grad[offset_of(y)] : A.loss, s);
                }
            }
            if (l0 + FL < NL) __syncthreads();
        }
    }
    if constexpr (!LDSACT) {
        __syncthreads();
        if (t == 0) atomicAdd(A.loss, loss[0]);
    }
}


// ------------------------------------------------------------------------------------------
// Inference: one wavefront per shot, no workgroup barriers.  The A/B/C weight fragments of all
// three layers sit in registers (9 matrices x 2 output tiles of 8 bf16 per lane), and each
// product covers the whole hidden width in one v_mfma_f32_16x16x32_bf16 (gfx950's double-K form,
// twice the rate of the 16x16x16 form per issued instruction).
// Products are formed transposed, D = W X^T, with the output rows of W permuted so that after
// the two products of a layer (two 16-feature output tiles) a lane holds 8 consecutive output
// features of one node -- the same feature group the next product reads -- and results leave
// as one packed 16-byte word.  The neighbour means enter by linearity,
//     A m_i = (1/deg_i) sum_{j in N(i)} A h_j,     C g_j = (1/deg_j) sum_{i in N(j)} C c_i,
// so each neighbour's bf16 feature words feed the MFMA directly (no unpacking or vector sums)
// and the 1/deg scaling is applied to the float32 accumulator.  Neighbour lists are padded to
// the maximum degree with a zero sentinel row.  Compared with net_train_kernel (the training
// forward) the means are not rounded to bf16 before the product; everything else matches.
// ------------------------------------------------------------------------------------------
constexpr int kInferWavesMax = 11;  // one workgroup of up to 11 wavefronts per CU, else 5 (two per CU)

__host__ __device__ inline size_t infer_shared_bytes(int n, int m, int dr, int dc) {
    return al16(sizeof(float) * SV_N) + al16(sizeof(uint16_t) * ((size_t)pad16(m) * dr + (size_t)pad16(n) * dc)) +
           al16(sizeof(float) * ((size_t)pad16(m) + pad16(n) + n));
}
// Per wavefront: fault and check feature rows (bf16 x 32 each), plus one zero sentinel row each
// for the padding of irregular neighbour lists (a code with every row and every column of full
// weight pads nothing but its 16-row tiles, whose results are discarded), and one signed byte
// per check of the padded tiles for the syndrome sign (0 on padding).
__host__ __device__ inline bool infer_regular(const DevGraph &g) {
    return g.min_rw == g.max_rw && g.min_cw == g.max_cw;
}
__host__ __device__ inline size_t infer_wave_bytes(int n, int m, bool regular) {
    return al16(sizeof(uint16_t) * ((size_t)pad16(n) + pad16(m) + (regular ? 0 : 2)) * HID) + al16((size_t)pad16(m));
}

// Feature rows are 64 B: 32 bf16 as four 16-byte groups of 8 features.  Group q of node v sits at
// group position q ^ f(v), f(v) = ((v >> 1) & 3) ^ ((v >> 3) & 1), of its row.  Over 16 consecutive
// nodes (a tile) and a fixed group, any 8 aligned nodes then cover all 8 16-byte slots of a
// 128-byte bank window and any 4 nodes equal mod 4 all 4 slots of their 64-byte quarter of a
// 256-byte window, so the tile's 16-byte reads and writes are free of bank conflicts with either
// width of LDS bank set.  The swizzled row offset srow(v) = 64 v | (f(v) << 4) carries the
// swizzle: group q of node v is at srow(v) ^ 16 q, and the neighbour tables hold srow() of each
// neighbour, so a gather costs one XOR per load.  f depends on bits 1..3 of v only, so the row
// of node 16 rt + r sits at 1024 rt + srow(r).
__host__ __device__ __forceinline__ int srow(int node) {
    return node * 64 | ((((node >> 1) & 3) ^ ((node >> 3) & 1)) << 4);
}
// Features 8q .. 8q+7 of the node with swizzled row offset so: the operand a lane of group q
// supplies to v_mfma_f32_16x16x32_bf16 (lane l: column l & 15, k = 8 (l >> 4) .. +7).
__device__ __forceinline__ bf16x8v lds_group(const unsigned char *base, int so, int q16) {
    return *(const bf16x8v *)(base + (so ^ q16));
}
__device__ __forceinline__ float4v mfma32(bf16x8v a, bf16x8v b, float4v c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

template <int DR, int DC>
__global__ __launch_bounds__(64 * kInferWavesMax) void net_infer_kernel(NetArgs A) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = threadIdx.x;
    const int n = A.g.n, m = A.g.m, NP = pad16(n), MP = pad16(m);
    const int dr = DR ? DR : A.g.max_rw, dc = DC ? DC : A.g.max_cw;
    float *sv = (float *)smem;
    uint16_t *nbc = (uint16_t *)(smem + al16(sizeof(float) * SV_N));  // [MP][dr] byte offsets into H
    uint16_t *nbf = nbc + (size_t)MP * dr;                             // [NP][dc] byte offsets into C
    float *rdc = (float *)((unsigned char *)nbc + al16(sizeof(uint16_t) * ((size_t)MP * dr + (size_t)NP * dc)));
    float *rdf = rdc + MP, *lam = rdf + NP;
    const bool reg = infer_regular(A.g);
    const int nwav = blockDim.x >> 6;
    unsigned char *wbase = smem + infer_shared_bytes(n, m, dr, dc) + (size_t)wave * infer_wave_bytes(n, m, reg);
    const int sent = reg ? 0 : 1;                    // sentinel rows present
    uint16_t *H = (uint16_t *)wbase;                 // (NP + sent) x 32, row NP (if present) is zero
    uint16_t *Cf = H + (size_t)(NP + sent) * HID;    // (MP + sent) x 32, row MP (if present) is zero
    int8_t *sg = (int8_t *)(wbase + al16(sizeof(uint16_t) * ((size_t)NP + MP + 2 * sent) * HID));  // +-1 per check
    unsigned char *Hb = (unsigned char *)H, *Cb = (unsigned char *)Cf;

    for (int x = t; x < SV_N; x += blockDim.x) {
        float v;
        if (x < SV_B0) v = A.theta[P_W0 + x];
        else if (x < SV_A) v = A.theta[P_B0 + (x - SV_B0)];
        else if (x < SV_BL) { const int l = (x - SV_A) >> 5; v = A.theta[P_LAYER + l * P_LSTRIDE + P_a + ((x - SV_A) & 31)]; }
        else if (x < SV_W) { const int l = (x - SV_BL) >> 5; v = A.theta[P_LAYER + l * P_LSTRIDE + P_b + ((x - SV_BL) & 31)]; }
        else if (x < SV_BO) v = A.theta[P_W + (x - SV_W)];
        else v = A.theta[P_BO];
        sv[x] = v;
    }
    for (int x = t; x < MP * dr; x += blockDim.x) {
        const int i = x / dr, k = x - i * dr;
        int v = sent * NP;
        if (i < m) {
            const int e0 = A.g.row_ptr[i], e1 = A.g.row_ptr[i + 1];
            if (e0 + k < e1) v = A.g.col_idx[e0 + k];
        }
        nbc[x] = (uint16_t)srow(v);
    }
    for (int x = t; x < NP * dc; x += blockDim.x) {
        const int j = x / dc, k = x - j * dc;
        int v = sent * MP;
        if (j < n) {
            const int c0 = A.g.col_ptr[j], c1 = A.g.col_ptr[j + 1];
            if (c0 + k < c1) v = A.g.row_idx[c0 + k];
        }
        nbf[x] = (uint16_t)srow(v);
    }
    for (int x = t; x < MP; x += blockDim.x) {
        const int d = x < m ? A.g.row_ptr[x + 1] - A.g.row_ptr[x] : 0;
        rdc[x] = d > 0 ? 1.0f / (float)d : 0.f;
    }
    for (int x = t; x < NP; x += blockDim.x) {
        const int d = x < n ? A.g.col_ptr[x + 1] - A.g.col_ptr[x] : 0;
        rdf[x] = d > 0 ? 1.0f / (float)d : 0.f;
        if (x < n) lam[x] = A.lam[x];
    }
    // sentinel rows (never written again)
    if (sent && lane < 16) {
        ((uint32_t *)(H + (size_t)NP * HID))[lane] = 0u;
        ((uint32_t *)(Cf + (size_t)MP * HID))[lane] = 0u;
    }
    __syncthreads();

    // A-operand fragments of v_mfma_f32_16x16x32_bf16 (the whole hidden width in one product).
    // Output tile ot's row r computes feature 8 (r >> 2) + 4 ot + (r & 3), so that the lane
    // holding rows 4 q8 .. +3 of both tiles holds features 8 q8 .. 8 q8 + 7: one whole feature
    // group, stored as one 16-byte word.  wf[mat][ot] = W[8 (r16 >> 2) + 4 ot + (r16 & 3)][8 q8 .. +7]
    const int r16 = lane & 15, q8 = lane >> 4;
    bf16x8v wf[9][2];
#pragma unroll
    for (int mat = 0; mat < 9; mat++) {
        const int layer = mat / 3, which = mat % 3;
        const float *W = A.theta + P_LAYER + layer * P_LSTRIDE + (which == 0 ? P_A : which == 1 ? P_B : P_C);
#pragma unroll
        for (int ot = 0; ot < 2; ot++) {
            const float *w = W + (8 * (r16 >> 2) + 4 * ot + (r16 & 3)) * HID + 8 * q8;
            wf[mat][ot] = __builtin_bit_cast(bf16x8v, make_uint4(pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]),
                                                                pack_bf16x2(w[4], w[5]), pack_bf16x2(w[6], w[7])));
        }
    }

    // per lane: the tile row's swizzled offset is 1024 rt + srow(lane & 15), and the lane reads,
    // and after a product writes, feature group q8 of that row (byte offset go within the tile)
    const int q16 = q8 << 4, go = srow(r16) ^ q16;
    const int total = A.list ? *A.list_count : A.count;
    for (int item = blockIdx.x * nwav + wave; item < total; item += gridDim.x * nwav) {
        const int shot = A.list ? A.list[item] : item;
        const uint8_t *syn = A.syn + (size_t)shot * m;
        const float *llr = A.llr + (size_t)shot * n;
        for (int i = lane; i < MP; i += 64) sg[i] = i < m ? ((syn[i] & 1) ? -1 : 1) : 0;
        // input layer: lane j computes tanh once and writes its fault's 32 features (4 x 16 B).
        // Padding nodes (j >= n) get relu(b0): no neighbour list names them and no output reads them.
        for (int j = lane; j < NP; j += 64) {
            float x0 = 0.f, x1 = 0.f;
            if (j < n) { x0 = tanhf(llr[j] * 0.125f); x1 = lam[j] * 0.125f; }
            const int so = srow(j);
#pragma unroll
            for (int f8 = 0; f8 < HID; f8 += 8) {
                uint32_t w[4];
#pragma unroll
                for (int h2 = 0; h2 < 4; h2++) {
                    const int f = f8 + 2 * h2;
                    const float v0 = fmaxf(sv[SV_W0 + f * 2] * x0 + sv[SV_W0 + f * 2 + 1] * x1 + sv[SV_B0 + f], 0.f);
                    const float v1 = fmaxf(sv[SV_W0 + f * 2 + 2] * x0 + sv[SV_W0 + f * 2 + 3] * x1 + sv[SV_B0 + f + 1], 0.f);
                    w[h2] = pack_bf16x2(v0, v1);
                }
                *(uint4 *)(Hb + (so ^ ((f8 >> 3) << 4))) = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int l = 0; l < NL; l++) {
            // checks: c_i = relu((1/deg_i) sum_j A h_j + sigma_i a)
            for (int rt = 0; rt < MP / 16; rt++) {
                const int i = rt * 16 + r16;
                float4v acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                const uint16_t *nb = nbc + i * dr;
#pragma unroll
                for (int k = 0; k < (DR ? DR : dr); k++) {
                    const bf16x8v x = lds_group(Hb, nb[k], q16);
#pragma unroll
                    for (int ot = 0; ot < 2; ot++) acc[ot] = mfma32(wf[l * 3 + 0][ot], x, acc[ot]);
                }
                const float rd = rdc[i], sgn = (float)sg[i];
                uint32_t w[4];
#pragma unroll
                for (int ot = 0; ot < 2; ot++) {
                    const float4v av = *(const float4v *)(sv + SV_A + l * HID + 8 * q8 + 4 * ot);
                    float v[4];
#pragma unroll
                    for (int q = 0; q < 4; q++) v[q] = fmaxf(rd * acc[ot][q] + sgn * av[q], 0.f);
                    w[2 * ot] = pack_bf16x2(v[0], v[1]);
                    w[2 * ot + 1] = pack_bf16x2(v[2], v[3]);
                }
                *(uint4 *)(Cb + rt * 1024 + go) = make_uint4(w[0], w[1], w[2], w[3]);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // faults: h_j = relu(B h_j + b + (1/deg_j) sum_i C c_i), b entering as the accumulator of
            // B h_j (in place: a lane reads and writes only its own node's words; padding rows
            // are computed like the rest and never read)
            for (int rt = 0; rt < NP / 16; rt++) {
                const int j = rt * 16 + r16;
                const bf16x8v h = *(const bf16x8v *)(Hb + rt * 1024 + go);
                float4v as[2], an[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int ot = 0; ot < 2; ot++)
                    as[ot] = mfma32(wf[l * 3 + 1][ot], h, *(const float4v *)(sv + SV_BL + l * HID + 8 * q8 + 4 * ot));
                const uint16_t *nb = nbf + j * dc;
#pragma unroll
                for (int k = 0; k < (DC ? DC : dc); k++) {
                    const bf16x8v y = lds_group(Cb, nb[k], q16);
#pragma unroll
                    for (int ot = 0; ot < 2; ot++) an[ot] = mfma32(wf[l * 3 + 2][ot], y, an[ot]);
                }
                const float rd = rdf[j];
                uint32_t w[4];
#pragma unroll
                for (int ot = 0; ot < 2; ot++) {
                    float v[4];
#pragma unroll
                    for (int q = 0; q < 4; q++) v[q] = fmaxf(rd * an[ot][q] + as[ot][q], 0.f);
                    w[2 * ot] = pack_bf16x2(v[0], v[1]);
                    w[2 * ot + 1] = pack_bf16x2(v[2], v[3]);
                }
                *(uint4 *)(Hb + rt * 1024 + go) = make_uint4(w[0], w[1], w[2], w[3]);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        for (int j = lane; j < n; j += 64) {
            float d = sv[SV_BO];
            const int so = srow(j);
#pragma unroll
            for (int f8 = 0; f8 < 4; f8++) {
                const uint4 v = *(const uint4 *)(Hb + (so ^ (f8 << 4)));
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int h2 = 0; h2 < 4; h2++) {
                    d += sv[SV_W + f8 * 8 + 2 * h2] * __uint_as_float(w[h2] << 16);
                    d += sv[SV_W + f8 * 8 + 2 * h2 + 1] * __uint_as_float(w[h2] & 0xffff0000u);
                }
            }
            A.llr_out[(size_t)shot * n + j] = llr[j] + d;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}


// ------------------------------------------------------------------------------------------
// Large-graph inference (graphs whose features do not fit in LDS, e.g. the 936 x 8800 detector
// error model): one workgroup per shot, its wavefronts splitting the 16-node tiles of each
// phase, features in a workgroup-private slice of the device workspace (kept in the last-level
// cache across the grid).  The arithmetic is that of net_infer_kernel: transposed products on
// v_mfma_f32_16x16x32_bf16 with the output rows of W permuted so that a lane ends a layer holding
// one whole 8-feature group (one 16-byte store), neighbour means by linearity on the float32
// accumulator, zero sentinel rows for padding.  Fault rows are stored sorted by degree (row r
// holds fault perm[r]), so the 16 faults of a tile have equal or near-equal degree and a tile
// gathers only up to its own largest degree (tdeg[tile]) instead of the code's; the network
// treats every node alike and each neighbour sum keeps its order, so the row order changes no
// result.  The fault phase issues the loads of two tiles before their products; the check
// phase loads the next group's table entries while the current group's gathers are in flight.
// The input layer is never stored: layer 0 recomputes a fault's first-layer features from its
// 8-byte inputs (tanh(L/8), lambda/8) where it needs them, and the last fault phase applies the
// output layer to its own bf16-rounded features instead of storing them.
// ------------------------------------------------------------------------------------------
constexpr int kBigWaves = 16;
constexpr int kGather = 10;      // check-phase gathers in flight per tile
constexpr int kFaultGather = 6;  // fault-phase gathers per tile and pass (heavier tiles loop)
constexpr int kFaultTiles = 2;   // fault tiles per pass

// Fault row order of the large-graph kernel: faults sorted by degree, largest first (stable);
// rows n .. pad16(n)-1 are padding (-1).
static void big_fault_order(const std::vector<int32_t> &col_ptr, int n, std::vector<int32_t> &perm,
                            std::vector<int32_t> &rowof, std::vector<int32_t> &tdeg) {
    const int NP = pad16(n);
    int maxd = 0;
    for (int j = 0; j < n; j++) maxd = std::max(maxd, col_ptr[j + 1] - col_ptr[j]);
    std::vector<int> start(maxd + 2, 0);
    for (int j = 0; j < n; j++) start[maxd - (col_ptr[j + 1] - col_ptr[j]) + 1]++;
    for (int d = 1; d <= maxd + 1; d++) start[d] += start[d - 1];
    perm.assign(NP, -1);
    rowof.assign(n, 0);
    for (int j = 0; j < n; j++) {
        const int r = start[maxd - (col_ptr[j + 1] - col_ptr[j])]++;
        perm[r] = j;
        rowof[j] = r;
    }
    tdeg.assign(NP / 16, 0);
    for (int r = 0; r < n; r++) {
        const int j = perm[r];
        tdeg[r >> 4] = std::max(tdeg[r >> 4], col_ptr[j + 1] - col_ptr[j]);
    }
}

__global__ void big_tables_kernel(DevGraph g, const int32_t *perm, const int32_t *rowof, uint32_t *nbc, uint32_t *nbf,
                                  float *rdc, float *rdf) {
    const int NP = pad16(g.n), MP = pad16(g.m), dr = g.max_rw, dc = g.max_cw;
    const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    for (size_t x = tid; x < (size_t)MP * dr; x += stride) {
        const int i = (int)(x / dr), k = (int)(x % dr);
        uint32_t off = (uint32_t)NP * 64u;
        if (i < g.m && g.row_ptr[i] + k < g.row_ptr[i + 1]) off = (uint32_t)rowof[g.col_idx[g.row_ptr[i] + k]] * 64u;
        nbc[x] = off;
    }
    for (size_t x = tid; x < (size_t)NP * dc; x += stride) {
        const int r = (int)(x / dc), k = (int)(x % dc), j = perm[r];
        uint32_t off = (uint32_t)MP * 64u;
        if (j >= 0 && g.col_ptr[j] + k < g.col_ptr[j + 1]) off = (uint32_t)g.row_idx[g.col_ptr[j] + k] * 64u;
        nbf[x] = off;
    }
    for (size_t x = tid; x < (size_t)MP; x += stride) {
        const int d = x < (size_t)g.m ? g.row_ptr[x + 1] - g.row_ptr[x] : 0;
        rdc[x] = d > 0 ? 1.0f / (float)d : 0.f;
    }
    for (size_t x = tid; x < (size_t)NP; x += stride) {
        const int j = perm[x];
        const int d = j >= 0 ? g.col_ptr[j + 1] - g.col_ptr[j] : 0;
        rdf[x] = d > 0 ? 1.0f / (float)d : 0.f;
    }
}

// dynamic LDS of net_infer_big_kernel: syndrome signs and the u16 fault neighbour table (the
// kernel also holds 20 KB of static LDS)
__host__ __device__ inline size_t big_dyn_lds(const DevGraph &g) {
    return al16(sizeof(float) * (size_t)g.m) + al16(sizeof(uint16_t) * (size_t)pad16(g.n) * g.max_cw);
}
// per-workgroup slice: fault rows (NP + 1 with the zero row), check rows (MP + 1), and each fault
// row's inputs (x0, x1) as a float pair (NP + 1: the zero row's entry is read, then discarded)
__host__ __device__ inline size_t big_slice_bytes(int n, int m) {
    return al16(sizeof(uint16_t) * ((size_t)pad16(n) + 1 + pad16(m) + 1) * HID) +
           al16(sizeof(float) * 2 * ((size_t)pad16(n) + 1));
}

__device__ __forceinline__ bf16x8v gload(const unsigned char *base, uint32_t off) {
    return *(const bf16x8v *)(base + off);
}

__global__ __launch_bounds__(64 * kBigWaves) void net_infer_big_kernel(NetArgs A) {
    __shared__ __align__(16) float sv[SV_N];
    __shared__ uint4 wfl[9 * 2 * 64];  // weight fragments [mat][ot][lane], output rows permuted
    extern __shared__ __align__(16) unsigned char smem[];  // sg: m floats; then fault neighbour rows
    const int lane = threadIdx.x & 63, t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = A.g.n, m = A.g.m, NP = pad16(n), MP = pad16(m), dr = A.g.max_rw, dc = A.g.max_cw;
    float *sg = (float *)smem;
    // the fault phase's neighbour lists as u16 check rows (MP = the zero row), read from LDS
    uint16_t *nbf16 = (uint16_t *)(smem + al16(sizeof(float) * (size_t)m));
    for (int x = t; x < NP * dc; x += blockDim.x) nbf16[x] = (uint16_t)(A.nbf[x] >> 6);
    unsigned char *Hb = A.act + (size_t)blockIdx.x * A.act_stride;
    unsigned char *Cb = Hb + (size_t)(NP + 1) * 64;

    for (int x = t; x < SV_N; x += blockDim.x) {
        float v;
        if (x < SV_B0) v = A.theta[P_W0 + x];
        else if (x < SV_A) v = A.theta[P_B0 + (x - SV_B0)];
        else if (x < SV_BL) { const int l = (x - SV_A) >> 5; v = A.theta[P_LAYER + l * P_LSTRIDE + P_a + ((x - SV_A) & 31)]; }
        else if (x < SV_W) { const int l = (x - SV_BL) >> 5; v = A.theta[P_LAYER + l * P_LSTRIDE + P_b + ((x - SV_BL) & 31)]; }
        else if (x < SV_BO) v = A.theta[P_W + (x - SV_W)];
        else v = A.theta[P_BO];
        sv[x] = v;
    }
    // A-operand fragment (mat, ot) of lane l: W[8 (r >> 2) + 4 ot + (r & 3)][8 q .. 8 q + 7], r = l & 15,
    // q = l >> 4 (the output-row order of net_infer_kernel)
    for (int x = t; x < 9 * 2 * 64; x += blockDim.x) {
        const int l = x & 63, ot = (x >> 6) & 1, mat = x >> 7;
        const int layer = mat / 3, which = mat % 3, r = l & 15, q = l >> 4;
        const float *W = A.theta + P_LAYER + layer * P_LSTRIDE + (which == 0 ? P_A : which == 1 ? P_B : P_C);
        const float *w = W + (8 * (r >> 2) + 4 * ot + (r & 3)) * HID + 8 * q;
        wfl[x] = make_uint4(pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]), pack_bf16x2(w[4], w[5]),
                            pack_bf16x2(w[6], w[7]));
    }
    if (t < 16) {  // sentinel rows (never written again)
        ((uint32_t *)(Hb + (size_t)NP * 64))[t] = 0u;
        ((uint32_t *)(Cb + (size_t)MP * 64))[t] = 0u;
    }
    const int r16 = lane & 15, q8 = lane >> 4, q16 = q8 << 4;
    __syncthreads();
    auto frag = [&](int mat, int ot) { return __builtin_bit_cast(bf16x8v, wfl[(mat * 2 + ot) * 64 + lane]); };
    auto store_group = [&](unsigned char *p, const float4v &v0, const float4v &v1) {
        *(uint4 *)p = make_uint4(pack_bf16x2(v0[0], v0[1]), pack_bf16x2(v0[2], v0[3]), pack_bf16x2(v1[0], v1[1]),
                                 pack_bf16x2(v1[2], v1[3]));
    };

    // first-layer features 8 q8 .. +7 of a fault from its inputs (x0, x1) = (tanh(L/8), lambda/8)
    // (the parameters are read from LDS at each use rather than held in registers)
    auto h0_group = [&](float x0, float x1) {
        const float4v *w0 = (const float4v *)(sv + SV_W0 + 16 * q8), *b0 = (const float4v *)(sv + SV_B0 + 8 * q8);
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; i++)
            v[i] = fmaxf(fmaf(w0[i >> 1][2 * (i & 1)], x0, fmaf(w0[i >> 1][2 * (i & 1) + 1], x1, b0[i >> 2][i & 3])), 0.f);
        return __builtin_bit_cast(bf16x8v, make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                      pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])));
    };
    // the slice's per-row inputs: x1 = lambda/8 once per launch, x0 = tanh(L/8) per shot
    float2 *X = (float2 *)(Cb + (size_t)(MP + 1) * 64);
    for (int r = t; r <= NP; r += blockDim.x) {
        const int j = r < NP ? A.perm[r] : -1;
        X[r] = make_float2(0.f, j >= 0 ? A.lam[j] * 0.125f : 0.f);
    }
    const uint32_t sentinel_off = (uint32_t)NP * 64u;

    const int total = A.list ? *A.list_count : A.count;
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        const int shot = A.list ? A.list[item] : item;
        const uint8_t *syn = A.syn + (size_t)shot * m;
        const float *llr = A.llr + (size_t)shot * n;
        for (int i = t; i < m; i += blockDim.x) sg[i] = (syn[i] & 1) ? -1.f : 1.f;
        // the input layer is not stored: layer 0 recomputes a fault's first-layer features from
        // its 8-byte inputs wherever it needs them (padding rows get x0 = 0 and are never read)
        for (int r = t; r < NP; r += blockDim.x) {
            const int j = A.perm[r];
            X[r].x = j >= 0 ? tanhf(llr[j] * 0.125f) : 0.f;
        }
        __syncthreads();
        auto layer = [&](auto Lc) {
            constexpr int l = decltype(Lc)::value;
            // checks: c_i = relu((1/deg_i) sum_j A h_j + sigma_i a)
            {
                const bf16x8v a0 = frag(l * 3, 0), a1 = frag(l * 3, 1);
                const float4v av0 = *(const float4v *)(sv + SV_A + l * HID + 8 * q8);
                const float4v av1 = *(const float4v *)(sv + SV_A + l * HID + 8 * q8 + 4);
                for (int rt = wave; rt < MP / 16; rt += kBigWaves) {
                    const int i = rt * 16 + r16;
                    float4v acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
                    const uint32_t *nb = A.nbc + (size_t)i * dr;
                    uint32_t off[kGather];
#pragma unroll
                    for (int k = 0; k < kGather; k++) off[k] = k < dr ? nb[k] : sentinel_off;
                    for (int k0 = 0; k0 < dr; k0 += kGather) {
                        bf16x8v x[kGather];
                        if constexpr (l == 0) {
                            float2 xi[kGather];
#pragma unroll
                            for (int k = 0; k < kGather; k++) xi[k] = X[off[k] >> 6];
#pragma unroll
                            for (int k = 0; k < kGather; k++) {
                                // the zero row of padded lists stays zero
                                x[k] = off[k] == sentinel_off ? bf16x8v{} : h0_group(xi[k].x, xi[k].y);
                            }
                        } else {
#pragma unroll
                            for (int k = 0; k < kGather; k++) x[k] = gload(Hb, off[k] + q16);
                        }
#pragma unroll
                        for (int k = 0; k < kGather; k++)
                            off[k] = k0 + kGather + k < dr ? nb[k0 + kGather + k] : sentinel_off;
#pragma unroll
                        for (int k = 0; k < kGather; k++) {
                            acc0 = mfma32(a0, x[k], acc0);
                            acc1 = mfma32(a1, x[k], acc1);
                        }
                    }
                    const float rd = A.rdc[i], sgn = i < m ? sg[i] : 0.f;
                    float4v v0, v1;
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        v0[q] = fmaxf(rd * acc0[q] + sgn * av0[q], 0.f);
                        v1[q] = fmaxf(rd * acc1[q] + sgn * av1[q], 0.f);
                    }
                    store_group(Cb + (size_t)i * 64 + q16, v0, v1);
                }
            }
            __syncthreads();
            // faults: h_j = relu(B h_j + b + (1/deg_j) sum_i C c_i), b entering as the accumulator
            // of B h_j; in place (own rows only).  The last layer stores no features: it applies
            // the output layer to its bf16-rounded features and writes L' for its faults.
            {
                const bf16x8v b0 = frag(l * 3 + 1, 0), b1 = frag(l * 3 + 1, 1);
                const bf16x8v c0 = frag(l * 3 + 2, 0), c1 = frag(l * 3 + 2, 1);
                const float4v bv0 = *(const float4v *)(sv + SV_BL + l * HID + 8 * q8);
                const float4v bv1 = *(const float4v *)(sv + SV_BL + l * HID + 8 * q8 + 4);
                const int ntiles = NP / 16;
                // one pass: kFaultTiles tiles, each gathering D check rows per fault (the pass's
                // largest tile degree; the tables pad shorter lists with the zero row), every load
                // issued before the first product
                auto pass = [&](auto Dc, int rt0) {
                    constexpr int D = decltype(Dc)::value;
                    bf16x8v h[kFaultTiles], y[kFaultTiles][D];
                    float2 xo[kFaultTiles];
#pragma unroll
                    for (int tt = 0; tt < kFaultTiles; tt++) {
                        const int rt = rt0 + tt * kBigWaves;
                        const int r = (rt < ntiles ? rt : rt0) * 16 + r16;
                        if constexpr (l == 0) xo[tt] = X[r];
                        else h[tt] = gload(Hb, (uint32_t)r * 64u + q16);
                        const uint16_t *nb = nbf16 + (size_t)r * dc;
#pragma unroll
                        for (int k = 0; k < D; k++) y[tt][k] = gload(Cb, (uint32_t)nb[k] * 64u + q16);
                    }
#pragma unroll
                    for (int tt = 0; tt < kFaultTiles; tt++) {
                        const int rt = rt0 + tt * kBigWaves;
                        if (rt >= ntiles) continue;
                        const int r = rt * 16 + r16;
                        if constexpr (l == 0) h[tt] = h0_group(xo[tt].x, xo[tt].y);
                        float4v an0 = {0.f, 0.f, 0.f, 0.f}, an1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int k = 0; k < D; k++) {
                            an0 = mfma32(c0, y[tt][k], an0);
                            an1 = mfma32(c1, y[tt][k], an1);
                        }
                        if (D == kFaultGather) {  // tiles heavier than kFaultGather
                            const int dt = A.tdeg[rt];
                            for (int k = kFaultGather; k < dt; k++) {
                                const bf16x8v z = gload(Cb, (uint32_t)nbf16[(size_t)r * dc + k] * 64u + q16);
                                an0 = mfma32(c0, z, an0);
                                an1 = mfma32(c1, z, an1);
                            }
                        }
                        const float4v as0 = mfma32(b0, h[tt], bv0), as1 = mfma32(b1, h[tt], bv1);
                        const float rd = A.rdf[r];
                        float4v v0, v1;
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            v0[q] = fmaxf(rd * an0[q] + as0[q], 0.f);
                            v1[q] = fmaxf(rd * an1[q] + as1[q], 0.f);
                        }
                        if constexpr (l + 1 < NL) {
                            store_group(Hb + (size_t)r * 64 + q16, v0, v1);
                        } else {
                            // output layer: d_j = b_o + w . h_j over the bf16-rounded features,
                            // 8 per lane, then summed over the 4 lanes of the fault
                            const uint32_t w[4] = {pack_bf16x2(v0[0], v0[1]), pack_bf16x2(v0[2], v0[3]),
                                                   pack_bf16x2(v1[0], v1[1]), pack_bf16x2(v1[2], v1[3])};
                            const float4v *wo = (const float4v *)(sv + SV_W + 8 * q8);
                            float d = 0.f;
#pragma unroll
                            for (int i = 0; i < 4; i++) {
                                d += wo[i >> 1][2 * (i & 1)] * __uint_as_float(w[i] << 16);
                                d += wo[i >> 1][2 * (i & 1) + 1] * __uint_as_float(w[i] & 0xffff0000u);
                            }
                            d += __shfl_xor(d, 16, 64);
                            d += __shfl_xor(d, 32, 64);
                            const int j = A.perm[r];
                            if (q8 == 0 && j >= 0) A.llr_out[(size_t)shot * n + j] = llr[j] + (sv[SV_BO] + d);
                        }
                    }
                };
                for (int rt0 = wave; rt0 < ntiles; rt0 += kFaultTiles * kBigWaves) {
                    int D = 1;
#pragma unroll
                    for (int tt = 0; tt < kFaultTiles; tt++)
                        if (rt0 + tt * kBigWaves < ntiles) D = max(D, A.tdeg[rt0 + tt * kBigWaves]);
                    switch (D) {
                        case 1: pass(std::integral_constant<int, 1>{}, rt0); break;
                        case 2: pass(std::integral_constant<int, 2>{}, rt0); break;
                        case 3: pass(std::integral_constant<int, 3>{}, rt0); break;
                        case 4: pass(std::integral_constant<int, 4>{}, rt0); break;
                        case 5: pass(std::integral_constant<int, 5>{}, rt0); break;
                        default: pass(std::integral_constant<int, kFaultGather>{}, rt0); break;
                    }
                }
            }
            __syncthreads();
        };
        static_assert(NL == 3, "layers are instantiated one by one");
        layer(std::integral_constant<int, 0>{});
        layer(std::integral_constant<int, 1>{});
        layer(std::integral_constant<int, 2>{});
    }
}

// p[0 .. n) and *q
__global__ void zero_f32(float *p, int n, float *q) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.f;
    else if (i == n) *q = 0.f;
}

__global__ void adam_kernel(float *theta, const float *grad, float *m1, float *m2, int n, float lr, float b1t, float b2t) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = grad[i];
    const float a = 0.9f * m1[i] + 0.1f * g;
    const float b = 0.999f * m2[i] + 0.001f * g * g;
    m1[i] = a;
    m2[i] = b;
    theta[i] -= lr * (a / (1.f - b1t)) / (sqrtf(b / (1.f - b2t)) + 1e-8f);
}

}  // namespace

static size_t net_shared_bytes(const DevGraph &g, bool limit) {
    size_t o[5];
    return net_shared_layout(g.n, g.m, g.nnz, limit, o);
}
static size_t net_act_bytes(const DevGraph &g, bool tight) {
    size_t o[5];
    return net_act_layout(g.n, g.m, tight, o);
}
static size_t net_train_lds(const DevGraph &g, TrainPlace p) {
    const size_t shared = net_shared_bytes(g, false);
    if (p == kTrainWorkspace) return shared;
    const size_t act = net_act_bytes(g, p == kTrainTight) + (p == kTrainLds ? kNetTransposed : 0);
    return shared + std::max(act, al16(net_flush_bytes(p)));
}
// Activations in LDS where a thread covers each fault and each check of a shot (a row's offset then fits 16
// bits) and they fit.  1,000 shots of a code of 176 faults and 88 checks: kTrainTight 131 us, in the workspace
// 761; of 150 faults and 75 checks: kTrainLds 115, in the workspace 750.
static TrainPlace net_train_place(const DevGraph &g) {
    if (std::max(pad16(g.n), pad16(g.m)) > kTrainThreads) return kTrainWorkspace;
    for (TrainPlace p : {kTrainLds, kTrainTight})
        if (net_train_lds(g, p) <= 159 * 1024) return p;
    return kTrainWorkspace;
}

// Wavefronts per inference workgroup: 11 in one workgroup when they fit in a CU's 160 KB of LDS
// (11 wavefronts need 170 VGPRs or fewer: three per SIMD), else 5 (two workgroups per CU).
static int infer_waves(const DevGraph &g) {
    const size_t sh = infer_shared_bytes(g.n, g.m, g.max_rw, g.max_cw), w = infer_wave_bytes(g.n, g.m, infer_regular(g));
    return sh + (size_t)kInferWavesMax * w <= 160 * 1024 ? kInferWavesMax : 5;
}
static size_t infer_lds_bytes(const DevGraph &g) {
    return infer_shared_bytes(g.n, g.m, g.max_rw, g.max_cw) +
           (size_t)infer_waves(g) * infer_wave_bytes(g.n, g.m, infer_regular(g));
}

// Inference launch: grid sized for the device, one wavefront per shot; the neighbour loops are
// unrolled for codes of maximum row / column weight 6 / 3 (the bivariate bicycle codes), and run
// to the code's maximum weights otherwise.
template <int UR, int UF>
static hipError_t launch_infer_t(const NetArgs &a, int max_items, int num_cus, hipStream_t st) {
    const size_t lds = infer_lds_bytes(a.g);
    hipError_t e = hipFuncSetAttribute((const void *)net_infer_kernel<UR, UF>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int nw = infer_waves(a.g);
    const int per_cu = std::max<int>(1, (int)((160 * 1024) / lds));
    const int grid = std::max(1, std::min((max_items + nw - 1) / nw, num_cus * per_cu));
    hipLaunchKernelGGL((net_infer_kernel<UR, UF>), dim3(grid), dim3(64 * nw), lds, st, a);
    return hipGetLastError();
}
static hipError_t launch_infer(const NetArgs &a, int max_items, int num_cus, hipStream_t st) {
    if (a.g.max_rw == 6 && a.g.max_cw == 3) return launch_infer_t<6, 3>(a, max_items, num_cus, st);
    return launch_infer_t<0, 0>(a, max_items, num_cus, st);
}

}  // namespace qlsd

using namespace qlsd;

struct qlsd_net_s {
    qlsd_code code;
    DevGraph g;
    float *d_lam = nullptr, *d_theta = nullptr, *d_m1 = nullptr, *d_m2 = nullptr, *d_grad = nullptr, *d_loss = nullptr;
    int step = 0;
    int num_cus = 0;
    bool wave_infer = false;          // inference by net_infer_kernel (LDS-resident, wave per shot)
    unsigned char *d_act = nullptr;   // training activations when they do not fit in LDS (lazy)
    size_t act_stride = 0;
    int act_slices = 0;
    // large-graph inference (net_infer_big_kernel): neighbour tables, and the net's own feature
    // workspace for qlsd_net_forward (decoders bring their own, see qlsd_decoder_set_net)
    uint32_t *d_nbc = nullptr, *d_nbf = nullptr;
    float *d_rdc = nullptr, *d_rdf = nullptr;
    int32_t *d_perm = nullptr, *d_rowof = nullptr, *d_tdeg = nullptr;  // fault rows sorted by degree
    unsigned char *d_iws = nullptr;
};

namespace qlsd {
// Gradient launch: one workgroup per shot at a time; activations in LDS or in the net's workspace
// slices.
static hipError_t launch_train(qlsd_net_s *net, NetArgs a, int grid, hipStream_t st) {
    if (net->act_stride && !net->d_act &&
        hipMalloc((void **)&net->d_act, net->act_stride * net->act_slices) != hipSuccess) {
        net->d_act = nullptr;
        return hipErrorOutOfMemory;
    }
    const TrainPlace place = net_train_place(a.g);
    const size_t lds = net_train_lds(a.g, place);
    if (place == kTrainWorkspace) {
        a.act = net->d_act;
        a.act_stride = net->act_stride;
        grid = std::min(grid, net->act_slices);
    }
    auto go = [&](auto kernel) {
        const hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(std::max(grid, 1)), dim3(kTrainThreads), lds, st, a);
        return hipGetLastError();
    };
    if (place == kTrainWorkspace) return go(net_train_kernel<kTrainWorkspace, 0, 0>);
    if (place == kTrainTight) return go(net_train_kernel<kTrainTight, 0, 0>);
    const DevGraph &g = a.g;
    const bool reg63 = g.min_rw == 6 && g.max_rw == 6 && g.min_cw == 3 && g.max_cw == 3;
    return reg63 ? go(net_train_kernel<kTrainLds, 6, 3>) : go(net_train_kernel<kTrainLds, 0, 0>);
}
// Slices of the large-graph inference workspace: one per compute unit, so the grid's features
// (about 0.7 MB per slice for the detector error model) stay in the last-level cache.
static int big_slices(const qlsd_net_s *net) { return net->num_cus; }
size_t net_infer_workspace_bytes(const qlsd_net_s *net) {
    return net->wave_infer ? 0 : big_slice_bytes(net->g.n, net->g.m) * (size_t)big_slices(net);
}
static hipError_t launch_infer_big(const qlsd_net_s *net, NetArgs a, unsigned char *ws, int max_items, hipStream_t st) {
    a.act = ws;
    a.act_stride = big_slice_bytes(a.g.n, a.g.m);
    a.nbc = net->d_nbc;
    a.nbf = net->d_nbf;
    a.rdc = net->d_rdc;
    a.rdf = net->d_rdf;
    a.perm = net->d_perm;
    a.tdeg = net->d_tdeg;
    const int grid = std::max(1, std::min(max_items, big_slices(net)));
    const size_t lds = big_dyn_lds(a.g);
    hipError_t e = hipFuncSetAttribute((const void *)net_infer_big_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(net_infer_big_kernel, dim3(grid), dim3(64 * kBigWaves), lds, st, a);
    return hipGetLastError();
}
// Inference of max_items shots (a.list / a.count say which); ws: a feature workspace of
// net_infer_workspace_bytes(net) for large graphs (nullptr: the net's own).
static hipError_t run_forward(qlsd_net_s *net, const NetArgs &a, int max_items, unsigned char *ws, hipStream_t st) {
    if (net->wave_infer) return launch_infer(a, max_items, net->num_cus, st);
    if (!ws) {
        if (!net->d_iws && hipMalloc((void **)&net->d_iws, net_infer_workspace_bytes(net)) != hipSuccess) {
            net->d_iws = nullptr;
            return hipErrorOutOfMemory;
        }
        ws = net->d_iws;
    }
    return launch_infer_big(net, a, ws, max_items, st);
}
}  // namespace qlsd

extern "C" {

qlsd_status qlsd_net_create(qlsd_code code, const double *priors, const float *params, qlsd_net *out) {
    if (!out || !code || !priors || !params) { set_last_error("NULL argument"); return QLSD_E_INVALID; }
    *out = nullptr;
    const DevGraph g = code_graph(code);
    // u16 CSR/CSC tables in LDS next to the weights
    if (g.n >= 65535 || g.nnz >= 65535 || net_shared_bytes(g, true) > 159 * 1024) {
        set_last_error("graph too large for the refinement network (u16 tables in LDS)");
        return QLSD_E_UNSUPPORTED;
    }
    std::vector<float> lam(g.n);
    for (int j = 0; j < g.n; j++) {
        if (!(priors[j] > 0.0 && priors[j] < 1.0)) { set_last_error("prior %d not in (0,1)", j); return QLSD_E_PRIOR; }
        lam[j] = (float)log((1.0 - priors[j]) / priors[j]);
    }
    qlsd_net net = new (std::nothrow) qlsd_net_s();
    if (!net) { set_last_error("host allocation failed"); return QLSD_E_NOMEM; }
    net->code = code;
    net->g = g;
    bool ok = hipMalloc((void **)&net->d_lam, sizeof(float) * g.n) == hipSuccess &&
              hipMalloc((void **)&net->d_theta, sizeof(float) * NPAR) == hipSuccess &&
              hipMalloc((void **)&net->d_m1, sizeof(float) * NPAR) == hipSuccess &&
              hipMalloc((void **)&net->d_m2, sizeof(float) * NPAR) == hipSuccess &&
              hipMalloc((void **)&net->d_grad, sizeof(float) * NPAR) == hipSuccess &&
              hipMalloc((void **)&net->d_loss, sizeof(float) * 4) == hipSuccess &&
              hipMemcpy(net->d_lam, lam.data(), sizeof(float) * g.n, hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(net->d_theta, params, sizeof(float) * NPAR, hipMemcpyHostToDevice) == hipSuccess &&
              hipMemset(net->d_m1, 0, sizeof(float) * NPAR) == hipSuccess &&
              hipMemset(net->d_m2, 0, sizeof(float) * NPAR) == hipSuccess;
    int dev = 0;
    hipDeviceProp_t prop;
    ok = ok && hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess;
    if (!ok) {
        qlsd_net_destroy(net);
        set_last_error("device allocation failed");
        return QLSD_E_NOMEM;
    }
    net->num_cus = prop.multiProcessorCount;
    // wave-per-shot inference needs u16 byte offsets of feature rows (64 B each) and LDS room
    net->wave_infer = pad16(g.n) + 1 <= 1023 && pad16(g.m) + 1 <= 1023 && infer_lds_bytes(g) <= 160 * 1024;
    if (net_train_place(g) == kTrainWorkspace) {  // training activations in a device workspace (allocated at first use)
        net->act_stride = (net_act_bytes(g, false) + 255) & ~size_t(255);
        net->act_slices = net->num_cus;
    }
    if (!net->wave_infer) {
        const int NP = pad16(g.n), MP = pad16(g.m);
        if (MP + 1 > 65535 || big_dyn_lds(g) + 20 * 1024 > 159 * 1024) {
            qlsd_net_destroy(net);
            set_last_error("graph too large for the refinement's inference kernel");
            return QLSD_E_UNSUPPORTED;
        }
        std::vector<int32_t> col_ptr(g.n + 1), perm, rowof, tdeg;
        ok = (size_t)(NP + 1) * 64 < (1ull << 32) && (size_t)(MP + 1) * 64 < (1ull << 32) &&
             hipMemcpy(col_ptr.data(), g.col_ptr, sizeof(int32_t) * (g.n + 1), hipMemcpyDeviceToHost) == hipSuccess;
        if (ok) big_fault_order(col_ptr, g.n, perm, rowof, tdeg);
        ok = ok && hipMalloc((void **)&net->d_nbc, sizeof(uint32_t) * (size_t)MP * g.max_rw) == hipSuccess &&
             hipMalloc((void **)&net->d_nbf, sizeof(uint32_t) * (size_t)NP * g.max_cw) == hipSuccess &&
             hipMalloc((void **)&net->d_rdc, sizeof(float) * MP) == hipSuccess &&
             hipMalloc((void **)&net->d_rdf, sizeof(float) * NP) == hipSuccess &&
             hipMalloc((void **)&net->d_perm, sizeof(int32_t) * NP) == hipSuccess &&
             hipMalloc((void **)&net->d_rowof, sizeof(int32_t) * g.n) == hipSuccess &&
             hipMalloc((void **)&net->d_tdeg, sizeof(int32_t) * (NP / 16)) == hipSuccess &&
             hipMemcpy(net->d_perm, perm.data(), sizeof(int32_t) * NP, hipMemcpyHostToDevice) == hipSuccess &&
             hipMemcpy(net->d_rowof, rowof.data(), sizeof(int32_t) * g.n, hipMemcpyHostToDevice) == hipSuccess &&
             hipMemcpy(net->d_tdeg, tdeg.data(), sizeof(int32_t) * (NP / 16), hipMemcpyHostToDevice) == hipSuccess;
        if (ok) {
            hipLaunchKernelGGL(big_tables_kernel, dim3(256), dim3(256), 0, 0, g, net->d_perm, net->d_rowof, net->d_nbc,
                               net->d_nbf, net->d_rdc, net->d_rdf);
            ok = hipGetLastError() == hipSuccess && hipDeviceSynchronize() == hipSuccess;
        }
        if (!ok) {
            qlsd_net_destroy(net);
            set_last_error("device allocation of the inference tables failed");
            return QLSD_E_NOMEM;
        }
    }
    *out = net;
    return QLSD_OK;
}

qlsd_status qlsd_net_set_priors(qlsd_net net, const double *priors) {
    if (!net || !priors) { set_last_error("NULL argument"); return QLSD_E_INVALID; }
    std::vector<float> lam(net->g.n);
    for (int j = 0; j < net->g.n; j++) {
        if (!(priors[j] > 0.0 && priors[j] < 1.0)) { set_last_error("prior %d not in (0,1)", j); return QLSD_E_PRIOR; }
        lam[j] = (float)log((1.0 - priors[j]) / priors[j]);
    }
    if (hipMemcpy(net->d_lam, lam.data(), sizeof(float) * net->g.n, hipMemcpyHostToDevice) != hipSuccess) {
        set_last_error("hipMemcpy failed");
        return QLSD_E_DEVICE;
    }
    return QLSD_OK;
}

qlsd_status qlsd_net_set_params(qlsd_net net, const float *params) {
    if (!net || !params) { set_last_error("NULL argument"); return QLSD_E_INVALID; }
    if (hipMemcpy(net->d_theta, params, sizeof(float) * NPAR, hipMemcpyHostToDevice) != hipSuccess) {
        set_last_error("hipMemcpy failed");
        return QLSD_E_DEVICE;
    }
    return QLSD_OK;
}

qlsd_status qlsd_net_get_params(qlsd_net net, float *params) {
    if (!net || !params) { set_last_error("NULL argument"); return QLSD_E_INVALID; }
    if (hipDeviceSynchronize() != hipSuccess ||
        hipMemcpy(params, net->d_theta, sizeof(float) * NPAR, hipMemcpyDeviceToHost) != hipSuccess) {
        set_last_error("hipMemcpy failed");
        return QLSD_E_DEVICE;
    }
    return QLSD_OK;
}

static NetArgs net_args(qlsd_net net) {
    NetArgs a;
    memset(&a, 0, sizeof(a));
    a.g = net->g;
    a.lam = net->d_lam;
    a.theta = net->d_theta;
    return a;
}

qlsd_status qlsd_net_forward(qlsd_net net, const uint8_t *syndromes, const float *llr, int32_t B, float *llr_out,
                             void *stream) {
    if (!net || B < 0 || (B > 0 && (!syndromes || !llr || !llr_out))) { set_last_error("bad arguments"); return QLSD_E_INVALID; }
    if (B == 0) return QLSD_OK;
    NetArgs a = net_args(net);
    a.syn = syndromes;
    a.llr = llr;
    a.llr_out = llr_out;
    a.count = B;
    if (run_forward(net, a, B, nullptr, (hipStream_t)stream) != hipSuccess) {
        set_last_error("net launch failed");
        return QLSD_E_DEVICE;
    }
    return QLSD_OK;
}

static qlsd_status grad_impl(qlsd_net net, const uint8_t *syn, const float *llr, const uint8_t *err, int32_t B,
                             float *grad, float *loss, hipStream_t st) {
    hipLaunchKernelGGL(zero_f32, dim3((NPAR + 1 + 255) / 256), dim3(256), 0, st, grad, NPAR, loss);
    NetArgs a = net_args(net);
    a.syn = syn;
    a.llr = llr;
    a.err = err;
    a.count = B;
    a.grad = grad;
    a.loss = loss;
    a.inv_total = 1.f / ((float)B * (float)net->g.n);
    const int grid = std::min(B, net->num_cus);
    if (launch_train(net, a, grid, st) != hipSuccess) { set_last_error("net launch failed"); return QLSD_E_DEVICE; }
    return QLSD_OK;
}

qlsd_status qlsd_net_gradient(qlsd_net net, const uint8_t *syndromes, const float *llr, const uint8_t *errors,
                              int32_t B, float *grad, float *loss, void *stream) {
    if (!net || B < 1 || !syndromes || !llr || !errors || !grad || !loss) { set_last_error("bad arguments"); return QLSD_E_INVALID; }
    return grad_impl(net, syndromes, llr, errors, B, grad, loss, (hipStream_t)stream);
}

qlsd_status qlsd_net_train_step(qlsd_net net, const uint8_t *syndromes, const float *llr, const uint8_t *errors,
                                int32_t B, float lr, void *stream) {
    if (!net || B < 1 || !syndromes || !llr || !errors) { set_last_error("bad arguments"); return QLSD_E_INVALID; }
    hipStream_t st = (hipStream_t)stream;
    qlsd_status s = grad_impl(net, syndromes, llr, errors, B, net->d_grad, net->d_loss, st);
    if (s != QLSD_OK) return s;
    net->step++;
    const float b1t = powf(0.9f, (float)net->step), b2t = powf(0.999f, (float)net->step);
    hipLaunchKernelGGL(adam_kernel, dim3((NPAR + 255) / 256), dim3(256), 0, st, net->d_theta, net->d_grad, net->d_m1,
                       net->d_m2, NPAR, lr, b1t, b2t);
    if (hipGetLastError() != hipSuccess) { set_last_error("adam launch failed"); return QLSD_E_DEVICE; }
    return QLSD_OK;
}

void qlsd_net_destroy(qlsd_net net) {
    if (!net) return;
    hipFree(net->d_lam);
    hipFree(net->d_theta);
    hipFree(net->d_m1);
    hipFree(net->d_m2);
    hipFree(net->d_grad);
    hipFree(net->d_loss);
    hipFree(net->d_act);
    hipFree(net->d_nbc);
    hipFree(net->d_nbf);
    hipFree(net->d_rdc);
    hipFree(net->d_rdf);
    hipFree(net->d_perm);
    hipFree(net->d_rowof);
    hipFree(net->d_tdeg);
    hipFree(net->d_iws);
    delete net;
}

}  // extern "C"

namespace qlsd {
// Refinement of the LLRs of the listed shots, in place (decode path).
hipError_t net_refine_listed(qlsd_net_s *net, const float *lam, const uint8_t *syn, float *llr, const int *list,
                             const int *list_count, int max_count, unsigned char *ws, hipStream_t st) {
    NetArgs a = net_args(net);
    a.lam = lam;  // the decoder's prior LLRs, so one net serves decoders of any noise strength
    a.syn = syn;
    a.llr = llr;
    a.llr_out = llr;
    a.list = list;
    a.list_count = list_count;
    a.count = max_count;
    return run_forward(net, a, max_count, ws, st);
}
void net_graph_dims(const qlsd_net_s *net, int *m, int *n) {
    *m = net->g.m;
    *n = net->g.n;
}
const float *net_loss_ptr(qlsd_net net) { return net->d_loss; }
}  // namespace qlsd
