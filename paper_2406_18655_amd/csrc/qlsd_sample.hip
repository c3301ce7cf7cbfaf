// Code-capacity noise on the GPU: Philox4x64-10 uniforms (Salmon et al., SC'11), e_j = [u < p_j],
// s = H e, and logical-failure flags of residuals.  The stream convention is stated in
// include/qlsd_sample.h; every thread computes one Philox block (four consecutive outputs of one
// key), so a shot row's faults come from consecutive counters of its 4096-shot block.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "../../include/qlsd_sample.h"
#include "qlsd_internal.h"

using namespace qlsd;

struct qlsd_sampler_s {
    qlsd_code code;
    DevGraph g;
    uint64_t *d_thr;   // n: a fault flips iff its 64-bit output is below this
    int k;             // logical rows (0: word error)
    int parts;         // threads that share a logical row (failure_kernel)
    int64_t ones, steps;  // entries of the logical rows; 64-entry steps of failure_wide_kernel over a shot
    int *d_lrp, *d_lci;
};

namespace {

constexpr int kBlockShots = 4096;

// Published Philox4x64 constants: round multipliers and Weyl key increments.
constexpr uint64_t kM0 = 0xD2E7470EE14C6C93ull, kM1 = 0xCA5A826395121157ull;
constexpr uint64_t kW0 = 0x9E3779B97F4A7C15ull, kW1 = 0xBB67AE8584CAA73Bull;

__device__ __forceinline__ void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1) {
#pragma unroll
    for (int r = 0; r < 10; r++) {
        if (r) { k0 += kW0; k1 += kW1; }
        const uint64_t lo0 = kM0 * c[0], hi0 = __umul64hi(kM0, c[0]);
        const uint64_t lo1 = kM1 * c[2], hi1 = __umul64hi(kM1, c[2]);
        const uint64_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
    }
}

// One thread per Philox block: the four outputs 4w .. 4w + 3 of one 4096-shot block's key are four
// consecutive bytes of the row-major error array, written as one word where it is aligned.  Whether
// u = (x >> 11) 2^-53 < p is decided on the integers (x < thr, thr = ceil(2^53 p) << 11).  Bound by the
// generator's 64 x 64-bit products: 65,536 shots of 144 faults 38.6 -> 25.0 us (with 64-bit divisions and a byte
// store per output before).
// w0 .. w1: the words of every block that can hold requested shots; blockIdx.y: 4096-shot block.
__global__ __launch_bounds__(256) void sample_errors_kernel(const uint64_t *thr, int n, uint32_t magic, uint64_t seed,
                                                            int64_t start, int B, uint8_t *e, int64_t first_block,
                                                            int64_t w0, int64_t w1) {
    const int64_t w = w0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= w1) return;
    const int64_t blk = first_block + blockIdx.y;
    // output 4w of the block is byte `at` of the error array
    const int64_t at = (blk * kBlockShots - start) * n + 4 * w, total = (int64_t)B * n;
    if (at + 3 < 0 || at >= total) return;
    uint64_t c[4] = {(uint64_t)w + 1ull, 0ull, 0ull, 0ull};  // counter w + 1 of this block's key
    philox4x64_10(c, seed, (uint64_t)blk);
    // fault of output 4w: 4w mod n, by a multiply-high with ceil(2^32 / n) (at most one too large for
    // 4w < 2^32), or by division where 4w may not fit
    int j;
    if (magic) {
        const uint32_t q = (uint32_t)(4 * w);
        j = (int)(q - __umulhi(q, magic) * (uint32_t)n);
        if (j < 0) j += n;
    } else {
        j = (int)((4 * w) % n);
    }
    uint32_t bytes = 0;
#pragma unroll
    for (int u = 0; u < 4; u++) {
        bytes |= (c[u] < thr[j] ? 1u : 0u) << (8 * u);
        j = j + 1 == n ? 0 : j + 1;
    }
    if (at >= 0 && at + 3 < total && (((uintptr_t)e + (uintptr_t)at) & 3) == 0) {
        *(uint32_t *)(e + at) = bytes;
    } else {
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (at + u >= 0 && at + u < total) e[at + u] = (uint8_t)((bytes >> (8 * u)) & 1u);
    }
}

// Bit-sliced shots: a workgroup takes `words` groups of 32 shots and holds, per fault, one 32-bit word
// per group (bit s: shot s), so one exclusive or serves 32 shots.  Reading the byte rows once, as words,
// is what is left: 65,536 shots of [[144,12,12]] syndromes 35.7 -> 6.3 us, failures 54.8 -> 9.7 us (a
// thread per detector, or a wavefront per shot, read single bytes before).
constexpr int kMaxWords = 8;

// Fills bits[j * words + g] with bit 0 of x[shot][j] (xor y[shot][j]) over the 32 shots of group g.
template <bool TWO>
__device__ __forceinline__ void slice_rows(const uint8_t *x, const uint8_t *y, int n, int B, int64_t shot0, int words,
                                           uint32_t *bits) {
    const bool wide = (n & 3) == 0 && (((uintptr_t)x | (TWO ? (uintptr_t)y : 0)) & 3) == 0;
    const int per = wide ? n / 4 : n;  // loads per row
    for (int it = threadIdx.x; it < per * words; it += blockDim.x) {
        const int g = it / per, q = it - g * per;
        const int64_t b0 = shot0 + 32 * g;
        const int rows = (int)min((int64_t)32, B - b0);
        if (wide) {
            // byte k of acc[s / 8]: bit s mod 8 = fault 4q + k of shot s
            uint32_t acc[4] = {0u, 0u, 0u, 0u};
            const uint8_t *px = x + b0 * n + 4 * q, *py = TWO ? y + b0 * n + 4 * q : nullptr;
            if (rows == 32) {
#pragma unroll
                for (int s = 0; s < 32; s++) {
                    uint32_t v = *(const uint32_t *)(px + (int64_t)s * n);
                    if (TWO) v ^= *(const uint32_t *)(py + (int64_t)s * n);
                    acc[s >> 3] |= (v & 0x01010101u) << (s & 7);
                }
            } else {
                for (int s = 0; s < rows; s++) {
                    uint32_t v = *(const uint32_t *)(px + (int64_t)s * n);
                    if (TWO) v ^= *(const uint32_t *)(py + (int64_t)s * n);
                    const uint32_t m = (v & 0x01010101u) << (s & 7);
#pragma unroll
                    for (int k = 0; k < 4; k++) acc[k] |= (s >> 3) == k ? m : 0u;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; k++)
                bits[(4 * q + k) * words + g] = ((acc[0] >> (8 * k)) & 0xffu) | ((acc[1] >> (8 * k)) & 0xffu) << 8 |
                                                ((acc[2] >> (8 * k)) & 0xffu) << 16 | ((acc[3] >> (8 * k)) & 0xffu) << 24;
        } else {
            uint32_t acc = 0u;
            for (int s = 0; s < rows; s++) {
                uint32_t v = x[(b0 + s) * n + q];
                if (TWO) v ^= y[(b0 + s) * n + q];
                acc |= (v & 1u) << s;
            }
            bits[q * words + g] = acc;
        }
    }
}

// s = H x: per detector and group, the exclusive or of its faults' words; then the rows as bytes.
__global__ void syndrome_kernel(const int32_t *row_ptr, const int32_t *col_idx, int m, int n, int B, int words,
                                const uint8_t *x, uint8_t *s) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *bits = (uint32_t *)smem, *sw = bits + (size_t)n * words;
    const int64_t shot0 = (int64_t)blockIdx.x * 32 * words;
    slice_rows<false>(x, nullptr, n, B, shot0, words, bits);
    __syncthreads();
    for (int it = threadIdx.x; it < m * words; it += blockDim.x) {
        const int i = it / words, g = it - i * words;
        uint32_t acc = 0u;
        for (int e = row_ptr[i]; e < row_ptr[i + 1]; e++) acc ^= bits[col_idx[e] * words + g];
        sw[it] = acc;
    }
    __syncthreads();
    const int shots = (int)min((int64_t)32 * words, B - shot0);
    uint8_t *out = s + shot0 * m;
    if ((m & 3) == 0 && (((uintptr_t)s) & 3) == 0) {
        const int per = m / 4;
        for (int it = threadIdx.x; it < per * shots; it += blockDim.x) {
            const int b = it / per, i = 4 * (it - b * per);
            const uint32_t *w = sw + i * words + (b >> 5);
            uint32_t v = 0u;
#pragma unroll
            for (int k = 0; k < 4; k++) v |= ((w[k * words] >> (b & 31)) & 1u) << (8 * k);
            *(uint32_t *)(out + 4 * (int64_t)it) = v;
        }
    } else {
        for (int it = threadIdx.x; it < m * shots; it += blockDim.x) {
            const int b = it / m, i = it - b * m;
            out[it] = (uint8_t)((sw[i * words + (b >> 5)] >> (b & 31)) & 1u);
        }
    }
}

// Residual parity against each logical row (k = 0: any nonzero fault), 32 shots a word.  `parts` threads
// share a row of one group (1: rows of at most kPart entries): one thread per row takes 380 us for a single
// row of 4,400 entries, where the rest takes 12.
constexpr int kPart = 16;
__global__ void failure_kernel(const uint8_t *e, const uint8_t *c, int n, int B, int k, const int *lrp, const int *lci,
                               int parts, int words, uint8_t *fail) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *bits = (uint32_t *)smem, *fw = bits + (size_t)n * words;
    uint32_t *par = fw + words;  // parts > 1: each row's parity, k per group
    const int64_t shot0 = (int64_t)blockIdx.x * 32 * words;
    if (threadIdx.x < words) fw[threadIdx.x] = 0u;
    if (parts > 1)
        for (int it = threadIdx.x; it < k * words; it += blockDim.x) par[it] = 0u;
    slice_rows<true>(e, c, n, B, shot0, words, bits);
    __syncthreads();
    if (k == 0) {
        for (int g = 0; g < words; g++) {
            uint32_t any = 0u;
            for (int j = threadIdx.x; j < n; j += blockDim.x) any |= bits[j * words + g];
            if (any) atomicOr(&fw[g], any);
        }
    } else {
        for (int64_t it = threadIdx.x; it < (int64_t)k * words * parts; it += blockDim.x) {
            const int row = (int)(it / parts), q = row / words, g = row - q * words;
            uint32_t acc = 0u;
            for (int x = lrp[q] + (int)(it - (int64_t)row * parts); x < lrp[q + 1]; x += parts) acc ^= bits[lci[x] * words + g];
            if (acc && parts == 1) atomicOr(&fw[g], acc);
            if (acc && parts > 1) atomicXor(&par[row], acc);
        }
        if (parts > 1) {
            __syncthreads();
            for (int it = threadIdx.x; it < k * words; it += blockDim.x)
                if (par[it]) atomicOr(&fw[it % words], par[it]);
        }
    }
    __syncthreads();
    const int shots = (int)min((int64_t)32 * words, B - shot0);
    for (int b = threadIdx.x; b < shots; b += blockDim.x) fail[shot0 + b] = (uint8_t)((fw[b >> 5] >> (b & 31)) & 1u);
}

// For matrices whose bit-sliced shots do not fit in LDS (more than about 35,000 faults), and where they
// are faster (syndromes_by_shot, failures_by_shot): a thread per (shot, detector), and a wavefront per shot.
__global__ void syndrome_wide_kernel(const int32_t *row_ptr, const int32_t *col_idx, int m, int n, int B,
                                     const uint8_t *x, uint8_t *s) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)B * m) return;
    const int64_t b = t / m;
    const int i = (int)(t % m);
    const uint8_t *row = x + b * n;
    uint8_t acc = 0;
    for (int e = row_ptr[i]; e < row_ptr[i + 1]; e++) acc ^= row[col_idx[e]];
    s[t] = acc & 1;
}
__global__ void failure_wide_kernel(const uint8_t *e, const uint8_t *c, int n, int B, int k, const int *lrp,
                                    const int *lci, uint8_t *fail) {
    const int lane = threadIdx.x & 63;
    const int64_t b = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    if (b >= B) return;
    const uint8_t *er = e + b * n, *cr = c + b * n;
    bool f = false;
    if (k == 0) {
        bool any = false;
        for (int j = lane; j < n; j += 64) any |= (er[j] ^ cr[j]) & 1;
        f = __ballot(any) != 0ull;
    } else {
        for (int q = 0; q < k && !f; q++) {
            int par = 0;
            for (int x = lrp[q] + lane; x < lrp[q + 1]; x += 64) par ^= (er[lci[x]] ^ cr[lci[x]]) & 1;
            f = (__popcll(__ballot(par != 0)) & 1) != 0;
        }
    }
    if (lane == 0) fail[b] = f ? 1 : 0;
}

// Groups of 32 shots per workgroup (0: the sliced rows do not fit), its threads and LDS; extra: LDS words
// per group beside the n of the rows.  Small matrices take up to kMaxWords groups while about two
// workgroups per compute unit remain; large ones one, on 1024 threads.
struct Slices { int words, threads; size_t lds; };
Slices slices_for(int n, int extra, int B) {
    constexpr size_t kLds = 150 * 1024, kShare = 24 * 1024;
    Slices s{0, 256, 0};
    const size_t per = sizeof(uint32_t) * ((size_t)n + extra);
    if (per > kLds) return s;
    s.words = 1;
    while (s.words < kMaxWords && 2 * s.words * per <= kShare && (int64_t)B > (int64_t)32 * 2 * s.words * 512) s.words *= 2;
    if (n > 2048) s.threads = 1024;
    s.lds = per * s.words;
    return s;
}

// Whether failure_wide_kernel is the faster one: it reads only the entries of the logical rows, the
// bit-sliced kernel every fault, 32 shots to a workgroup at least.  Its time follows the 64-entry steps of
// a shot, one after the other (every row waits for the one before), the steps of all shots and the cache
// lines they touch; the sliced kernel's the whole rows.  In us beyond a launch, fitted to both kernels over
// 41 to 8,800 faults, no, 1 to 64 logical rows of 5 to 4,400 entries and 8 to 65,536 shots (the slower one
// costs up to 5x: 65,536 shots of 2,000 faults with one row of 5, 14 us against 60; 20,000 shots of 2,000
// faults with 64 rows of 40, 308 against 24; 200 shots of 8,800 with 8 rows of 1,100, 33 against 15).  Over
// that grid the choice is within 14% of the faster one but for a single row of thousands (up to 1.9x).
bool failures_by_shot(int n, int k, int64_t ones, int64_t steps, int B) {
    const double rows = k > 0 ? k : 1, lines = std::min(2.0 * (k > 0 ? (double)ones : (double)n), n / 64.0 + 2.0);
    const double chain = rows + 0.35 * ((double)steps - rows);
    const double shot = 0.3 * std::max(chain - 8.0, 0.0) + (2.5e-5 * (double)steps + 2e-5 * lines) * B;
    const double wide = (n > 1024 ? 2.0 : 0.0) + (n > 4096 ? 3.0 : 0.0);
    const double sliced = 4.0 + wide * std::min(B, 32) / 32.0 + (double)B * n / 2.8e6;
    return shot <= sliced;
}

// Whether syndrome_wide_kernel (a thread per detector of a shot) is the faster one: few shots in groups of
// 32 leave most of the device idle.  Its time follows the entries of all shots' checks, and the longest
// check where that is long; the sliced kernel's hardly changes.  Measured over 41 to 8,800 faults, both
// in us beside a launch: 100 shots of 8,800 faults (26,672 entries) 9.9 against 17.6, 300 shots 21.6 / 18.7;
// 300 shots of 1,600 (5,425 entries) 7.8 / 9.5, 1,000 shots 10.3 / 9.2; 1,000 shots of 900 (3,051 entries)
// 7.7 / 8.0, 3,000 shots 13.6 / 8.4; checks of about 85 entries 18 / 15 at any number of shots.
bool syndromes_by_shot(const DevGraph &g, int B) { return g.max_rw <= 48 && (int64_t)B * g.nnz < 3500000; }

qlsd_status sfail(qlsd_status st, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    char buf[256];
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    set_last_error("%s", buf);
    return st;
}

}  // namespace

extern "C" {

qlsd_status qlsd_sampler_create(qlsd_code code, const double *priors, int32_t k, const int32_t *l_row_ptr,
                                const int32_t *l_col_idx, qlsd_sampler *out) {
    set_last_error("");
    if (!out) return sfail(QLSD_E_INVALID, "out is NULL");
    *out = nullptr;
    if (!code || !priors || k < 0 || (k > 0 && (!l_row_ptr || !l_col_idx)))
        return sfail(QLSD_E_INVALID, "NULL code/priors or bad logicals");
    const DevGraph g = code_graph(code);
    for (int j = 0; j < g.n; j++)
        if (!(priors[j] > 0.0 && priors[j] < 1.0)) return sfail(QLSD_E_PRIOR, "prior %d = %g not in (0,1)", j, priors[j]);
    const int nl = k > 0 ? l_row_ptr[k] : 0;
    for (int x = 0; x < nl; x++)
        if (l_col_idx[x] < 0 || l_col_idx[x] >= g.n) return sfail(QLSD_E_INVALID, "logical column out of range");
    qlsd_sampler s = new (std::nothrow) qlsd_sampler_s();
    if (!s) return sfail(QLSD_E_NOMEM, "host allocation failed");
    s->code = code;
    s->g = g;
    s->k = k;
    int heaviest = 0;
    s->ones = nl;
    s->steps = k > 0 ? 0 : (g.n + 63) / 64;
    for (int q = 0; q < k; q++) {
        const int w = l_row_ptr[q + 1] - l_row_ptr[q];
        heaviest = std::max(heaviest, w);
        s->steps += (w + 63) / 64;
    }
    s->parts = std::max(1, (heaviest + kPart - 1) / kPart);
    // (x >> 11) 2^-53 < p  <=>  x >> 11 < ceil(2^53 p)  <=>  x < ceil(2^53 p) << 11; p < 1, so 2^53 p, which
    // is exact, is below 2^53
    uint64_t *thr = new (std::nothrow) uint64_t[g.n];
    hipError_t e = thr ? hipMalloc((void **)&s->d_thr, sizeof(uint64_t) * g.n) : hipErrorOutOfMemory;
    for (int j = 0; thr && j < g.n; j++) thr[j] = (uint64_t)ceil(priors[j] * 0x1p53) << 11;
    if (e == hipSuccess) e = hipMemcpy(s->d_thr, thr, sizeof(uint64_t) * g.n, hipMemcpyHostToDevice);
    delete[] thr;
    if (e == hipSuccess) e = hipMalloc((void **)&s->d_lrp, sizeof(int) * (k + 1));
    if (e == hipSuccess && k > 0) e = hipMemcpy(s->d_lrp, l_row_ptr, sizeof(int) * (k + 1), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMalloc((void **)&s->d_lci, sizeof(int) * (nl > 0 ? nl : 1));
    if (e == hipSuccess && nl > 0) e = hipMemcpy(s->d_lci, l_col_idx, sizeof(int) * nl, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        qlsd_sampler_destroy(s);
        return sfail(QLSD_E_NOMEM, "sampler device allocation failed: %s", hipGetErrorString(e));
    }
    *out = s;
    return QLSD_OK;
}

qlsd_status qlsd_sample(qlsd_sampler s, uint64_t seed, int64_t start, int32_t B, uint8_t *errors,
                        uint8_t *syndromes, void *stream) {
    set_last_error("");
    if (!s || start < 0 || B < 0 || (B > 0 && !errors)) return sfail(QLSD_E_INVALID, "bad sampler call");
    if (B == 0) return QLSD_OK;
    hipStream_t st = (hipStream_t)stream;
    const int n = s->g.n;
    const int64_t first = start / kBlockShots, last = (start + B - 1) / kBlockShots;
    // words of a block: all of them, or, within one block, those of the requested shots
    int64_t w0 = 0, w1 = (int64_t)kBlockShots / 4 * n;
    if (first == last) {
        const int64_t r0 = start - first * kBlockShots;
        w0 = r0 * n / 4;
        w1 = ((r0 + B) * n + 3) / 4;
    }
    const uint32_t magic = n > 1 && (int64_t)kBlockShots * n < (1ll << 31) ? (uint32_t)(((1ull << 32) + n - 1) / n) : 0u;
    const int64_t gx = (w1 - w0 + 255) / 256;
    // at most 65,535 blocks of 4096 shots a launch
    for (int64_t b0 = first; b0 <= last; b0 += 65535)
        hipLaunchKernelGGL(sample_errors_kernel, dim3((unsigned)gx, (unsigned)std::min<int64_t>(65535, last - b0 + 1)),
                           dim3(256), 0, st, s->d_thr, n, magic, seed, start, B, errors, b0, w0, w1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sfail(QLSD_E_DEVICE, "sample launch: %s", hipGetErrorString(e));
    if (syndromes) return qlsd_syndromes(s, errors, B, syndromes, stream);
    return QLSD_OK;
}

qlsd_status qlsd_syndromes(qlsd_sampler s, const uint8_t *x, int32_t B, uint8_t *syndromes, void *stream) {
    set_last_error("");
    if (!s || B < 0 || (B > 0 && (!x || !syndromes))) return sfail(QLSD_E_INVALID, "bad syndrome call");
    if (B == 0) return QLSD_OK;
    const Slices k = slices_for(s->g.n, s->g.m, B);
    hipError_t e = hipSuccess;
    if (k.words > 0 && !syndromes_by_shot(s->g, B)) {
        e = hipFuncSetAttribute((const void *)syndrome_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds);
        if (e != hipSuccess) return sfail(QLSD_E_DEVICE, "syndrome launch: %s", hipGetErrorString(e));
        const int64_t shots = 32ll * k.words;
        hipLaunchKernelGGL(syndrome_kernel, dim3((unsigned)((B + shots - 1) / shots)), dim3(k.threads), k.lds,
                           (hipStream_t)stream, s->g.row_ptr, s->g.col_idx, s->g.m, s->g.n, B, k.words, x, syndromes);
    } else {
        const int64_t total = (int64_t)B * s->g.m;
        hipLaunchKernelGGL(syndrome_wide_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                           s->g.row_ptr, s->g.col_idx, s->g.m, s->g.n, B, x, syndromes);
    }
    e = hipGetLastError();
    return e == hipSuccess ? QLSD_OK : sfail(QLSD_E_DEVICE, "syndrome launch: %s", hipGetErrorString(e));
}

qlsd_status qlsd_failures(qlsd_sampler s, const uint8_t *errors, const uint8_t *corrections, int32_t B,
                          uint8_t *fail, void *stream) {
    set_last_error("");
    if (!s || B < 0 || (B > 0 && (!errors || !corrections || !fail))) return sfail(QLSD_E_INVALID, "bad failure call");
    if (B == 0) return QLSD_OK;
    const Slices k = slices_for(s->g.n, s->parts > 1 ? 1 + s->k : 1, B);
    hipError_t e = hipSuccess;
    if (k.words > 0 && !failures_by_shot(s->g.n, s->k, s->ones, s->steps, B)) {
        e = hipFuncSetAttribute((const void *)failure_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds);
        if (e != hipSuccess) return sfail(QLSD_E_DEVICE, "failure launch: %s", hipGetErrorString(e));
        const int64_t shots = 32ll * k.words;
        hipLaunchKernelGGL(failure_kernel, dim3((unsigned)((B + shots - 1) / shots)), dim3(k.threads), k.lds,
                           (hipStream_t)stream, errors, corrections, s->g.n, B, s->k, s->d_lrp, s->d_lci, s->parts, k.words, fail);
    } else {
        hipLaunchKernelGGL(failure_wide_kernel, dim3((unsigned)((B + 3) / 4)), dim3(256), 0, (hipStream_t)stream, errors,
                           corrections, s->g.n, B, s->k, s->d_lrp, s->d_lci, fail);
    }
    e = hipGetLastError();
    return e == hipSuccess ? QLSD_OK : sfail(QLSD_E_DEVICE, "failure launch: %s", hipGetErrorString(e));
}

void qlsd_sampler_destroy(qlsd_sampler s) {
    if (!s) return;
    hipFree(s->d_thr);
    hipFree(s->d_lrp);
    hipFree(s->d_lci);
    delete s;
}

}  // extern "C"
