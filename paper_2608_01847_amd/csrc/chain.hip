// End-to-end chaining of the scale-learning step: the transposed weight operand of dX_hat = dY W_hat
// (fp32, and bf16 shapes that dx_mfma_kernel does not take) and the KL-Top objective on logits (Sec. 4.1: the paper trains end to end with the KL-Top loss,
// k = 1000, following the method it cites for that loss).
#include <cmath>
#include <type_traits>

#include "focus_device.h"
#include "internal.h"

namespace focus {

namespace {

// ------------------------------------------------------------------------------------------------
// out[c][r] = in[r][c] for an R x C matrix, 64 x 64 tiles staged through LDS (rows of 64 elements
// read and written contiguously; the padded column breaks bank conflicts of the transposed reads).
template <typename T>
__global__ void __launch_bounds__(256) transpose_kernel(const T *__restrict__ in, int64_t R, int64_t C,
                                                         T *__restrict__ out) {
    __shared__ T tile[64][65];
    const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int i = ty; i < 64; i += 4) {
        const int64_t r = r0 + i, c = c0 + tx;
        if (r < R && c < C) tile[i][tx] = in[r * C + c];
    }
    __syncthreads();
    for (int i = ty; i < 64; i += 4) {
        const int64_t c = c0 + i, r = r0 + tx;
        if (c < C && r < R) out[c * R + r] = tile[tx][i];
    }
}

// ------------------------------------------------------------------------------------------------
// KL-Top. Keys order fp32 values as unsigned integers (negative values flipped, positive ones with
// the sign bit set); -0 is taken as +0 so that equal values have equal keys.
__device__ __forceinline__ uint32_t order_key(float f) {
    uint32_t b = __float_as_uint(f);
    b = b == 0x80000000u ? 0u : b;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

template <int IN>
__device__ __forceinline__ float load_logit(const void *p, int64_t i) {
    if (IN == kBF16) return bf16_bits_to_f32(reinterpret_cast<const uint16_t *>(p)[i]);
    return reinterpret_cast<const float *>(p)[i];
}

// the key of logit i; for bf16 logits only the high 16 bits carry information (the low half of a
// flipped negative value would be all ones), so they alone are kept
template <int IN>
__device__ __forceinline__ uint32_t logit_key(float v) {
    const uint32_t k = order_key(v);
    return IN == kBF16 ? (k & 0xFFFF0000u) : k;
}

template <int IN>
__device__ __forceinline__ void store_logit(void *p, int64_t i, float v) {
    if (IN == kBF16) reinterpret_cast<uint16_t *>(p)[i] = (uint16_t)f32_to_bf16_bits(v);
    else reinterpret_cast<float *>(p)[i] = v;
}

// Logits of elements base + t + 256 u (u = 0 .. kTrips - 1) of a row: a thread's next kTrips elements
// in its usual order, loaded before any is used so that kTrips loads are in flight at once (the passes
// are bound by the latency of rows that no longer fit the caches: 16 in flight took the 8192 x 151936
// call from 9.2 to 7.3 ms, 8 or 32 less far). An index past the row is clamped to its last element
// (V >= 1), so every load is unconditional and in bounds; the callers ignore those positions. The
// element order of each thread, and so every result bit, is that of one element per trip.
constexpr int kTrips = 16;
template <int IN>
__device__ __forceinline__ void load_trips(const void *p, int64_t base, int t, int64_t V, float (&v)[kTrips]) {
#pragma unroll
    for (int u = 0; u < kTrips; u++) {
        const int64_t i = base + t + 256 * u;
        v[u] = load_logit<IN>(p, i < V ? i : V - 1);
    }
}

// inclusive scan of one value per thread over the workgroup (256 threads), in thread order
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *buf) {
    const int t = threadIdx.x;
    buf[t] = v;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const uint32_t add = t >= off ? buf[t - off] : 0u;
        __syncthreads();
        buf[t] += add;
        __syncthreads();
    }
    const uint32_t r = buf[t];
    __syncthreads();
    return r;
}

// One workgroup per token row, in one of two ways. Both give the same selected set (the teacher's k
// largest logits, ties at the k-th value in index order) and the same per-element formulas; the sums
// run in a fixed order in each, so every result is deterministic.
//  * Sample-select (SAMPLE), when the k largest are a small part of a row (see kl_sample_rank): the r-th largest of 3,072 teacher keys,
//    r with a binomial margin of 3 standard deviations over the expected count, lies below the k-th
//    largest key almost always (10 rows of 8,192 miss at k = 1,000 of 151,936 on independent logits). The
//    sample is 384 evenly spaced runs of 8 adjacent keys (keys spaced singly touch nearly every memory line
//    of the row). A sample that misleads (logits correlated along the row) costs time only, never a result.
//    One pass over both rows, 16 bytes per load, gathers the elements at or above that key (about 1.8 k) into
//    per-wave LDS lists in index order; the k-th largest key, the tie cut (up to kTieMax ties at it), the
//    softmax statistics and the KL terms then come from LDS, and dZ leaves once, in order: a segment of the
//    row at a time, zeros with the gathered elements' gradients scattered into them in LDS, as 16-byte stores.
//    Bound by memory on long rows (two reads of the logits' rows, one write; the sample re-reads up to a
//    tenth) and by the latency of the LDS phases, which the rows per CU (bf16 four, fp32 three) hide for each other, on
//    short ones.
//    8,192 x 151,936 bf16 logits, k = 1,000: 1.78 ms (4.2 TB/s), where 2-byte loads, zeros stored on the way and
//    the gathered elements' gradients scattered over them took 2.26; 4,096 x 32,000: 0.21 ms (3.7 TB/s).
//  * The passes below whenever the gathered set misses the k-th largest key, overflows the lists or
//    holds too many ties, or the row is short or k large: a radix select of the k-th largest teacher key (8-bit digits from
//    the top, LDS histograms); if fewer ties at that key are admitted than exist, the index of the
//    last admitted tie (256 elements per trip, ballots for the in-trip ranks); online softmax
//    statistics of both rows over the selected set (per thread, then a fixed tree); KL terms and dZ_s
//    (zero outside the set). Rows that never take the sample have a kernel without it: as one kernel with it, whose
//    LDS lets three fp32 rows onto a CU, 1,000 x 60,000 fp32 logits at k = 1,900 took 833 us, now 677 (805 before the
//    two ways shared their LDS), 4,000 x 12,000 bf16 ones at 2,500 586, now 525.
constexpr int kSample = 3072;          // sampled teacher keys (12 per thread)
constexpr int kCand = 3072;            // gathered elements (LDS lists of 768 per wave)
constexpr int kPerWave = kCand / 4;
// Shortest row of the sample: its runs of 8 keys are 10 elements apart or more, and k = 1,000 passes
// the rule on r below from V = 4,472 on. (4,096 x 32,000 takes 1.34 ms by the passes, 0.21 by the
// sample.)
constexpr int64_t kSampleMinV = 4096;
constexpr int kTieMax = 1024;           // ties at the threshold key the gathered path resolves
constexpr int kSegBytes = 8192;         // dZ segment in LDS (two of them)
template <int IN, bool SAMPLE>
__global__ void __launch_bounds__(256)
kl_top_kernel(const void *__restrict__ Zs, const void *__restrict__ Zt, int64_t V, int k, double inv_T,
              void *__restrict__ dZs, double *__restrict__ row_loss, uint32_t *flag, int r) {
    using elem_t = typename std::conditional<IN == kBF16, uint16_t, uint32_t>::type;  // a logit's bits
    constexpr int kEsz = sizeof(elem_t);
    constexpr int E = 16 / kEsz;  // logits per 16 bytes
    // LDS by hand, because rows per CU hide each other's latency (bf16: 34 KB, four rows): the lists' indices and
    // student logits (later gradients) first, then a region that holds the histograms, the lists' teacher
    // logits and the ties, and after them the two dZ segments. The passes below put their arrays over the lists, or
    // without the sample into 10 KB of their own (the registers then let four rows onto a CU in fp32 too).
    constexpr int kIdxOff = 0, kBOff = kCand * 4, kRegion = kBOff + kCand * kEsz;
    constexpr int kAOff = kRegion + 3 * 256 * 4, kTieOff = kAOff + kCand * kEsz;
    constexpr int kLds = SAMPLE ? std::max(kTieOff + kTieMax * 4, kRegion + 2 * kSegBytes) : 16;
    __shared__ __attribute__((aligned(16))) char lds[kLds];
    uint32_t *const cand_idx = reinterpret_cast<uint32_t *>(lds + kIdxOff);
    elem_t *const cand_b = reinterpret_cast<elem_t *>(lds + kBOff);
    uint32_t(*const hist)[256] = reinterpret_cast<uint32_t(*)[256]>(lds + kRegion);
    elem_t *const cand_a = reinterpret_cast<elem_t *>(lds + kAOff);
    uint32_t *const tie_idx = reinterpret_cast<uint32_t *>(lds + kTieOff);
    char *const stage = lds + kRegion;
    __shared__ double own_s[2][256], own_d[256];
    __shared__ float own_m[2][256];
    __shared__ uint32_t own_scan[256], own_hist[256];
    double(*const red_s)[256] = SAMPLE ? reinterpret_cast<double(*)[256]>(lds) : own_s;
    double *const red_d = SAMPLE ? reinterpret_cast<double *>(lds + 4096) : own_d;
    float(*const red_m)[256] = SAMPLE ? reinterpret_cast<float(*)[256]>(lds + 6144) : own_m;
    uint32_t *const scan_buf = SAMPLE ? reinterpret_cast<uint32_t *>(lds + 8192) : own_scan;
    uint32_t *const hist0 = SAMPLE ? hist[0] : own_hist;
    static_assert(8192 + 1024 <= kRegion, "the passes' arrays lie below the histograms");
    __shared__ uint32_t sel_digit, sel_above;
    __shared__ uint32_t wave_cnt[4], wave_n[4], tie_cnt;
    __shared__ float wave_m[2][4];
    __shared__ double wave_s[3][4];
    __shared__ int64_t cut_sh;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t row = blockIdx.x;
    const char *zs = reinterpret_cast<const char *>(Zs) + row * V * kEsz;
    const char *zt = reinterpret_cast<const char *>(Zt) + row * V * kEsz;
    char *dz = reinterpret_cast<char *>(dZs) + row * V * kEsz;
    const bool all = (int64_t)k >= V;
    bool bad = false;
    constexpr int kPasses = IN == kBF16 ? 2 : 4;  // 8-bit digits of a key (bf16 keys have zero low 16 bits)

    // online softmax statistics of one selected pair of logits (sums of exp(z - max) in double: the
    // loss needs their logs to ~1e-12)
    auto online_stats = [](float a, float b, float &mt, double &st, float &ms, double &ss) {
        if (a > mt) {
            st = st * exp((double)mt - (double)a) + 1.0;
            mt = a;
        } else {
            st += exp((double)a - (double)mt);
        }
        if (b > ms) {
            ss = ss * exp((double)ms - (double)b) + 1.0;
            ms = b;
        } else {
            ss += exp((double)b - (double)ms);
        }
    };
    // log-sum-exp of each row over the selected set from every thread's statistics (a fixed tree):
    // lt_d for the teacher and dl = lt_d - ls_d, in double
    auto row_lse = [&](float mt, double st, float ms, double ss, double &lt_d, double &dl) {
        red_m[0][t] = mt, red_s[0][t] = st, red_m[1][t] = ms, red_s[1][t] = ss;
        __syncthreads();
        for (int off = 128; off > 0; off >>= 1) {
            if (t < off) {
                for (int q = 0; q < 2; q++) {
                    const float m1 = red_m[q][t], m2 = red_m[q][t + off];
                    const double s1 = red_s[q][t], s2 = red_s[q][t + off];
                    const float m = fmaxf(m1, m2);
                    const double s = (m1 == -INFINITY ? 0.0 : s1 * exp((double)m1 - (double)m)) +
                                     (m2 == -INFINITY ? 0.0 : s2 * exp((double)m2 - (double)m));
                    red_m[q][t] = m;
                    red_s[q][t] = s;
                }
            }
            __syncthreads();
        }
        lt_d = (double)red_m[0][0] + log(red_s[0][0]);
        dl = lt_d - ((double)red_m[1][0] + log(red_s[1][0]));
        __syncthreads();
    };
    // KL term of one selected element, -p_t d, added to kl; returns dZ_s = (p_s - p_t) / T. With
    // d = log p_s - log p_t, p_s - p_t = p_t expm1(d) keeps its relative accuracy where the two
    // probabilities nearly cancel.
    auto kl_term = [&](float a, float b, double lt_d, double dl, double &kl) {
        const double pt = exp((double)a - lt_d);
        const double d = ((double)b - (double)a) + dl;
        kl -= pt * d;
        return (float)(pt * expm1(d) * inv_T);
    };
    // the row's KL from every thread's part (a fixed tree)
    auto row_total = [&](double kl) {
        red_d[t] = kl;
        __syncthreads();
        for (int off = 128; off > 0; off >>= 1) {
            if (t < off) red_d[t] += red_d[t + off];
            __syncthreads();
        }
        if (t == 0) row_loss[row] = red_d[0];
    };

    bool done = false;
    if constexpr (SAMPLE) {
        // One histogram pass of a select: counts of add()'s bins (0..255) in one of three histograms, then
        // every wave finds by itself the bin that holds the rem-th largest element (rem becomes its rank within
        // the bin). Histogram p % 3 is cleared again after the next pass's barrier, when every wave has read it,
        // and two passes before its next use.
        int pass = 0;
        for (int i = t; i < 3 * 256; i += 256) hist[i >> 8][i & 255] = 0u;
        auto find_bin = [&](auto add, uint32_t &rem) {
            uint32_t *const h = hist[pass % 3];
            add([&](uint32_t bin) { atomicAdd(&h[bin], 1u); });
            __syncthreads();
            hist[(pass + 2) % 3][t] = 0u;
            pass++;
            const uint4 c = *reinterpret_cast<const uint4 *>(&h[252 - 4 * lane]);  // bins 255 - 4 lane downwards
            const uint32_t sum = c.x + c.y + c.z + c.w;
            uint32_t incl = sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t up = __shfl_up(incl, off, 64);
                incl += lane >= off ? up : 0u;
            }
            uint32_t above = incl - sum, bin = 255u - 4u * (uint32_t)lane;
            const bool here = above < rem && rem <= incl;
            if (rem > above + c.w) {
                above += c.w, bin--;
                if (rem > above + c.z) {
                    above += c.z, bin--;
                    if (rem > above + c.y) above += c.y, bin--;
                }
            }
            const int src = __ffsll((unsigned long long)__ballot(here)) - 1;
            rem -= (uint32_t)__shfl((int)above, src, 64);
            return (uint32_t)__shfl((int)bin, src, 64);
        };
        // the rem-th largest key of the keys that for_keys hands out; `fixed` bits from the top are `pre`
        auto radix = [&](auto for_keys, uint32_t pre, int fixed, uint32_t &rem) {
            uint32_t msk = fixed ? ~0u << (32 - fixed) : 0u;
            for (int shift = 24 - fixed; shift >= 32 - 8 * kPasses; shift -= 8) {
                const uint32_t d = find_bin([&](auto count) {
                    for_keys([&](uint32_t key) {
                        if ((key & msk) == pre) count((key >> shift) & 255u);
                    });
                }, rem);
                pre |= d << shift;
                msk |= 0xFFu << shift;
            }
            return pre;
        };
        // ---- the sample: 8 adjacent keys from each of kSample / 8 evenly spaced elements (rows of at
        // least kSampleMinV keep the runs apart), its r-th largest the gather bound ----
        uint32_t sk[kSample / 256];
#pragma unroll
        for (int u = 0; u < kSample / 256; u++)
            sk[u] = logit_key<IN>(load_logit<IN>(zt, (int64_t)((t + 256 * u) >> 3) * V / (kSample / 8) + ((t + 256 * u) & 7)));
        __syncthreads();  // the histograms are clear
        uint32_t rem_s = (uint32_t)r;
        const uint32_t lower = radix([&](auto fn) {
#pragma unroll
            for (int u = 0; u < kSample / 256; u++) fn(sk[u]);
        }, 0u, 0, rem_s);
        // the bound as a value: an element whose key is at or above `lower` is not below it. (Not "at or above it": a
        // NaN's key is above all others, or below them with its sign set, and the select below is by key.)
        const float lowf = __uint_as_float(((lower & 0x80000000u) ? lower ^ 0x80000000u : ~lower) &
                                           (IN == kBF16 ? 0xFFFF0000u : 0xFFFFFFFFu));
        // ---- one pass over both rows: the elements at or above the bound into this wave's list ----
        // 16-byte pieces start where the teacher row's address is a multiple of 16: `head` elements before the
        // first, npiece whole ones, the rest after the last. The student row takes 16-byte loads if its
        // address has the same remainder, as it has for whole tensors.
        const uint32_t mis = (uint32_t)(reinterpret_cast<uintptr_t>(zt) & 15u) / kEsz;
        const int64_t head = mis ? E - mis : 0, npiece = (V - head) / E;
        const bool same_s = ((reinterpret_cast<uintptr_t>(zs) ^ reinterpret_cast<uintptr_t>(zt)) & 15u) == 0;
        const bool same_d = ((reinterpret_cast<uintptr_t>(dz) ^ reinterpret_cast<uintptr_t>(zt)) & 15u) == 0;
        const elem_t *const zt_p = reinterpret_cast<const elem_t *>(zt) + head;
        const elem_t *const zs_p = reinterpret_cast<const elem_t *>(zs) + head;
        const uint64_t below = (1ull << lane) - 1ull;
        uint32_t wn = 0u;  // elements this wave has met at or above the bound (wave-uniform)
        const uint32_t seg = (uint32_t)wave * kPerWave;
        auto value = [](uint32_t word, int half) {  // logit `half` of a word (fp32: the word)
            return __uint_as_float(IN == kBF16 ? (half ? word & 0xFFFF0000u : word << 16) : word);
        };
        auto put = [&](uint32_t slot, int64_t i, uint32_t a, uint32_t b) {
            if (slot < (uint32_t)kPerWave) {
                cand_a[seg + slot] = (elem_t)a;
                cand_b[seg + slot] = (elem_t)b;
                cand_idx[seg + slot] = (uint32_t)i;
            }
        };
        // one element per lane (the row's ends), lanes in index order
        auto gather_one = [&](int64_t i, bool valid) {
            elem_t a = 0, b = 0;
            if (valid) a = reinterpret_cast<const elem_t *>(zt)[i], b = reinterpret_cast<const elem_t *>(zs)[i];
            const float av = value(a, 0), bv = value(b, 0);
            bad = bad || (valid && (!(__builtin_fabsf(av) < INFINITY) || !(__builtin_fabsf(bv) < INFINITY)));
            const bool cand = valid && !(av < lowf);
            const uint64_t m = __ballot(cand);
            if (cand) put(wn + (uint32_t)__popcll(m & below), i, a, b);
            wn += (uint32_t)__popcll(m);
        };
        auto gather = [&](int64_t p, bool valid, const uint4 &wa, const uint4 &wb) {
            const uint32_t a[4] = {wa.x, wa.y, wa.z, wa.w}, b[4] = {wb.x, wb.y, wb.z, wb.w};
            uint32_t mask = 0u, inf = 0u;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                if constexpr (IN == kBF16) {
                    // bit 15 of a half: its exponent is all ones (no carry crosses the halves)
                    inf |= ((a[q] & 0x7FFF7FFFu) + 0x00800080u) | ((b[q] & 0x7FFF7FFFu) + 0x00800080u);
                    mask |= (value(a[q], 0) < lowf ? 0u : 1u) << (2 * q);
                    mask |= (value(a[q], 1) < lowf ? 0u : 1u) << (2 * q + 1);
                } else {
                    inf |= ((a[q] & 0x7FFFFFFFu) + 0x00800000u) | ((b[q] & 0x7FFFFFFFu) + 0x00800000u);
                    mask |= (value(a[q], 0) < lowf ? 0u : 1u) << q;
                }
            }
            bad = bad || (valid && (inf & 0x80008000u & (IN == kBF16 ? ~0u : 0x80000000u)));
            mask = valid ? mask : 0u;
            if (__ballot(mask != 0u) == 0ull) return;
            // slots in index order: the set bits of the lanes below, from one ballot per bit of the count
            const uint32_t n = (uint32_t)__popc(mask);
            uint32_t slot = wn;
#pragma unroll
            for (int bit = 0; (1 << bit) <= E; bit++) {
                const uint64_t m = __ballot((n >> bit) & 1u);
                slot += (uint32_t)__popcll(m & below) << bit;
                wn += (uint32_t)__popcll(m) << bit;
            }
            const int64_t i0 = head + p * E;
            while (mask) {
                const int e = __builtin_ctz(mask);
                mask &= mask - 1u;
                const int q = IN == kBF16 ? e >> 1 : e, sh = IN == kBF16 ? (e & 1) * 16 : 0;
                const uint32_t va = q < 2 ? (q ? a[1] : a[0]) : (q == 2 ? a[2] : a[3]);
                const uint32_t vb = q < 2 ? (q ? b[1] : b[0]) : (q == 2 ? b[2] : b[3]);
                put(slot++, i0 + e, va >> sh, vb >> sh);
            }
        };
        // both rows are read once here: the non-temporal policy (8,192 x 151,936: 5% faster)
        auto stream = [](const elem_t *p) {
            typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
            return make_uint4(v.x, v.y, v.z, v.w);
        };
        auto load_b = [&](int64_t p) {
            if (same_s) return stream(zs_p + p * E);
            uint32_t w[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                if constexpr (IN == kBF16) w[q] = (uint32_t)zs_p[p * E + 2 * q] | (uint32_t)zs_p[p * E + 2 * q + 1] << 16;
                else w[q] = zs_p[p * E + q];
            }
            return make_uint4(w[0], w[1], w[2], w[3]);
        };
        if (wave == 0 && head) gather_one(lane, lane < head);
        // wave w takes 64-piece blocks w, w + 4, ..; kU of them are loaded before any is used. A piece past the
        // last is clamped to it (npiece >= 1 here), so every load is unconditional, and left out.
        constexpr int kU = 4;
        for (int64_t blk = wave; blk * 64 < npiece; blk += 4 * kU) {
            uint4 wa[kU], wb[kU];
#pragma unroll
            for (int u = 0; u < kU; u++) {
                const int64_t p = std::min<int64_t>((blk + 4 * u) * 64 + lane, npiece - 1);
                wa[u] = stream(zt_p + p * E);
                wb[u] = load_b(p);
            }
#pragma unroll
            for (int u = 0; u < kU; u++) {
                const int64_t p = (blk + 4 * u) * 64 + lane;
                gather(p, p < npiece, wa[u], wb[u]);
            }
        }
        if (wave == 3) gather_one(head + npiece * E + lane, lane < V - head - npiece * E);  // fewer than E
        if (lane == 0) wave_n[wave] = wn;
        __syncthreads();
        const uint32_t nw[4] = {wave_n[0], wave_n[1], wave_n[2], wave_n[3]};
        const bool fits = nw[0] <= (uint32_t)kPerWave && nw[1] <= (uint32_t)kPerWave &&
                          nw[2] <= (uint32_t)kPerWave && nw[3] <= (uint32_t)kPerWave;
        if (fits && (uint64_t)nw[0] + nw[1] + nw[2] + nw[3] >= (uint64_t)k) {
            // every element at or above the k-th largest key is in the lists
            const uint32_t o1 = nw[0], o2 = o1 + nw[1], o3 = o2 + nw[2], ntot = o3 + nw[3];
            auto for_cands = [&](auto fn) {
                for (uint32_t j = (uint32_t)t; j < ntot; j += 256u) {
                    const uint32_t w = (j >= o1) + (j >= o2) + (j >= o3);
                    fn(w * kPerWave + j - (w == 0 ? 0u : w == 1 ? o1 : w == 2 ? o2 : o3));
                }
            };
            auto a_at = [&](uint32_t s) { return value(cand_a[s], 0); };
            auto b_at = [&](uint32_t s) { return value(cand_b[s], 0); };
            auto key_at = [&](uint32_t s) { return logit_key<IN>(a_at(s)); };
            auto for_keys = [&](auto fn) { for_cands([&](uint32_t s) { fn(key_at(s)); }); };
            // The gathered keys start at `lower` and the k-th lies close to it: a first pass over the keys' high
            // halves relative to the bound's resolves it unless it is 255 or more above
            uint32_t rem = (uint32_t)k;
            const uint32_t low16 = lower >> 16;
            const uint32_t d = find_bin([&](auto count) {
                for_keys([&](uint32_t key) { count(std::min((key >> 16) - low16, 255u)); });
            }, rem);
            uint32_t thr;
            if (d < 255u) {
                thr = radix(for_keys, (low16 + d) << 16, 16, rem);
            } else {
                rem = (uint32_t)k;
                thr = radix(for_keys, 0u, 0, rem);
            }
            // ties at the threshold key: the first rem of them in index order are selected
            if (t == 0) tie_cnt = 0u;
            __syncthreads();
            uint32_t my_ties = 0u;
            for_cands([&](uint32_t s) { my_ties += key_at(s) == thr ? 1u : 0u; });
            if (my_ties) atomicAdd(&tie_cnt, my_ties);  // an integer count: the order of the additions is immaterial
            __syncthreads();
            if (tie_cnt <= (uint32_t)kTieMax) {
                int64_t cut = V;
                if (rem < tie_cnt) {
                    // The rem-th smallest index among the ties. A wave's list is in index order, so
                    // each wave compacts the ties of its own list, in order, into its region of
                    // tie_idx; a tie's rank among all ties is its place in its region plus the ties
                    // of smaller index in the other three regions (binary searches).
                    const uint32_t nown = nw[wave];
                    uint32_t mine_n = 0u;
                    for (uint32_t j0 = 0; j0 < nown; j0 += 64u) {
                        const uint32_t j = j0 + (uint32_t)lane;
                        mine_n += (uint32_t)__popcll(__ballot(j < nown && key_at(seg + j) == thr));
                    }
                    if (lane == 0) wave_cnt[wave] = mine_n;
                    __syncthreads();
                    const uint32_t off[5] = {0u, wave_cnt[0], wave_cnt[0] + wave_cnt[1],
                                             wave_cnt[0] + wave_cnt[1] + wave_cnt[2],
                                             wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3]};
                    uint32_t pos = off[wave];
                    for (uint32_t j0 = 0; j0 < nown; j0 += 64u) {
                        const uint32_t j = j0 + (uint32_t)lane;
                        const bool tie = j < nown && key_at(seg + j) == thr;
                        const uint64_t m = __ballot(tie);
                        if (tie) tie_idx[pos + (uint32_t)__popcll(m & below)] = cand_idx[seg + j];
                        pos += (uint32_t)__popcll(m);
                    }
                    __syncthreads();
                    for (uint32_t e = (uint32_t)t; e < off[4]; e += 256u) {
                        const int we = (e >= off[1]) + (e >= off[2]) + (e >= off[3]);
                        const uint32_t mine = tie_idx[e];
                        uint32_t rank = e - off[we];
                        for (int w = 0; w < 4; w++) {
                            if (w == we) continue;
                            uint32_t lo = off[w], hi = off[w + 1];
                            while (lo < hi) {
                                const uint32_t mid = (lo + hi) >> 1;
                                if (tie_idx[mid] < mine) lo = mid + 1u;
                                else hi = mid;
                            }
                            rank += lo - off[w];
                        }
                        if (rank + 1u == rem) cut_sh = (int64_t)mine + 1;
                    }
                    __syncthreads();
                    cut = cut_sh;
                }
                auto chosen = [&](uint32_t s) {
                    const uint32_t key = key_at(s);
                    return key > thr || (key == thr && (int64_t)cand_idx[s] < cut);
                };
                // maxima, then sums of exp(z - max) in double, of both rows over the selected set: per thread,
                // per wave by exchanges, then over the four waves in order
                float mt = -INFINITY, ms = -INFINITY;
                for_cands([&](uint32_t s) {
                    if (chosen(s)) mt = fmaxf(mt, a_at(s)), ms = fmaxf(ms, b_at(s));
                });
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    mt = fmaxf(mt, __shfl_xor(mt, off, 64));
                    ms = fmaxf(ms, __shfl_xor(ms, off, 64));
                }
                if (lane == 0) wave_m[0][wave] = mt, wave_m[1][wave] = ms;
                __syncthreads();
                mt = fmaxf(fmaxf(wave_m[0][0], wave_m[0][1]), fmaxf(wave_m[0][2], wave_m[0][3]));
                ms = fmaxf(fmaxf(wave_m[1][0], wave_m[1][1]), fmaxf(wave_m[1][2], wave_m[1][3]));
                double st = 0.0, ss = 0.0;
                for_cands([&](uint32_t s) {
                    if (chosen(s)) st += exp((double)a_at(s) - (double)mt), ss += exp((double)b_at(s) - (double)ms);
                });
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) st += __shfl_xor(st, off, 64), ss += __shfl_xor(ss, off, 64);
                if (lane == 0) wave_s[0][wave] = st, wave_s[1][wave] = ss;
                __syncthreads();
                st = ((wave_s[0][0] + wave_s[0][1]) + wave_s[0][2]) + wave_s[0][3];
                ss = ((wave_s[1][0] + wave_s[1][1]) + wave_s[1][2]) + wave_s[1][3];
                const double lt_d = (double)mt + log(st), dl = lt_d - ((double)ms + log(ss));
                double kl = 0.0;
                for_cands([&](uint32_t s) {
                    const float g = chosen(s) ? kl_term(a_at(s), b_at(s), lt_d, dl, kl) : 0.0f;
                    cand_b[s] = (elem_t)(IN == kBF16 ? f32_to_bf16_bits(g) : __float_as_uint(g));
                });
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) kl += __shfl_xor(kl, off, 64);
                if (lane == 0) wave_s[2][wave] = kl;
                __syncthreads();
                if (t == 0) row_loss[row] = ((wave_s[2][0] + wave_s[2][1]) + wave_s[2][2]) + wave_s[2][3];
                // every wave is done with the teacher's logits: both segments zero
                for (int i = t; i < 2 * kSegBytes / 16; i += 256) reinterpret_cast<uint4 *>(stage)[i] = make_uint4(0u, 0u, 0u, 0u);
                __syncthreads();
                // ---- dZ: position p of the segments is element p - mis, so that 16-byte stores are aligned when
                // dZ's address has the teacher's remainder (otherwise element by element). One barrier per
                // segment: a buffer is cleared as it is read out, before the barrier that precedes the
                // scatter into it. ----
                constexpr int kSeg = kSegBytes / kEsz;
                uint32_t j = 0u;  // this wave's next gathered element
                elem_t *const dz_e = reinterpret_cast<elem_t *>(dz);
                for (int64_t s0 = 0; s0 < V + mis; s0 += kSeg) {
                    char *const buf = stage + ((s0 / kSeg) & 1) * kSegBytes;
                    for (;;) {
                        const bool have = j + (uint32_t)lane < nw[wave];
                        const int64_t p = have ? (int64_t)cand_idx[seg + j + lane] + mis : 0;
                        const bool in = have && p < s0 + kSeg;
                        if (in) reinterpret_cast<elem_t *>(buf)[p - s0] = cand_b[seg + j + lane];
                        const uint32_t n = (uint32_t)__popcll(__ballot(in));
                        j += n;
                        if (n < 64u) break;
                    }
                    __syncthreads();
#pragma unroll
                    for (int u = 0; u < kSegBytes / 16 / 256; u++) {
                        const int c = t + 256 * u;
                        const int64_t i0 = s0 + (int64_t)c * E - mis;  // first element of the piece
                        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
                        u32x4 *const src = reinterpret_cast<u32x4 *>(buf) + c;
                        const u32x4 v = *src;
                        *src = u32x4{0u, 0u, 0u, 0u};
                        if (same_d && i0 >= 0 && i0 + E <= V) {
                            __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dz_e + i0));
                        } else {
#pragma unroll
                            for (int e = 0; e < E; e++) {
                                const uint32_t w = v[IN == kBF16 ? e / 2 : e];
                                if (i0 + e >= 0 && i0 + e < V) dz_e[i0 + e] = (elem_t)(IN == kBF16 ? w >> (16 * (e & 1)) : w);
                            }
                        }
                    }
                }
                done = true;
            }
        }
        // otherwise the passes below decide and write dZ
        __syncthreads();
    }

    if (!done) {
        // ---- threshold key: the k-th largest teacher key ----
        uint32_t prefix = 0u, pmask = 0u, remaining = (uint32_t)k;
        if (!all) {
            for (int p = 0; p < kPasses; p++) {
                const int shift = 24 - 8 * p;
                hist0[t] = 0u;
                __syncthreads();
                for (int64_t base = 0; base < V; base += 256 * kTrips) {
                    float v[kTrips];
                    load_trips<IN>(zt, base, t, V, v);
    #pragma unroll
                    for (int u = 0; u < kTrips; u++) {
                        const uint32_t key = logit_key<IN>(v[u]);
                        if (base + t + 256 * u < V && (key & pmask) == prefix) atomicAdd(&hist0[(key >> shift) & 255u], 1u);
                    }
                }
                __syncthreads();
                // bins in descending digit order: thread j holds digit 255 - j
                const uint32_t h = hist0[255 - t];
                const uint32_t incl = block_scan(h, scan_buf);
                if (incl - h < remaining && remaining <= incl) {
                    sel_digit = 255u - (uint32_t)t;
                    sel_above = incl - h;
                }
                __syncthreads();
                remaining -= sel_above;
                prefix |= sel_digit << shift;
                pmask |= 0xFFu << shift;
                __syncthreads();
            }
        }
        const uint32_t thr = prefix;  // with `all`, every element is selected
        // ---- ties at the threshold: admit the first `remaining` in index order ----
        int64_t cut = V;  // selected ties are those with index < cut
        if (!all) {
            uint32_t seen = 0u;
            bool found = false;
            for (int64_t base0 = 0; base0 < V && !found; base0 += 256 * kTrips) {
                float v[kTrips];
                load_trips<IN>(zt, base0, t, V, v);
                for (int u = 0; u < kTrips; u++) {
                    const int64_t base = base0 + 256 * u;
                    if (base >= V) break;
                    const int64_t i = base + t;
                    const bool tie = i < V && logit_key<IN>(v[u]) == thr;
                    const uint64_t m = __ballot(tie);
                    if (lane == 0) wave_cnt[wave] = (uint32_t)__popcll(m);
                    __syncthreads();
                    uint32_t before = seen;
                    for (int w = 0; w < wave; w++) before += wave_cnt[w];
                    const uint32_t total = wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3];
                    const uint32_t rank = before + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                    __syncthreads();
                    if (seen + total >= remaining) {
                        // the remaining-th tie is in this trip: its index + 1 is the cut
                        if (tie && rank + 1u == remaining) red_d[0] = (double)(i + 1);
                        __syncthreads();
                        cut = (int64_t)red_d[0];
                        found = true;
                        break;
                    }
                    seen += total;
                }
            }
        }
        auto selected = [&](int64_t i, uint32_t key) { return all || key > thr || (key == thr && i < cut); };

        // ---- softmax statistics over the selected set (online per thread) ----
        float mt = -INFINITY, ms = -INFINITY;
        double st = 0.0, ss = 0.0;  // sums of exp(z - max) in double: the loss needs their logs to ~1e-12
        for (int64_t base = 0; base < V; base += 256 * kTrips) {
            float va[kTrips], vb[kTrips];
            load_trips<IN>(zt, base, t, V, va);
            load_trips<IN>(zs, base, t, V, vb);
            for (int u = 0; u < kTrips; u++) {
                const int64_t i = base + t + 256 * u;
                if (i >= V) break;
                const float a = va[u], b = vb[u];
                bad = bad || !(__builtin_fabsf(a) < INFINITY) || !(__builtin_fabsf(b) < INFINITY);
                if (!selected(i, logit_key<IN>(a))) continue;
                online_stats(a, b, mt, st, ms, ss);
            }
        }
        double lt_d, dl;
        row_lse(mt, st, ms, ss, lt_d, dl);

        // ---- KL(p_t || p_s) over the set and dZ_s = (p_s - p_t) / T ----
        double kl = 0.0;
        for (int64_t base = 0; base < V; base += 256 * kTrips) {
            float va[kTrips], vb[kTrips];
            load_trips<IN>(zt, base, t, V, va);
            load_trips<IN>(zs, base, t, V, vb);
            // a whole chunk's stores are unconditional: the compiler then counts the memory operations in flight exactly
            const bool whole = base + 256 * kTrips <= V;
            for (int u = 0; u < kTrips; u++) {
                const int64_t i = base + t + 256 * u;
                if (!whole && i >= V) break;
                const float a = va[u], b = vb[u];
                float g = 0.0f;
                if (selected(i, logit_key<IN>(a))) g = kl_term(a, b, lt_d, dl, kl);
                store_logit<IN>(dz, i, g);
            }
        }
        row_total(kl);
    }
    if (bad) raise_domain_flag(flag);
}

// loss = (sum of row losses) / T, in a fixed order
__global__ void __launch_bounds__(256) row_mean_kernel(const double *__restrict__ row_loss, int64_t T,
                                                        double *__restrict__ loss) {
    __shared__ double red[256];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < T; i += 256) acc += row_loss[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = red[0] / (double)T;
}

// zero fill of a 16-byte-aligned buffer (whole 16-byte words, then the tail bytes)
__global__ void __launch_bounds__(256) zero_fill_kernel(char *__restrict__ p, size_t bytes) {
    const size_t words = bytes / 16;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256)
        reinterpret_cast<uint4 *>(p)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (blockIdx.x == 0 && threadIdx.x < bytes % 16) p[words * 16 + threadIdx.x] = 0;
}

}  // namespace

hipError_t launch_zero_fill(void *p, size_t bytes, hipStream_t st) {
    const size_t words = bytes / 16;
    const unsigned grid = (unsigned)std::max<size_t>(1, std::min<size_t>((words + 255) / 256, kStreamGridCap));
    zero_fill_kernel<<<grid, 256, 0, st>>>(static_cast<char *>(p), bytes);
    return hipGetLastError();
}

hipError_t launch_transpose(int dt, const void *in, int64_t R, int64_t C, void *out, hipStream_t st) {
    const dim3 grid((unsigned)((C + 63) / 64), (unsigned)((R + 63) / 64));
    if (dt == kBF16)
        transpose_kernel<uint16_t><<<grid, 256, 0, st>>>(static_cast<const uint16_t *>(in), R, C,
                                                         static_cast<uint16_t *>(out));
    else
        transpose_kernel<float><<<grid, 256, 0, st>>>(static_cast<const float *>(in), R, C, static_cast<float *>(out));
    return hipGetLastError();
}

// Rank r of the sample's key that bounds the k-th largest logit from below, or 0 where the rows take the passes: the
// sample's expected count of the k largest with three standard deviations, if the lists hold what lies above it.
static int kl_sample_rank(int64_t V, int k) {
    const double kexp = (double)k * kSample / (double)V;
    const double r = std::ceil(kexp) + std::ceil(3.0 * std::sqrt(kexp)) + 2.0;
    return (int64_t)k < V && V >= kSampleMinV && r <= kSample / 4 && r * (double)V / kSample <= 0.65 * kCand ? (int)r : 0;
}

hipError_t launch_kl_top(int dt, const void *Zs, const void *Zt, int64_t T, int64_t V, int k, void *dZs,
                         double *row_loss, double *loss, uint32_t *flag, hipStream_t st) {
    const double inv_T = 1.0 / (double)T;
    const int r = kl_sample_rank(V, k);
#define KL(IN, S) kl_top_kernel<IN, S><<<(unsigned)T, 256, 0, st>>>(Zs, Zt, V, k, inv_T, dZs, row_loss, flag, r)
    if (dt == kBF16) { if (r) KL(kBF16, true); else KL(kBF16, false); }
    else { if (r) KL(kF32, true); else KL(kF32, false); }
#undef KL
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    row_mean_kernel<<<1, 256, 0, st>>>(row_loss, T, loss);
    return hipGetLastError();
}

}  // namespace focus
