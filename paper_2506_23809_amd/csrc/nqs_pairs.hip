// All pairs of samples on the matrix cores: the local energy summed over the
// pairs of S directly (Eq. 5 with the kets taken from S, the loop structure
// of Alg. 3), for batches small enough, or gathered enough, that comparing
// every pair costs less than grouping the samples or enumerating their
// flips.
//
// Every group of the table flips at most max_flip qubits, so a connected
// pair is within that Hamming distance.  With the bits of a sample as +-1,
// x . y = n_qubits - 2 distance(x, y): a tile of 32 x 32 pairs is one FP4
// matrix product per 64 qubits (products of +-1 summed in FP32, exact), the
// threshold sits in its C operand, and a pair is near where the result is
// positive.  The order of the qubits does not matter to the product, so the
// operands are made from the bit strings by a shift and a mask per eight
// qubits, where they are loaded.  Near pairs (the group index decides whether
// X = x ^ y is a flip of the table) are queued per wave and evaluated 64 at a
// time, the few groups with many terms (single excitations) in a queue of
// their own, so that a wave's lanes run alike.
//
// Determinism: each sample's contributions are added as double-doubles (one
// rounding of a sum whose error is below 2^-100 of its largest partial), so
// the bits of the result do not depend on the order of the additions.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/nqs.h"
#include "nqs_dev_common.hpp"
#include "nqs_device.hpp"

namespace nqs {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kPairsThreads = 512;
constexpr int kPairsWaves = kPairsThreads / 64;
constexpr int kPairsQueue = 128;  // entries per queue and wave (64 are taken at a time)
// Groups of more terms than this go through the queue of long groups (the
// double excitations of a molecule have 4 or 6 terms in one record, its
// single excitations 2 n_qubits - 2 and an occupation row).
constexpr uint32_t kShortTerms = 12;
// A queue entry is a sample's index above the six bits of its row.
static_assert(kJoinMaxSamples <= int64_t(1) << 26, "a sample's index fits a queue entry");

// A sample: its bits, log-amplitude and phase.
struct alignas(16) PairRec {
    uint64_t w0, w1;
    double la, ph;
};

// Clears the counters and control words of the launch, makes the sample
// checks of the hash build, and lays out the samples for the pair kernel:
// one 32-byte record each and the bits by tiles (3.6 us for 4,096 samples).
__global__ __launch_bounds__(256) void pairs_prep_kernel(
    DevTable tab, DevScratch sc, const uint64_t *__restrict__ samples,
    const int64_t *__restrict__ weights, const double *__restrict__ log_amp,
    const double *__restrict__ phase, int64_t n, uint32_t jparts, uint32_t jhit_words) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < static_cast<uint32_t>(kCounters * kCounterSlots)) sc.counters[s] = 0;
    if (s == 0) *sc.mixed = 0;
    if (sc.jctl && s < static_cast<uint32_t>(kJoinCtl)) sc.jctl[s] = 0;
    if (s < jparts) sc.jcnt[s] = 0u;
    if (s < jhit_words) sc.jhit[s] = 0u;
    const int nq = tab.n_qubits;
    // the bits of each tile of 32 samples, as the pair kernel's lanes read
    // them: 64 qubits kb of sample xl at [tile][kb][half][xl]
    if (s < (n + 31) / 32 * 32) {
        const int words = nq <= 63 ? 1 : 2;
        uint32_t *key = reinterpret_cast<uint32_t *>(sc.pkey) + (s >> 5) * words * 64 + (s & 31u);
        for (int kb = 0; kb < words; ++kb) {
            const uint64_t w = s < n ? samples[2 * static_cast<int64_t>(s) + kb] : 0ull;
            key[64 * kb] = static_cast<uint32_t>(w);
            key[64 * kb + 32] = static_cast<uint32_t>(w >> 32);
        }
    }
    if (s < n) {
        const int64_t i = s;
        const uint64_t w0 = samples[2 * i], w1 = samples[2 * i + 1];
        const bool bad = nq >= 64 ? ((w1 >> (nq - 64)) != 0) : ((w0 >> nq) != 0 || w1 != 0);
        if (bad || (weights && weights[i] < 0)) latch(sc.err, NQS_E_RANGE);
        reinterpret_cast<PairRec *>(sc.prec)[i] = PairRec{w0, w1, log_amp[i], phase[i]};
    }
}

template <int W>
__device__ __forceinline__ Key<W> rec_key(const PairRec &r) {
    Key<W> k;
    k.w[0] = r.w0;
    if constexpr (W == 2) k.w[W - 1] = r.w1;
    return k;
}

// Shared state of one wave.
struct PairsWave {
    uint32_t q[kPairsQueue];       // near pairs: x of the tile | y << 6
    uint2 lq[kPairsQueue];         // pairs whose group is long: the same, group
    double con[2][64];             // contributions of a batch (re, im)
    unsigned long long own[64];    // which of them belong to each x
};

// One block per 32 H samples x (blockIdx.x) and share of the samples y
// (blockIdx.y); its waves take the tiles of y in turn.
//
// Bound: per 32 x 32 pairs one (W = 1) or two FP4 MFMAs of 32 cycles, about
// ten VALU instructions where no pair is near, eight per 64 qubits to make
// the operand and 256 bytes W / H of bits from the caches (as finished
// operands 1 KB, no VALU instructions and no faster: 8,192 samples without a near
// pair 12.0 and 11.5 us at 40 qubits, 11.7 and 12.6 at 100); per near pair the
// gathers of its record, group and values and the FP64 amplitude ratio.
// Gathered samples are bound by VALU issue first and those gathers second:
// 37,843 at 40 qubits (17 M hits) 544 us, of which the VALU instructions take
// 350, the matrix cores 18, with 75 M requests to L2 (99% hits) and waves
// waiting 46% of their time; 20,001 at 100 qubits (7.7 M hits) 356 us, VALU
// 185, waiting 60%.
// Registers: 128 (four waves a SIMD); at 134 the 100-qubit form took 627 us
// instead of 508 for 20,001 gathered samples, at 96 it spilled (600).
template <int W, int H, bool DUMP, int P, bool SCV>
__global__ __launch_bounds__(kPairsThreads, 4) void pairs_kernel(
    DevTable tab, DevScratch sc, int64_t n, int32_t *__restrict__ hit_idx,
    uint32_t *__restrict__ sign_bits, int64_t sign_words) {
    if (!pairs_chosen(sc)) return;
    constexpr int R = 32 * H;  // samples x of the block
    __shared__ PairRec xs[R];
    __shared__ PairsWave waves[kPairsWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t x0 = static_cast<int64_t>(blockIdx.x) * R;
    const PairRec *__restrict__ rec = reinterpret_cast<const PairRec *>(sc.prec);
    if (threadIdx.x < R) {
        const int64_t i = x0 + threadIdx.x;
        // (no local record: the compiler would lay it out in LDS by the
        // launch packet, in host memory: 12 us)
        const int64_t at = i < n ? i : n - 1;
        xs[threadIdx.x].w0 = rec[at].w0;
        xs[threadIdx.x].w1 = rec[at].w1;
        xs[threadIdx.x].la = rec[at].la;
        xs[threadIdx.x].ph = rec[at].ph;
    }
    __syncthreads();
    PairsWave &me = waves[wave];
    // the sums of x: with 32 samples lane comp 32 + xl has component comp of
    // sample xl, with 64 lane x has both components of sample x
    const int half = lane >> 5, xl = lane & 31;
    Acc2 acc[H];
    unsigned long long n_probe = 0, n_hit = 0, n_term = 0;

    // the contributions con[.][0..63] of the lanes in valid (x: the lane's
    // sample of the tile) into the owners' sums
    auto deposit = [&](bool valid, uint32_t x, double re, double im) {
        me.con[0][lane] = re;
        me.con[1][lane] = im;
        if (lane < R) me.own[lane] = 0ull;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if (valid) atomicOr(&me.own[x], 1ull << lane);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        unsigned long long mine = me.own[H == 1 ? xl : lane];
        while (mine) {
            const int k = __builtin_ctzll(mine);
            mine &= mine - 1;
            if constexpr (H == 1) {
                acc[0].add(me.con[half][k]);
            } else {
                acc[0].add(me.con[0][k]);
                acc[1].add(me.con[1][k]);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    };
    // <x|H|y> psi(y) / psi(x) of a pair whose group is g
    auto evaluate = [&](const PairRec &x, const PairRec &y, int64_t i, int64_t g, uint32_t cnt,
                        double &re, double &im) {
        const Key<W> xk = rec_key<W>(x);
        if constexpr (P == NQS_FP64) {
            double h;
            if constexpr (SCV) {
                h = sc_element<W>(tab, xk, rec_key<W>(y));
            } else {
                uint32_t *row = (DUMP && sign_bits) ? sign_bits + i * sign_words : nullptr;
                h = group_sum<W, DUMP>(tab, g, xk, row, &n_term, cnt);
            }
            const double2 rat = amp_ratio_f64(y.la - x.la, y.ph - x.ph);
            re = h * rat.x;
            im = h * rat.y;
        } else {
            const AccF32 h = group_sum_f32<W>(tab, g, xk, &n_term, cnt);
            float rr, ri;
            ratio_f32(y.la - x.la, y.ph - x.ph, rr, ri);
            const float pre = h.s * rr, pim = h.s * ri;
            re = static_cast<double>(pre) + static_cast<double>(fmaf(h.s, rr, -pre) + h.c * rr);
            im = static_cast<double>(pim) + static_cast<double>(fmaf(h.s, ri, -pim) + h.c * ri);
        }
    };
    uint32_t qn = 0, ln = 0;  // queue lengths (the same in every lane)
    auto flush_long = [&](uint32_t m) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        const bool on = lane < static_cast<int>(m);
        uint32_t x = 0;
        double re = 0.0, im = 0.0;
        if (on) {
            const uint2 e = me.lq[lane];
            x = e.x & 63u;
            evaluate(xs[x], rec[e.x >> 6], x0 + x, e.y, 0u, re, im);
        }
        deposit(on, x, re, im);
    };
    auto flush = [&](uint32_t m) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        bool now = false, later = false;
        uint32_t e = 0, x = 0;
        int64_t g = -1;
        double re = 0.0, im = 0.0;
        if (lane < static_cast<int>(m)) {
            e = me.q[lane];
            x = e & 63u;
            const int64_t i = x0 + x, j = e >> 6;
            if (i != j) {
                const PairRec y = rec[j];
                const Key<W> xk = rec_key<W>(xs[x]), yk = rec_key<W>(y);
                Key<W> d;
                uint64_t any = 0;
                int pop = 0;
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    d.w[w] = xk.w[w] ^ yk.w[w];
                    any |= d.w[w];
                    pop += __popcll(d.w[w]);
                }
                if (any == 0ull) {
                    latch(sc.err, NQS_E_DUPLICATE);
                } else {
                    ++n_probe;
                    uint32_t cnt = 0;
                    if constexpr (SCV && !DUMP) {
                        // the flip table: every single and double that keeps
                        // the parity of both spin counts
                        int pa = __popcll(d.w[0] & tab.spin_a0);
                        if constexpr (W == 2) pa += __popcll(d.w[W - 1] & tab.spin_a1);
                        g = (pop == 2 || pop == 4) && (pa & 1) == 0 ? 0 : -1;
                    } else {
                        g = group_find<W, SCV>(tab, d, &cnt);
                    }
                    if constexpr (DUMP) {
                        if (hit_idx && g >= 0)
                            hit_idx[i * tab.n_groups + g] = static_cast<int32_t>(j);
                    }
                    if (g >= 0) {
                        ++n_hit;
                        later = SCV ? pop == 2 : cnt > kShortTerms;
                        now = !later;
                        if (now) evaluate(xs[x], y, i, g, cnt, re, im);
                    }
                }
            }
        }
        const uint64_t lm = __ballot(later);
        if (later) me.lq[ln + lanes_below(lm)] = make_uint2(e, static_cast<uint32_t>(g));
        ln += static_cast<uint32_t>(__popcll(lm));
        // (near pairs need not be connected)
        if (__ballot(now)) deposit(now, x, re, im);
        if (ln >= 64) {
            flush_long(64);
            ln -= 64;
            if (lane < static_cast<int>(ln)) me.lq[lane] = me.lq[64 + lane];
        }
    };

    // the x operands, resident; the C operand: near pairs come out positive
    const uint32_t *__restrict__ words = reinterpret_cast<const uint32_t *>(sc.pkey) + lane;
    const int tiles = static_cast<int>((n + 31) / 32);
    // half of the lane's sample of tile t, 32 qubits of k-block kb
    auto column = [&](int t, int kb) { return words[(t * W + kb) * 64]; };
    v8i xo[H][W];
    uint32_t x_in = 0;  // bits of the halves whose sample exists
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int t = static_cast<int>(blockIdx.x) * H + h;
#pragma unroll
        for (int kb = 0; kb < W; ++kb) xo[h][kb] = fp4_signs(column(t < tiles ? t : tiles - 1, kb));
        if (x0 + 32 * h + xl < n) x_in |= 0xFFFFu << (16 * (H - 1 - h));
    }
    const float thr = 0.5f - static_cast<float>(64 * W - 2 * tab.max_flip);
    v16f cthr;
#pragma unroll
    for (int r = 0; r < 16; ++r) cthr[r] = thr;
    // this wave's tiles: every step-th; with more waves than tiles several
    // share a tile, each taking every share-th of its values
    const int all = kPairsWaves * static_cast<int>(gridDim.y);
    const int share = all >= 2 * tiles ? (all >= 8 * tiles ? 8 : (all >= 4 * tiles ? 4 : 2)) : 1;
    const int step = all / share;
    int t = wave + kPairsWaves * static_cast<int>(blockIdx.y);
    // (values v = t / step modulo share)
    uint32_t mine = x_in;
    if (share > 1) {
        const uint32_t every = share == 2 ? 0x55555555u : (share == 4 ? 0x11111111u : 0x01010101u);
        mine &= every << (t / step);
        t %= step;
    }
    uint32_t next[W];
#pragma unroll
    for (int kb = 0; kb < W; ++kb) next[kb] = column(t < tiles ? t : tiles - 1, kb);
    for (; t < tiles; t += step) {
        v16f c[H];
        v8i yo[W];
#pragma unroll
        for (int kb = 0; kb < W; ++kb) yo[kb] = fp4_signs(next[kb]);
#pragma unroll
        for (int h = 0; h < H; ++h) {
            c[h] = cthr;
#pragma unroll
            for (int kb = 0; kb < W; ++kb)
                c[h] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(yo[kb], xo[h][kb], c[h], 4,
                                                                       4, 0, 0, 0, 0);
        }
#pragma unroll
        for (int kb = 0; kb < W; ++kb) next[kb] = column(t + step < tiles ? t + step : t, kb);
        float mx = c[0][0];
#pragma unroll
        for (int v = 1; v < 16 * H; v += 2) {
            const int w = v + 1 < 16 * H ? v + 1 : v;
            mx = fmaxf(fmaxf(mx, c[v >> 4][v & 15]), c[w >> 4][w & 15]);
        }
        if (__ballot(mx > 0.0f) == 0ull) continue;
        // bit 16 H - 1 - v: value v = 16 h + r is positive (the lane's x is
        // 32 h + lane % 32, its y row 8 (r / 4) + 4 (lane / 32) + r % 4 of
        // the tile)
        uint32_t neg = 0;
#pragma unroll
        for (int v = 0; v < 16 * H; ++v)
            neg = (neg << 1) | (__float_as_uint(c[v >> 4][v & 15]) >> 31);
        uint32_t near = ~neg & mine;
        const int64_t y0 = static_cast<int64_t>(t) * 32;
        if (y0 + 32 > n) {
#pragma unroll
            for (int v = 0; v < 16 * H; ++v)
                if (y0 + 8 * ((v & 15) >> 2) + 4 * half + (v & 3) >= n)
                    near &= ~(1u << (16 * H - 1 - v));
        }
        for (;;) {
            const uint64_t any = __ballot(near != 0u);
            if (!any) break;
            if (near) {
                const uint32_t v = static_cast<uint32_t>(__builtin_clz(near)) - (32 - 16 * H);
                near &= ~(0x80000000u >> (v + 32 - 16 * H));
                const uint32_t y = static_cast<uint32_t>(y0) + 8 * ((v & 15u) >> 2) +
                                   4 * static_cast<uint32_t>(half) + (v & 3u);
                me.q[qn + lanes_below(any)] = (static_cast<uint32_t>(xl) + 32 * (v >> 4)) | (y << 6);
            }
            qn += static_cast<uint32_t>(__popcll(any));
            if (qn >= 64) {
                flush(64);
                qn -= 64;
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                if (lane < static_cast<int>(qn)) me.q[lane] = me.q[64 + lane];
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            }
        }
    }
    if (qn) flush(qn);
    if (ln) flush_long(ln);
    // the waves' sums in wave order (through the contribution arrays), one
    // component at a time
#pragma unroll
    for (int h = 0; h < H; ++h) {
        __syncthreads();
        me.con[0][lane] = acc[h].hi;
        me.con[1][lane] = acc[h].lo;
        __syncthreads();
        if (wave == h) {
            Acc2 s;
            for (int w = 0; w < kPairsWaves; ++w)
                s.add(waves[w].con[0][lane], waves[w].con[1][lane]);
            const int comp = H == 1 ? half : h;
            const int64_t i = x0 + (H == 1 ? xl : lane);
            if (i < n) {
                if (gridDim.y == 1) {
                    sc.ppart[2 * i + comp] = s.value();
                } else {
                    double *p =
                        sc.ppart + 4 * (static_cast<int64_t>(blockIdx.y) * n + i) + 2 * comp;
                    p[0] = s.hi;
                    p[1] = s.lo;
                }
            }
        }
    }
    // counters, one set of atomics per wave
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        n_probe += __shfl_xor(n_probe, off);
        n_hit += __shfl_xor(n_hit, off);
        n_term += __shfl_xor(n_term, off);
    }
    if (lane == 0) {
        count_add(sc.counters, 1, n_probe);
        count_add(sc.counters, 2, n_hit);
        count_add(sc.counters, 3, n_term);
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
        count_add(sc.counters, 4,
                  static_cast<unsigned long long>(n) * static_cast<unsigned long long>(n - 1));
}

}  // namespace

// 32 + 8 or 16 bytes per sample, the latter for whole tiles: within the
// hash's 64 or 96 (128 slots at least).
void pairs_scratch_layout(int64_t n, char *base, DevScratch *sc) {
    sc->prec = base;
    sc->pkey = base + sizeof(PairRec) * n;
}

hipError_t launch_pairs_prep(const DevTable &tab, const DevScratch &sc, const uint64_t *samples,
                             const int64_t *weights, const double *log_amp, const double *phase,
                             int64_t n, hipStream_t st) {
    const uint32_t jparts = sc.jctl ? static_cast<uint32_t>(sc.join_parts) : 0u;
    const uint32_t jhw =
        sc.jctl ? static_cast<uint32_t>((tab.join_blocks * n + 31) / 32) : 0u;
    int64_t span = (n + 31) / 32 * 32;
    const int64_t least[] = {kCounters * kCounterSlots, kJoinCtl, jparts, jhw};
    for (int64_t v : least) span = v > span ? v : span;
    hipLaunchKernelGGL(pairs_prep_kernel, dim3(static_cast<unsigned>((span + 255) / 256)),
                       dim3(256), 0, st, tab, sc, samples, weights, log_amp, phase, n,
                       jparts, jhw);
    return hipGetLastError();
}

hipError_t launch_pairs(const DevTable &tab, const DevScratch &sc, int64_t n, int precision,
                        int32_t *hit_idx, uint32_t *sign_bits, int64_t sign_words,
                        hipStream_t st) {
    const bool dump = hit_idx || sign_bits;
    const bool f32 = precision == NQS_FP32_KAHAN && !dump && !tab.sc;
    const bool wide = n > kPairsWide;
    const int64_t rows = wide ? 64 : 32;
    const dim3 grid(static_cast<unsigned>((n + rows - 1) / rows),
                    static_cast<unsigned>(sc.pairs_split));
#define NQS_AP(Wd, D, Pr, SCI)                                                                  \
    do {                                                                                        \
        if (wide)                                                                               \
            hipLaunchKernelGGL((pairs_kernel<Wd, 2, D, Pr, SCI>), grid, dim3(kPairsThreads), 0, \
                               st, tab, sc, n, hit_idx, sign_bits, sign_words); \
        else                                                                                    \
            hipLaunchKernelGGL((pairs_kernel<Wd, 1, D, Pr, SCI>), grid, dim3(kPairsThreads), 0, \
                               st, tab, sc, n, hit_idx, sign_bits, sign_words); \
    } while (0)
    const bool w1 = tab.n_qubits <= 63;
    if (tab.sc) {
        if (w1) {
            if (dump) NQS_AP(1, true, NQS_FP64, true); else NQS_AP(1, false, NQS_FP64, true);
        } else {
            if (dump) NQS_AP(2, true, NQS_FP64, true); else NQS_AP(2, false, NQS_FP64, true);
        }
    } else if (w1) {
        if (dump) NQS_AP(1, true, NQS_FP64, false);
        else if (f32) NQS_AP(1, false, NQS_FP32_KAHAN, false);
        else NQS_AP(1, false, NQS_FP64, false);
    } else {
        if (dump) NQS_AP(2, true, NQS_FP64, false);
        else if (f32) NQS_AP(2, false, NQS_FP32_KAHAN, false);
        else NQS_AP(2, false, NQS_FP64, false);
    }
#undef NQS_AP
    return hipGetLastError();
}

}  // namespace nqs
