// batch_ffn.hip -- the gate/up half of the expert FFN of 2 to 16 decode tokens (gfx950).
//
// A decode batch is bound by the bytes of the distinct experts that it selects (61 on average for 16
// tokens of top-8 over 256 Zipf-routed experts: 384 MB of bf16).  Two kernels read each weight once:
// on the matrix cores a weight tile is loaded straight into registers in their lane layout and multiplied
// with all of its expert's tokens at once, so that a wave has nothing to do per token and its loads stay in
// flight; with one wave per row pair the tokens follow one another, and a block starts after two dependent
// loads instead of a search over all the pairs.  rows_faster() says which call takes which.
#include "internal.h"
#include "device_common.h"

namespace moe {
namespace {

using namespace dev;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kMaxPairs = MOE_MAX_DECODE_TOKENS * MOE_MAX_TOPK;  // (token, rank) pairs of a call

// High halves of two floats as a bf16 pair (lo's in the low half).
__device__ __forceinline__ uint32_t high_halves(float lo, float hi) {
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

// Eight fp32 values -> three bf16x8 terms whose sum is exact: each term takes the top 8 significant bits
// of what the terms before it leave (truncation: no finite value overflows, and 24 bits take three terms).
// PAIRS: the order 0,4,1,5,2,6,3,7 (int4 weights).
template <bool PAIRS>
__device__ __forceinline__ void split3(const float *v, bf16x8 &t1, bf16x8 &t2, bf16x8 &t3) {
    uint32_t a[4], b[4], c[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x0 = v[PAIRS ? e : 2 * e], x1 = v[PAIRS ? e + 4 : 2 * e + 1];
        a[e] = high_halves(x0, x1);
        const float r0 = x0 - __uint_as_float(__float_as_uint(x0) & 0xffff0000u);
        const float r1 = x1 - __uint_as_float(__float_as_uint(x1) & 0xffff0000u);
        b[e] = high_halves(r0, r1);
        const float q0 = r0 - __uint_as_float(__float_as_uint(r0) & 0xffff0000u);
        const float q1 = r1 - __uint_as_float(__float_as_uint(r1) & 0xffff0000u);
        c[e] = high_halves(q0, q1);
    }
    t1 = __builtin_bit_cast(bf16x8, make_uint4(a[0], a[1], a[2], a[3]));
    t2 = __builtin_bit_cast(bf16x8, make_uint4(b[0], b[1], b[2], b[3]));
    t3 = __builtin_bit_cast(bf16x8, make_uint4(c[0], c[1], c[2], c[3]));
}

// The eight signed nibbles q of a dword as bf16 q / 16 (exact), in the order 0,4,1,5,2,6,3,7.  Two bit operations per
// pair give 24 + q instead, but sums that carry 24 times the sum of the other factors round at that size: 9 tokens,
// H 2048, I 2048, top-16 + shared: 2.4e-7 from 64 bits in 227 us, q / 16: 1.7e-7 in 231 us, one wave per row pair: 2.2e-7
// in 495 us (16 tokens, I 512, top-8 of 256 + shared: 54, 57 and 135 us).
__device__ __forceinline__ bf16x8 nibbles_16th(uint32_t v) {
    uint32_t p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        p[e] = high_halves(__builtin_amdgcn_cvt_off_f32_i4(int(v >> (4 * e))), __builtin_amdgcn_cvt_off_f32_i4(int(v >> (4 * e + 16))));
    return __builtin_bit_cast(bf16x8, make_uint4(p[0], p[1], p[2], p[3]));
}

// One row's dot product in fp32, element by element: what a sum of three-term products that is not finite is taken
// from.  Those terms give NaN for an infinite factor (inf - inf in the split, 0 times inf in a term that is zero or
// a step past the wave's share) and can overflow on the way; a row-wise dot product gives what the factors give.
template <int DT>
__device__ __forceinline__ float row_dot(const uint8_t *blob, int row, const float *x, int H, int I) {
    const uint8_t *w = blob + row * row_bytes_of(DT, H);
    const auto *sc = reinterpret_cast<const uint16_t *>(blob + size_t(I) * H) + size_t(row) * (H / 128);  // (int4)
    float acc = 0.f;
#pragma unroll 1
    for (int c = 0; c < H; c += 32) {
        float part = 0.f;
#pragma unroll 1
        for (int h = c; h < c + 32; ++h) {
            float v;
            if constexpr (DT == BF16) v = bf16_bits_to_float(reinterpret_cast<const uint16_t *>(w)[h]);
            else v = float(int(__builtin_amdgcn_sbfe(uint32_t(w[h / 2]), 4 * (h & 1), 4)));
            part = fmaf(v, x[h], part);
        }
        acc += DT == INT4 ? bf16_bits_to_float(sc[c / 128]) * part : part;
    }
    return acc;
}

// How a block walks an expert's gate/up matrix.  A step is one 16-byte weight load per lane and 16-row tile:
// lane (lr = l % 16, lg = l / 16) holds row lr, elements STEP / 4 * lg onward of the step, and the same
// elements of token lr.  An item is TILES tiles of one expert; its eight waves take contiguous shares of the
// steps, CS (at most MAXS) of them at a time in registers.  CHAINS: independent fp32 sums of the leading
// products, so that a chain of roundings is no longer than a lane's in a row-wise dot product.
template <int DT> struct Walk;
template <> struct Walk<BF16> { static constexpr int STEP = 32, TILES = 1, MAXS = 8, CHAINS = 2; };
template <> struct Walk<INT4> { static constexpr int STEP = 128, TILES = 2, MAXS = 2, CHAINS = 1; };

constexpr int kBatchWaves = 8, kBatchBlock = kBatchWaves * kWave;
constexpr int kBatchGrid = 256;  // one persistent block per compute unit

// The call's experts, found by every block for itself (no launch groups the pairs first): group n's blob as a
// byte offset from `pool` and its key; each pair's key (-1: a pair that contributes nothing).  A group holds
// at most 16 pairs: an expert has more only where tokens name it twice, and then takes several groups.
struct BatchGroups {
    alignas(16) int ids[kMaxPairs];  // (read four at a time)
    int n;
    long long off[kMaxPairs + 1];
    long long group_key[kMaxPairs + 1];  // -1: the shared expert's group (every token)
    long long key[kMaxPairs];            // 16 * expert + (the pair's rank among its expert's pairs) / 16
    float weight[kMaxPairs];
    int per_wave[kMaxPairs / kWave];
};
static_assert(offsetof(BatchGroups, ids) % 16 == 0 && alignof(BatchGroups) % 16 == 0);

__device__ __forceinline__ void find_groups(BatchGroups &G, int P, int E, const int32_t *__restrict__ ids,
                                            const int32_t *__restrict__ slot_of, const float *__restrict__ weights,
                                            const uint8_t *pool, size_t expert_bytes, const uint8_t *shared_w, int *err) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    int e = -1, s = -1;
    if (tid < kMaxPairs) {
        float w = 0.f;
        if (tid < P) {
            e = ids[tid];
            w = weights[tid];
        }
        const bool in = e >= 0 && e < E;
        G.ids[tid] = in ? e : -1;
        G.weight[tid] = w;
        if (in) s = slot_of ? slot_of[e] : e;
        if (tid < P && blockIdx.x == 0) {
            if (!in) atomicOr(err, kErrRange);
            else if (s < 0) atomicOr(err, kErrNotResident);
        }
    }
    __syncthreads();
    bool first = false;
    long long key = -1;
    unsigned long long firsts = 0;
    if (tid < kMaxPairs) {
        int rank = 0;
        const int4 *v = reinterpret_cast<const int4 *>(G.ids);
        const int nq = min(P, (wave + 1) * kWave);  // (the pairs before any of this wave's)
        for (int q = 0; q < nq; q += 4) {
            const int4 o = v[q / 4];
            rank += (o.x == e && q < tid) + (o.y == e && q + 1 < tid) + (o.z == e && q + 2 < tid) + (o.w == e && q + 3 < tid);
        }
        if (s >= 0) key = 16ll * e + rank / 16;
        G.key[tid] = key;
        first = s >= 0 && rank % 16 == 0;
        firsts = __ballot(first);
        if (lane == 0) G.per_wave[wave] = __popcll(firsts);
    }
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kMaxPairs / kWave; ++w) {
        before += w < wave ? G.per_wave[w] : 0;
        all += G.per_wave[w];
    }
    if (first) {
        const int n = before + __popcll(firsts & ((1ull << lane) - 1ull));
        G.off[n] = (long long)s * (long long)expert_bytes;
        G.group_key[n] = key;
    }
    if (tid == 0) {
        G.n = all + (shared_w != nullptr);
        if (shared_w) {
            G.off[all] = (long long)(shared_w - pool);
            G.group_key[all] = -1;
        }
    }
    __syncthreads();
}

// act[p, i] = w_p * silu(W_g[i] . x_t) * (W_u[i] . x_t) for every (token, rank) pair p and the shared expert.
// Each block takes a contiguous share of the (expert, row tiles) items and streams their weights: the next
// item's are in flight while this one is multiplied, and the expert's tokens stay in registers from item to
// item.  The waves' partial products are added through LDS in wave order.  The weights (int4: as bf16 q / 16,
// the scale applied to each quantisation group's fp32 sum) meet the tokens' values as three bf16 terms, so
// that every product is exact and only the order of the fp32 sums differs from a row-wise dot product.
// Bound by HBM (large batches) or by the latency of a few items per block (small ones).  Measured against one
// wave per row pair that took its expert's tokens one after the other, behind a launch that grouped the pairs:
// 16 tokens, H 2048, I 512, 256 Zipf-routed bf16 experts + shared (251 MB): 54 + 16 -> 53 us, 4.7 TB/s; 5
// tokens on int4 experts of the same shape (31 MB): 31 + 6 -> 19 us.
template <int DT, int CS, bool ONE>  // ONE: a single pass over the reduction range
__global__ __launch_bounds__(kBatchBlock, 2) void batch_gateup_kernel(
    const float *__restrict__ x, int T, int H, int I, int E, int k, const int32_t *__restrict__ ids,
    const int32_t *__restrict__ slot_of, const uint8_t *__restrict__ pool, size_t expert_bytes,
    const uint8_t *__restrict__ shared_w, const float *__restrict__ weights, float *__restrict__ act, int *err) {
    using W = Walk<DT>;
    constexpr int MT = W::TILES, XV = W::STEP / 4, CH = W::CHAINS;  // XV: fp32 values per lane and step
    constexpr int SUB = DT == INT4 ? 4 : 1;                         // matrix products per step and term
    __shared__ float red[2][kBatchWaves][MT][4][kWave];
    __shared__ BatchGroups G;
    __shared__ int members[kBatchWaves][kMaxPairs];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int lr = lane % 16, lg = lane / 16;
    const int P = T * k;
    find_groups(G, P, E, ids, slot_of, weights, pool, expert_bytes, shared_w, err);

    int *mem = members[wave];  // the pairs of the expert at hand, ascending
    const int tiles = 2 * I / (16 * MT);
    const int items = G.n * tiles;
    const int it0 = int((long long)items * blockIdx.x / gridDim.x), it1 = int((long long)items * (blockIdx.x + 1) / gridDim.x);
    if (it0 >= it1) return;
    const int steps = H / W::STEP;
    const int chunks = ONE ? 1 : (steps + kBatchWaves * CS - 1) / (kBatchWaves * CS);  // passes over the reduction range
    const int share = (steps + kBatchWaves * chunks - 1) / (kBatchWaves * chunks);  // steps per wave and pass, <= CS
    const size_t rb = row_bytes_of(DT, H);
    const int KG = H / 128;

    struct Weights {
        uint4 w[CS][MT];
        uint32_t sc[DT == INT4 ? CS : 1][MT];
    } b0, b1;
    struct Unit {  // one pass over one item
        int it, g, tile, c;
    };
    auto next_unit = [&](Unit u) {
        if (++u.c == chunks) {
            u.c = 0;
            ++u.it;
            if (++u.tile == tiles) {
                u.tile = 0;
                ++u.g;
            }
        }
        return u;
    };
    // This wave's steps of pass c: [first, first + live)
    auto first_step = [&](int c) { return (c * kBatchWaves + wave) * share; };
    // (No branch around these loads, and no other load between them and their use: they are counted, and a
    // wait for one item's weights leaves the next one's in flight.  Past the block's last unit they all read
    // one line.)
    auto load = [&](Weights &b, const Unit &u) __attribute__((always_inline)) {
        const bool more = u.it < it1;
        const int row0 = u.tile * 16 * MT, s0 = first_step(u.c);
        const uint8_t *blob = pool + (more ? G.off[u.g] : 0);
        const size_t row = more ? size_t(row0 + lr) : 0;
        const uint8_t *wrow = blob + row * rb + 16 * lg;
        const uint16_t *srow = reinterpret_cast<const uint16_t *>(blob + (more ? size_t(I) * H : 0)) + row * KG;
        const size_t wt = more ? 16 * rb : 0, st = more ? 16 * KG : 0;  // from tile to tile
        const int last = more ? steps - 1 : 0;
#pragma unroll
        for (int r = 0; r < CS; ++r) {
            const int s = min(s0 + r, last);  // (past the end: loaded, not multiplied)
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                b.w[r][j] = load16_stream(wrow + j * wt + size_t(s) * 64);
                if constexpr (DT == INT4) b.sc[r][j] = srow[j * st + s];
            }
        }
    };

    bf16x8 xt[CS][SUB][3];
    floatx4 lead[CH][MT], tail[MT];
    int cnt = 0, g_at = -1;
    auto process = [&](Weights &b, const Unit &u, Weights &next, const Unit &un) __attribute__((always_inline)) {
        const int it = u.it, c = u.c, g = u.g;
        const int row0 = u.tile * 16 * MT, s0 = first_step(c), live = min(share, steps - s0);
        const bool fresh = g != g_at;
        if (fresh) {
            g_at = g;
            const long long gk = G.group_key[g];
            if (gk < 0) {
                cnt = T;
                if (lane < T) mem[lane] = P + lane;
            } else {
                cnt = 0;
#pragma unroll
                for (int m = 0; m < kMaxPairs / kWave; ++m) {
                    const int p = m * kWave + lane;
                    const unsigned long long mask = __ballot(G.key[p] == gk);
                    if (mask >> lane & 1ull) mem[cnt + __popcll(mask & ((1ull << lane) - 1ull))] = p;
                    cnt += __popcll(mask);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
        if (fresh || chunks > 1) {
            // the tokens' values of this wave's steps (columns past the last token repeat it and are not stored;
            // steps past the wave's share take zeros)
            const int p = mem[min(lr, cnt - 1)];
            const float *xrow = x + size_t(p < P ? p / k : p - P) * H + XV * lg;
            float4 raw[CS][XV / 4];
#pragma unroll
            for (int r = 0; r < CS; ++r)
#pragma unroll
                for (int q = 0; q < XV / 4; ++q)
                    raw[r][q] = load_f4(reinterpret_cast<const float4 *>(xrow + size_t(min(s0 + r, steps - 1)) * W::STEP) + q);
#pragma unroll
            for (int r = 0; r < CS; ++r) {
                const uint32_t keep = r < live ? ~0u : 0u;
#pragma unroll
                for (int q = 0; q < XV / 4; ++q) {
                    float4 &f = raw[r][q];
                    f = make_float4(__uint_as_float(__float_as_uint(f.x) & keep), __uint_as_float(__float_as_uint(f.y) & keep),
                                    __uint_as_float(__float_as_uint(f.z) & keep), __uint_as_float(__float_as_uint(f.w) & keep));
                }
#pragma unroll
                for (int d = 0; d < SUB; ++d) {
                    const float4 a = raw[r][2 * d], bq = raw[r][2 * d + 1];
                    const float v[8] = {a.x, a.y, a.z, a.w, bq.x, bq.y, bq.z, bq.w};
                    split3<DT == INT4>(v, xt[r][d][0], xt[r][d][1], xt[r][d][2]);
                }
            }
        }
        load(next, un);
        // (the weights at hand pass through an empty asm after the next item's loads: those are all issued first)
#pragma unroll
        for (int r = 0; r < CS; ++r)
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                u32x4 v = {b.w[r][j].x, b.w[r][j].y, b.w[r][j].z, b.w[r][j].w};
                asm volatile("" : "+v"(v)::"memory");
                b.w[r][j] = make_uint4(v.x, v.y, v.z, v.w);
            }
        if (c == 0) {
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                tail[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int h = 0; h < CH; ++h) lead[h][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int r = 0; r < CS; ++r) {
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                const uint32_t wv[4] = {b.w[r][j].x, b.w[r][j].y, b.w[r][j].z, b.w[r][j].w};
                if constexpr (DT == BF16) {
                    const bf16x8 w = __builtin_bit_cast(bf16x8, b.w[r][j]);
                    tail[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[r][0][2], w, tail[j], 0, 0, 0);
                    lead[r % CH][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[r][0][0], w, lead[r % CH][j], 0, 0, 0);
                    tail[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[r][0][1], w, tail[j], 0, 0, 0);
                } else {
                    floatx4 hi = {0.f, 0.f, 0.f, 0.f}, lo = hi;
#pragma unroll
                    for (int d = 0; d < SUB; ++d) {
                        const bf16x8 w = nibbles_16th(wv[d]);
                        lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[r][d][2], w, lo, 0, 0, 0);
                        hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[r][d][0], w, hi, 0, 0, 0);
                        lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt[r][d][1], w, lo, 0, 0, 0);
                    }
                    const float sc = bf16_bits_to_float(b.sc[r][j]);
#pragma unroll
                    for (int q = 0; q < 4; ++q) lead[0][j][q] = fmaf(sc, 16.f * (hi[q] + lo[q]), lead[0][j][q]);
                }
            }
        }
        if (c + 1 < chunks) return;
        // lane holds C[token 4 lg + q][row lr] of each tile; two buffers, so that one barrier per item suffices
        auto &rd = red[it & 1];
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v = tail[j][q];
#pragma unroll
                for (int h = CH / 2; h > 0; h /= 2)
#pragma unroll
                    for (int i = 0; i < h; ++i) lead[i][j][q] += lead[i + h][j][q];
                rd[wave][j][q][lane] = v + lead[0][j][q];
            }
        __syncthreads();
        // 8 activations per tile and token: gate row 2i and up row 2i + 1
        const int i = tid % (8 * MT), col = tid / (8 * MT);
        if (col < cnt && col < 16) {
            const int j = i / 8, q = col % 4, l = 16 * (col / 4) + 2 * (i % 8);
            float gate = 0.f, up = 0.f;
#pragma unroll
            for (int w = 0; w < kBatchWaves; ++w) {
                gate += rd[w][j][q][l];
                up += rd[w][j][q][l + 1];
            }
            const int p = mem[col];
            const float wp = p < P ? G.weight[p] : 1.f;
            if (!(fabsf(gate) < INFINITY && fabsf(up) < INFINITY)) {
                const float *xt = x + size_t(p < P ? p / k : p - P) * H;
                gate = row_dot<DT>(pool + G.off[g], row0 + 2 * i, xt, H, I);
                up = row_dot<DT>(pool + G.off[g], row0 + 2 * i + 1, xt, H, I);
            }
            act[size_t(p) * I + row0 / 2 + i] = wp * (gate * __builtin_amdgcn_rcpf(1.f + __expf(-gate)) * up);
        }
    };
    Unit ua = {it0, it0 / tiles, it0 % tiles, 0};
    load(b0, ua);
    while (ua.it < it1) {
        const Unit ub = next_unit(ua);
        process(b0, ua, b1, ub);
        ua = next_unit(ub);
        if (ub.it < it1) process(b1, ub, b0, ua);
    }
}

// One wave per row pair (gate row 2i, up row 2i + 1): its weights are loaded once and applied to each token of the
// expert (fp32 experts always: fp32 matrix instructions measured no faster here, and their longer chains of roundings
// less exact).  Block (row pairs, p): for all the pairs of pair p's expert if p is the first of them (the
// other blocks leave: each wave finds the expert's pairs by ballots over the ids, so that no launch groups
// them first: 5.3 us of the 31.8 us of 7 tokens at H 1408, I 384); p = T * k is the shared expert.
// NCH is a row's exact number of 64-lane chunks (H 2560, bf16, 16 tokens of top-8 over 128 experts of I 768: 195 us
// with eight chunks for five, 155 with five).  PACKED: the weights are unpacked anew for every token, since unpacked
// they take twice the registers (bf16, H 4096: 216 and 2 waves per SIMD, 152 and 3; 4 tokens, I 1024: 65 -> 61 us).
template <int DT, int NCH, bool FULL, bool PACKED>
__global__ __launch_bounds__(kBlock) void batch_gateup_rows_kernel(
    const float *__restrict__ x, int T, int H, int I, int E, int k, const int32_t *__restrict__ ids,
    const int32_t *__restrict__ slot_of, const uint8_t *__restrict__ pool, size_t expert_bytes,
    const uint8_t *__restrict__ shared_w, const float *__restrict__ weights, float *__restrict__ act, int *err) {
    constexpr int EPC = Fmt<DT>::EPC;
    __shared__ int members[kBlock / kWave][kMaxPairs];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int g = blockIdx.y, P = T * k;
    int *mem = members[wave];  // the expert's pairs, ascending
    int cnt;
    const uint8_t *blob;
    if (g < P) {
        int id[kMaxPairs / kWave];
#pragma unroll
        for (int m = 0; m < kMaxPairs / kWave; ++m) id[m] = ids[min(m * kWave + lane, P - 1)];
        int e = 0;
#pragma unroll
        for (int m = 0; m < kMaxPairs / kWave; ++m)
            if (g / kWave == m) e = __builtin_amdgcn_readlane(id[m], g % kWave);
        if (e < 0 || e >= E) {
            if (blockIdx.x == 0 && tid == 0) atomicOr(err, kErrRange);
            return;
        }
        const int s = slot_of ? load_stream_word(slot_of + e) : e;
        cnt = 0;
        bool first = true;
#pragma unroll
        for (int m = 0; m < kMaxPairs / kWave; ++m) {
            const int p = m * kWave + lane;
            const unsigned long long mask = __ballot(p < P && id[m] == e);
            if (mask >> lane & 1ull) mem[cnt + __popcll(mask & ((1ull << lane) - 1ull))] = p;
            if (cnt == 0 && mask) first = m * kWave + int(__builtin_ctzll(mask)) == g;
            cnt += __popcll(mask);
        }
        if (!first) return;
        if (s < 0) {
            if (blockIdx.x == 0 && tid == 0) atomicOr(err, kErrNotResident);
            return;
        }
        blob = pool + size_t(s) * expert_bytes;
    } else {
        cnt = T;
        if (lane < T) mem[lane] = P + lane;
        blob = shared_w;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const size_t rb = row_bytes_of(DT, H);
    float xv[NCH][EPC];
    auto load_token = [&](int p) {
        const float *xt = x + size_t(p < P ? p / k : p - P) * H;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int col0 = (c * kWave + lane) * EPC;
            if (FULL || col0 < H) {
                load_x<DT>(xt, col0, xv[c]);
            } else {
#pragma unroll
                for (int q = 0; q < EPC; ++q) xv[c][q] = 0.f;
            }
        }
    };
    load_token(mem[0]);  // before the weights: loads retire in order, so waiting for x never waits for them
    bool again = false;
    for (int i = blockIdx.x * (kBlock / kWave) + wave; i < I; i += gridDim.x * (kBlock / kWave), again = true) {
        const uint8_t *gate = blob + size_t(2 * i) * rb + 16 * lane;
        uint4 wg[NCH], wu[NCH];
        float sg[DT == INT4 ? NCH : 1], su[DT == INT4 ? NCH : 1];
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int col0 = (c * kWave + lane) * EPC;
            const bool in = FULL || col0 < H;
            wg[c] = in ? load16_stream(gate + size_t(c) * 16 * kWave) : make_uint4(0, 0, 0, 0);
            wu[c] = in ? load16_stream(gate + rb + size_t(c) * 16 * kWave) : make_uint4(0, 0, 0, 0);
            if constexpr (DT == INT4) {
                const uint16_t *sc = reinterpret_cast<const uint16_t *>(blob + size_t(I) * H) + size_t(2 * i) * (H / 128) + col0 / 128;
                sg[c] = in ? bf16_bits_to_float(sc[0]) : 0.f;
                su[c] = in ? bf16_bits_to_float(sc[H / 128]) : 0.f;
            }
        }
        for (int q = 0; q < cnt; ++q) {
            const int p = mem[q];
            if (q > 0 || (again && cnt > 1)) load_token(p);
            const float wp = p < P ? weights[p] : 1.f;
            float ga = 0.f, ua = 0.f;
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                if constexpr (PACKED) {  // (unpacked again for every token: the compiler would keep them unpacked)
                    uint4 &a = wg[c], &b = wu[c];
                    asm volatile("" : "+v"(a.x), "+v"(a.y), "+v"(a.z), "+v"(a.w), "+v"(b.x), "+v"(b.y), "+v"(b.z), "+v"(b.w));
                }
                const float dg = chunk_dot<DT>(wg[c], xv[c]), du = chunk_dot<DT>(wu[c], xv[c]);
                ga += DT == INT4 ? dg * sg[c] : dg;
                ua += DT == INT4 ? du * su[c] : du;
            }
            ga = wave_sum(ga);
            ua = wave_sum(ua);
            if (lane == 0) act[size_t(p) * I + i] = wp * (ga * __builtin_amdgcn_rcpf(1.f + __expf(-ga)) * ua);
        }
    }
}

// Which kernel: one wave per row pair (true) or the matrix cores.  The matrix cores win where many of a wave's tokens
// would follow one another; their cost is the search before the first load and steps that fill no whole pass.  Row
// pairs / matrix cores, us for the whole FFN:
// bf16, by the tokens per expert T k / E and by T (the most chosen experts' tokens, and the shared expert's T).  H 2048,
// I 768, top-8 of 128: 55 / 60 at 6 tokens, 92 / 93 at 12, 117 / 113 at 16 (T k / E = 1); top-4 of 16: 28.1 / 30.6 at
// 6 (1.5), 39 / 37 at 10 (2.5); H 1024, I 1536, top-4 of 32: 41 / 43 at 10 (1.25), 56 / 54 at 16 (2).  With a shared
// expert: H 2048, I 512, top-8 of 256: 47 / 48 at 6, 59 / 57 at 8, 102 / 90 at 16; H 1024, I 768: 44 / 46 at 7, 58 /
// 57 at 10.  Up to H 768, and from 1025 to 1536, a quarter or more of a matrix-core pass's steps are empty: twice as
// many (H 512, I 3072, top-4 of 32, 16 tokens: 71 / 86; H 1280, I 512, top-8 of 256 + shared, 16 tokens: 75 / 79).
// Beyond H 2048 the matrix cores would read the tokens anew in every pass (H 2560, I 768, 16 tokens: 140 / 285).
// int4, by blocks times the tokens that follow one another, since a row pair's products cost several times the loads
// there: H 2048, I 128, top-1 of 16: 12.5 / 14.9 at 6 tokens (1152), 20.8 / 19.4 at 12 (4608); H 6144: 18.9 / 26.1
// at 4 (512), 42 / 44 at 12 (4608, where the line costs 4 %); H 2176, I 256, top-2 of 16: 15.3 / 17.3 at 4 (2048), 20 / 19.2 at 6 (4608); with a shared
// expert H 4096, I 128, top-2 of 8: 14.6 / 18.5 at 3 (1728), 24 / 22 at 5 (4800).
bool rows_faster(int T, int H, int I, int E, int k, int dtype, bool shared) {
    if (dtype == F32) return true;
    if (dtype == INT4) return H <= 8192 && (long long)(I / 4) * T * (k + shared) * T * (1 + shared) <= 2048;
    if (H > 2048) return true;
    const bool idle = H <= 768 || (H > 1024 && H <= 1536);
    const long long pairs = 40ll * T * k, limit = (shared ? 50ll : 60ll) * E * (idle ? 2 : 1);  // in units of E / 40
    return shared ? pairs + 5ll * T * E < limit : pairs + 3ll * (T > 8 ? T - 8 : 0) * E <= limit;
}

}  // namespace

hipError_t launch_batch_gateup(const float *x, int T, int H, int I, int E, int k, const int32_t *ids,
                               const float *weights, const int32_t *slot_of, const uint8_t *pool, size_t expert_bytes,
                               int dtype, const uint8_t *shared_w, float *act, int *err, hipStream_t s) {
    if (T < 2 || T > MOE_MAX_DECODE_TOKENS || k < 1 || k > MOE_MAX_TOPK || H % 128 || I % 128) return hipErrorInvalidValue;
#define GU_LAUNCH(DT, CS, ONE)                                                                                 \
    {                                                                                                          \
        batch_gateup_kernel<DT, CS, ONE><<<kBatchGrid, kBatchBlock, 0, s>>>(x, T, H, I, E, k, ids, slot_of, pool,   \
                                                                       expert_bytes, shared_w, weights, act, err); \
        return hipGetLastError();                                                                              \
    }
    if (rows_faster(T, H, I, E, k, dtype, shared_w != nullptr)) {
        const int pairs = T * k + (shared_w ? 1 : 0), quads = (I + kBlock / kWave - 1) / (kBlock / kWave);
        // Several row pairs per wave where a launch has several rounds of blocks: fewer prologues, and fewer blocks that
        // leave at once (bf16, I 2048, top-8 of 64, 4 tokens: H 2048 112 -> 103 us, H 512 45.6 -> 40.7, four pairs 38.8;
        // fp32, H 512, top-4 of 32, 16 tokens: 82 -> 73, four 76).  Not for small experts (H 1024, I 384, top-6 of 64, 16
        // tokens: 29 -> 33) and, for longer rows, with a shared expert, whose tokens would all follow one another twice
        // (H 2048, I 768, top-8 of 60, 4 tokens: 46 -> 49; H 512, I 768, top-8 of 64, 6 tokens: 25.5 -> 24.4).
        const int blocks = quads * pairs;
        const int per_wave = shared_w ? (H <= 512 && blocks >= 8192 ? 2 : 1)
                             : I < 768 || blocks < 4096 ? 1 : dtype == BF16 && H <= 512 && I >= 2048 ? 4 : 2;
        const dim3 grid(unsigned((quads + per_wave - 1) / per_wave), unsigned(pairs));
#define ROWS_LAUNCH(DT, N, FULL, PACKED)                                                                             \
    {                                                                                                                \
        batch_gateup_rows_kernel<DT, N, FULL, PACKED><<<grid, kBlock, 0, s>>>(x, T, H, I, E, k, ids, slot_of, pool,  \
                                                                              expert_bytes, shared_w, weights, act, err); \
        return hipGetLastError();                                                                                    \
    }
    // FULL: every lane's chunk slots lie inside the row, no bound checks.  PACKED where registers limit the waves of a
    // launch that fills the chip (bf16 rows that are not full: no; H 1792, I 512, top-6, 8 tokens: 40 against 45 us).
#define ROWS_CASE(DT, N)                                                                                             \
    if (dtype == DT && H <= N * kWave * Fmt<DT>::EPC) {                                                              \
        constexpr bool kPackFull = DT == BF16 && N >= 4, kPack = DT == INT4 && N >= 2;                                \
        if (H != N * kWave * Fmt<DT>::EPC) ROWS_LAUNCH(DT, N, false, kPack)                                          \
        if (!kPackFull || blocks < 2048) ROWS_LAUNCH(DT, N, true, kPack)                                    \
        ROWS_LAUNCH(DT, N, true, kPack || kPackFull)                                                                 \
    }
        ROWS_CASE(F32, 1) ROWS_CASE(F32, 2) ROWS_CASE(F32, 3) ROWS_CASE(F32, 4)
        ROWS_CASE(F32, 5) ROWS_CASE(F32, 6) ROWS_CASE(F32, 7) ROWS_CASE(F32, 8)
        ROWS_CASE(BF16, 1) ROWS_CASE(BF16, 2) ROWS_CASE(BF16, 3) ROWS_CASE(BF16, 4)
        ROWS_CASE(BF16, 5) ROWS_CASE(BF16, 6) ROWS_CASE(BF16, 7) ROWS_CASE(BF16, 8)
        ROWS_CASE(INT4, 1) ROWS_CASE(INT4, 2) ROWS_CASE(INT4, 3) ROWS_CASE(INT4, 4)
#undef ROWS_CASE
#undef ROWS_LAUNCH
        return hipErrorInvalidValue;
    }
    // the fewest steps per wave that hold a wave's share of the reduction range (longer int4 rows take passes)
#define GU_CASE(DT)                                                                       \
    if (dtype == DT) {                                                                    \
        const int share = (H / Walk<DT>::STEP + kBatchWaves - 1) / kBatchWaves;           \
        if (share <= Walk<DT>::MAXS / 2) GU_LAUNCH(DT, Walk<DT>::MAXS / 2, true)          \
        if (share <= Walk<DT>::MAXS) GU_LAUNCH(DT, Walk<DT>::MAXS, true)                  \
        if constexpr (DT == INT4) GU_LAUNCH(DT, Walk<DT>::MAXS, false)                    \
    }
    GU_CASE(BF16) GU_CASE(INT4)
#undef GU_CASE
#undef GU_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace moe
