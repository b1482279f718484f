// The consumer of the injected pages: attention logits of each request's
// query against the keys of its placed tokens, read back through the block
// table (Theorem "Chunked RoPE Injection", §5.1: a key rotated at position p
// scores against a query at position N exactly as the stored key would at
// relative position p - N; §3.3: the query follows the memory). Grouped-query
// heads: query head hq reads KV head hq / (Hq / H).
//
//   * the logits of one KV head are a small matrix product, its G query heads
//     times the tokens' keys, so they run on the matrix cores: 16 tokens x 16
//     rows per v_mfma_f32_16x16x32_bf16. The rotated query is fp32; it is split
//     exactly into three bf16 parts (8 + 8 + 8 significand bits), which take
//     three of the four rows of each query head and are added at the end,
//     smallest first. Products are exact, sums fp32, of at most 128 elements
//     each: relative error (2-norm) against 64 bits for D = 16 / 64 / 128 / 256 /
//     512: 6.0 / 7.7 / 8.6 / 9.0 / 9.4e-8, where one fp32 multiply-add per element summed over
//     D / 8 lanes gives 7.9 / 9.3 / 9.5 / 10.0 / 10.3e-8.
//   * one block per (share of the placed tokens, share of the heads, request),
//     whatever the capacity max_tokens: it maps its tokens to slots (512 at a
//     time), rotates its query heads to qpos[r] (one sine and
//     cosine per pair, fp64-reduced angles as the inject kernel's) and then its
//     waves take (head, 16 tokens) items. A wave loads an item's keys coalesced
//     (whole 128-byte lines), turns them into fragments through a part of LDS
//     of its own, and has the next item's loads in flight while it multiplies:
//     no barriers in the loop.
//   * a logit that comes out non-finite (an infinite or NaN operand, or a rotated
//     one past the largest bf16, has no split), and every logit of a query head
//     with a rotated element below 2^-100 (below 2^-110 the smallest bf16,
//     2^-133, cuts its lower parts short), is formed again in binary64 from the
//     fp32 rotation of the query in memory.
// Bound: the keys' bytes, and the set-up (two dependent round trips before the
// first key is asked for). 32 requests of 1,280-2,560 tokens, 32 / 8 heads of
// 128, 134 MB: 30.5 us = 4.4 TB/s; summing with fp32 multiply-adds, the query
// re-read from LDS for every token and every head's partial sums exchanged
// across lanes, took 187 us.
#include <algorithm>

#include "common.hpp"
#include "grid.hpp"
#include "launch.hpp"

namespace is {

constexpr int kConsThreads = 256;
constexpr int kConsWaves = kConsThreads / kWave;
constexpr int kConsMaxQ = 8192;     // Hq * D query elements
constexpr int kConsMaxG = 8;        // query heads per KV head
constexpr int kConsMaxTokens = 512; // tokens of a block mapped at a time
// Blocks per CU aimed at, and query parts a block may keep in shared memory
// (always at least one KV head's, 24 KiB at most) so that as many are resident:
// 32 requests of 1,280-2,560 tokens, 32 / 8 heads of 128: 8 heads (24 KiB) and
// 4 / 3 blocks per CU 47 / 35.5 us, 4 heads (12 KiB) and 3 / 4 / 5 / 8 blocks
// 36.7 / 33.5 / 40.5 / 35.7 us.
constexpr int kConsBlocksPerCu = 4;
constexpr int kConsQBytes = 13 << 10;
constexpr int kConsMaxHeads = kConsQBytes / (16 * 6);  // query heads of a block (D = 16)
static_assert(kConsMaxHeads >= kConsMaxG, "one KV head's query heads");

typedef __bf16 bf16x8_c __attribute__((ext_vector_type(8)));
typedef float f32x4_c __attribute__((ext_vector_type(4)));

// Keys are read once per call (a decode step returns to a layer after all the
// others): non-temporal loads, 30.5 against 33.5 us on the shape above.
__device__ __forceinline__ uint4 load_key(const uint4* p) {
    typedef uint32_t u32x4_nt __attribute__((ext_vector_type(4)));
    const u32x4_nt x = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt*>(p));
    return make_uint4(x.x, x.y, x.z, x.w);
}

struct ConsShared {
    int64_t slot[kConsMaxTokens];  // slot of each token of the block, -1: skipped
    float cs[IS_MAX_HEAD_DIM / 2], sn[IS_MAX_HEAD_DIM / 2];
    int32_t tiny[kConsMaxHeads];  // a query head's split may be cut short
    uint32_t flags;
    int32_t any_bad, any_tiny;
};

// A pair of query elements rotated by its angle.
__device__ __forceinline__ float2 rotate_pair(uint16_t e0, uint16_t e1, float cs, float sn) {
    const float x0 = __uint_as_float((uint32_t)e0 << 16), x1 = __uint_as_float((uint32_t)e1 << 16);
    return make_float2(fmaf(x0, cs, -(x1 * sn)), fmaf(x1, cs, x0 * sn));
}

// DC: head elements per step (min(D, 128)); RT: 4-head tiles (G <= 4 RT); WALK: a
// block's tokens may be more than are mapped at a time (the loop over them costs
// 20 registers, and those a fifth of the speed at 64 / 8 heads of 128).
template <int DC, int RT, bool WALK>
__global__ __launch_bounds__(kConsThreads) void paged_scores_kernel(
    const uint16_t* __restrict__ q, const int32_t* __restrict__ qpos,
    const uint4* __restrict__ paged_k, int32_t layer, const int32_t* __restrict__ block_table,
    int32_t page_size, int32_t start_pos, const int32_t* __restrict__ m_dev,
    float* __restrict__ scores, int32_t Hq, int32_t H, int32_t D, int64_t num_slots,
    int32_t max_blocks, int32_t max_tokens, float rope_theta, const double* __restrict__ inv_freq,
    int32_t interleaved, TokenRule rule, int32_t block_heads,
    uint32_t* __restrict__ status) {
    constexpr int KS = DC >= 32 ? DC / 32 : 1;   // matrix ops per step
    constexpr int UPL = DC / 8;                  // 16-byte units of a token's row per step
    constexpr int RPL = kWave / UPL;             // rows per load
    constexpr int NL = RPL >= 16 ? 1 : 16 / RPL; // loads per step
    constexpr int SH = UPL >= 16 ? 0 : (UPL == 8 ? 1 : (UPL == 4 ? 2 : 3));
    extern __shared__ __align__(16) uint16_t s_qp[];  // [3][block heads * G][D] query parts
    __shared__ ConsShared sh;
    __shared__ uint4 s_k[kConsWaves][16 * UPL];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = blockIdx.y;
    const int m = min(m_dev[r], max_tokens);
    // the block's tokens, [first, last)
    const TokenShare share = token_share(m, blockIdx.x, rule);
    if (share.first >= share.last) return;
    const int h0 = blockIdx.z * block_heads;
    const int nh = min(block_heads, H - h0);
    const int G = Hq / H;
    const int half = D >> 1;

    // ---- slots of the block's tokens; sine and cosine of every pair ----
    if (t == 0) { sh.flags = 0; sh.any_bad = 0; sh.any_tiny = 0; }
    for (int i = t; i < nh * G; i += kConsThreads) sh.tiny[i] = 0;
    const int32_t* btr = block_table + (int64_t)r * max_blocks;
    const uint16_t* qr = q + ((int64_t)r * Hq + h0 * G) * D;
    const int nqe = nh * G * D;
    const int nch = DC < 128 ? 1 : D / DC;
    const int upr = (H * D) >> 3;
    const uint4* kl = paged_k + (int64_t)layer * num_slots * upr;
    const int lrow = lane / UPL, lu = lane % UPL;
    const int kg = lane >> 4, col = lane & 15;
    float* out = scores + ((int64_t)r * Hq + h0 * G) * max_tokens;
    uint4* sk = s_k[wave];
    for (int64_t tok = share.first; tok < share.last; tok += kConsMaxTokens) {
        const int tok0 = (int)tok;
        const int ntok = min(kConsMaxTokens, share.last - tok0);
        const bool start = !WALK || tok0 == share.first;
        __syncthreads();
        uint32_t flags = 0;
        for (int i = t; i < ntok; i += kConsThreads) {
            const int64_t pos = (int64_t)start_pos + tok0 + i;
            const int64_t blk = pos / page_size;
            int64_t slot = -1;
            if (blk >= max_blocks) {
                flags |= IS_DEV_BT_SHORT;
            } else {
                const int32_t b = btr[blk];
                slot = (int64_t)b * page_size + pos % page_size;
                if (b < 0) { flags |= IS_DEV_BAD_BLOCK; slot = -1; }
                else if (slot >= num_slots) { flags |= IS_DEV_SLOT_RANGE; slot = -1; }
            }
            sh.slot[i] = slot;
        }
        if (flags) { atomicOr(&sh.flags, flags); sh.any_bad = 1; }
        if (start && t < half) {
            const double w = inv_freq ? inv_freq[t]
                                      : exp2(-(2.0 * (double)t / (double)D) * log2((double)rope_theta));
            const double a = (double)qpos[r] * w;
            const double nrev = rint(a * 0.15915494309189535);
            double red = fma(-nrev, 6.283185307179586, a);
            red = fma(-nrev, 2.4492935982947064e-16, red);
            float sn, cs;
            sincosf((float)red, &sn, &cs);
            sh.cs[t] = cs;
            sh.sn[t] = sn;
        }
        __syncthreads();
        const bool any_bad = sh.any_bad != 0;

        // ---- the wave's steps: (head, 16 tokens) items wave, wave + 4, ..., each
        // in D / DC steps ----
        const int groups = (ntok + 15) >> 4;
        const int items = nh * groups;
        auto load = [&](int item, int c, uint4 (&v)[NL]) {
            if (item >= items) return;
            const int h = item / groups, g = item - h * groups;
            const uint4* src = kl + (int64_t)(h0 + h) * (D >> 3) + c * UPL + lu;
            // (rows past the last token read the last one's key again)
            if (!any_bad) {
#pragma unroll
                for (int j = 0; j < NL; ++j) {
                    const int64_t s = sh.slot[min(g * 16 + (j * RPL + lrow) % 16, ntok - 1)];
                    v[j] = load_key(src + s * upr);
                }
            } else {
#pragma unroll
                for (int j = 0; j < NL; ++j) {
                    const int64_t s = sh.slot[min(g * 16 + (j * RPL + lrow) % 16, ntok - 1)];
                    v[j] = s >= 0 ? load_key(src + s * upr) : make_uint4(0, 0, 0, 0);
                }
            }
        };
        uint4 kv[NL];
        load(wave, 0, kv);

        // ---- the query heads, rotated and split ----
        for (int i = start ? t : nh * G * half; i < nh * G * half; i += kConsThreads) {
            const int hq = i / half, j = i - hq * half;
            const int i0 = hq * D + (interleaved ? 2 * j : j);
            const int i1 = hq * D + (interleaved ? 2 * j + 1 : j + half);
            const float2 y = rotate_pair(qr[i0], qr[i1], sh.cs[j], sh.sn[j]);
            float y0 = y.x, y1 = y.y;
            if ((y0 != 0.f && fabsf(y0) < 0x1p-100f) || (y1 != 0.f && fabsf(y1) < 0x1p-100f))
                sh.tiny[hq] = sh.any_tiny = 1;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const uint32_t w = pack_bf16x2(y0, y1);
                s_qp[p * nqe + i0] = (uint16_t)w;
                s_qp[p * nqe + i1] = (uint16_t)(w >> 16);
                y0 -= bf16_lo(w);
                y1 -= bf16_hi(w);
            }
        }
        __syncthreads();

        const bool any_tiny = sh.any_tiny != 0;

        // matrix row 4 g' + p of tile rt: part p of query head 4 rt + g' (p = 3
        // and heads past G: zero)
        uint4 fa[RT][KS];
        int have = -1;
        for (int item = wave; item < items; item += kConsWaves) {
            const int h = item / groups, g = item - h * groups;
            f32x4_c acc[RT], done[RT];  // (done: the steps before, each summed from zero)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt] = done[rt] = f32x4_c{};
            for (int c = 0; c < nch; ++c) {
                if (c > 0) {
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) {
                        done[rt] += acc[rt];
                        acc[rt] = f32x4_c{};
                    }
                }
#pragma unroll
                for (int j = 0; j < NL; ++j) {
                    const int row = j * RPL + lrow;
                    if (RPL <= 16 || row < 16) sk[row * UPL + (lu ^ ((row >> SH) & (UPL - 1)))] = kv[j];
                }
                if (c + 1 < nch) load(item, c + 1, kv);
                else load(item + kConsWaves, 0, kv);
                __builtin_amdgcn_sched_barrier(0);
                wave_lds_sync();
                if (have != h * nch + c) {
                    have = h * nch + c;
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            const int gq = 4 * rt + (col >> 2), p = col & 3;
                            const int e = c * DC + ks * 32 + kg * 8;
                            fa[rt][ks] = (gq < G && p < 3 && ks * 32 + kg * 8 < DC)
                                             ? *(const uint4*)(s_qp + p * nqe + (h * G + gq) * D + e)
                                             : make_uint4(0, 0, 0, 0);
                        }
                }
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const int u = ks * 4 + kg;
                    const uint4 fb = u < UPL ? sk[col * UPL + (u ^ ((col >> SH) & (UPL - 1)))]
                                             : make_uint4(0, 0, 0, 0);
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8_c, fa[rt][ks]), __builtin_bit_cast(bf16x8_c, fb),
                            acc[rt], 0, 0, 0);
                }
                wave_lds_sync();
            }
            // lane: query head 4 rt + lane / 16, token lane % 16, its three parts
            const int i = g * 16 + col;
            const int64_t slot = i < ntok ? sh.slot[i] : -1;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int gq = 4 * rt + kg;
                if (gq >= G || slot < 0) continue;
                const f32x4_c sum = DC < 128 ? acc[rt] : done[rt] + acc[rt];
                float s = (sum[2] + sum[1]) + sum[0];
                if (!(fabsf(s) <= 3.402823466e38f) || (any_tiny && sh.tiny[h * G + gq])) {
                    const uint16_t* kr = (const uint16_t*)(kl + slot * upr) + (int64_t)(h0 + h) * D;
                    const uint16_t* qh = qr + (h * G + gq) * D;
                    double s64 = 0.0;
                    for (int j = 0; j < half; ++j) {
                        const int e0 = interleaved ? 2 * j : j, e1 = interleaved ? 2 * j + 1 : j + half;
                        const float2 y = rotate_pair(qh[e0], qh[e1], sh.cs[j], sh.sn[j]);
                        s64 = fma((double)y.x, (double)__uint_as_float((uint32_t)kr[e0] << 16), s64);
                        s64 = fma((double)y.y, (double)__uint_as_float((uint32_t)kr[e1] << 16), s64);
                    }
                    s = (float)s64;
                }
                out[(int64_t)(h * G + gq) * max_tokens + tok0 + i] = s;
            }
        }
        if (!WALK) break;
    }
    if (t == 0 && sh.flags && status) atomicOr(status, sh.flags);
}

int consumer_max_q_elems() { return kConsMaxQ; }
int consumer_max_group() { return kConsMaxG; }

hipError_t launch_paged_scores(const void* q, const int32_t* qpos, const void* paged_k,
                               int32_t layer, const int32_t* block_table, int32_t page_size,
                               int32_t start_pos, const int32_t* m, float* scores, int32_t nq,
                               int32_t Hq, int32_t H, int32_t D, int64_t num_slots,
                               int32_t max_blocks, int32_t max_tokens, float rope_theta,
                               const double* inv_freq, int32_t interleaved, uint32_t* status,
                               hipStream_t st) {
    if (max_tokens == 0) return hipSuccess;
    const int64_t cus = compute_units();
    const int G = Hq / H;
    // as many heads of a token in one block as fit while that gives two blocks
    // per CU; with fewer tokens the heads are shared out, down to one per wave.
    // What is placed is not known here and may be far below max_tokens: 512
    // tokens a request are reckoned with (4 requests of 100 tokens in buffers for
    // 4,096, 32 heads of 32 and 128: 10.7 and 11.5 us by max_tokens, 6.3 and 8.3)
    int heads = std::max(1, std::min<int>(H, kConsQBytes / (G * D * 6)));
    const int64_t groups = std::min<int64_t>(32, token_groups(max_tokens));
    while (heads > kConsWaves && nq * groups * ((H + heads - 1) / heads) < 2 * cus)
        heads = std::max(kConsWaves, (heads + 1) / 2);
    const int shares = (H + heads - 1) / heads;
    const TokenRule rule = token_rule(max_tokens, (int64_t)nq * shares,
                                      (int)(kConsBlocksPerCu * cus), kConsMaxTokens / 16);
    dim3 grid(rule.blocks, (unsigned)nq, (unsigned)shares);
    const size_t lds = (size_t)heads * G * D * 6;
    const bool walk = rule.most > kConsMaxTokens / 16;
#define IS_SCORES_W(DC, RT, WALK)                                                                \
    hipLaunchKernelGGL((paged_scores_kernel<DC, RT, WALK>), grid, dim3(kConsThreads), lds,  \
                       st,                                                                       \
                       (const uint16_t*)q, qpos, (const uint4*)paged_k, layer, block_table,      \
                       page_size, start_pos, m, scores, Hq, H, D, num_slots, max_blocks,         \
                       max_tokens, rope_theta, inv_freq, interleaved, rule, heads, status)
#define IS_SCORES(DC, RT)                     \
    do {                                      \
        if (walk) IS_SCORES_W(DC, RT, true);  \
        else IS_SCORES_W(DC, RT, false);      \
    } while (0)
#define IS_SCORES_G(DC)            \
    do {                           \
        if (G <= 4) IS_SCORES(DC, 1); \
        else IS_SCORES(DC, 2);     \
    } while (0)
    if (D == 16) IS_SCORES_G(16);
    else if (D == 32) IS_SCORES_G(32);
    else if (D == 64) IS_SCORES_G(64);
    else IS_SCORES_G(128);
#undef IS_SCORES_G
#undef IS_SCORES
#undef IS_SCORES_W
    return hipGetLastError();
}

}  // namespace is
