// Prefill-time token selection (paper Section 3, "KV Pruning": keep s < n
// tokens chosen at prefill; the paper uses an attention-score method from the
// literature with the most recent tokens retained, Section 4 / Appendix B).
// The rule implemented is stated in kvqp.h at kvqp_compress:
//   votes  = column sums, over the W window rows of all query heads of a KV
//            head's group, of the causal Softmax(sm_scale q k^T) rows;
//   pooled = 1-D max-pool of the votes over the prefix;
//   keep   = the n_kept highest pooled scores, ties to the lower position,
//            listed in ascending position.
//
// Kernels.  The score matrix is a dense [Gq*W x D] x [D x L] contraction per
// KV head, so it runs on the matrix cores (v_mfma_f32_16x16x32_f16, binary32
// accumulation); everything after it is a bandwidth- or latency-bound sweep.
//   score_pass<STATS>  a reference and the exp-sum of every window row (pass 1)
//   stats_combine      merges the row statistics of the workgroups (where there are many: few are merged by the vote pass)
//   score_pass<VOTES>  recomputes the tiles, normalises, sums columns (pass 2)
//   pool_scores        max-pool the votes, count the pooled scores in bins
//   select_topk        find the cut, ordered compaction; scores within a relative
//                      2e-5 of the cut are first re-scored in binary64 so that
//                      binary32 rounding cannot move the cut
// score_pass (up to 128 window rows) and score_wide (more rows): keys stream through LDS once per
// pass in chunks of 64 shared by the four waves of a workgroup; query rows stay in registers as
// MFMA operands.
#include <algorithm>
#include <type_traits>

#include "kvqp_internal.h"

namespace kvqp {
namespace {

typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef uint32_t u4any __attribute__((ext_vector_type(4), aligned(2)));      // ... at any binary16 number's address
union Frag {
    h8v v;
    uint4 q;
    u4v u;
};

template <bool B> struct BoolC { static constexpr bool value = B; };
template <int I> struct IntC { static constexpr int value = I; };

constexpr int kThreads = 256;
constexpr int kRowsPerWave = 32;        // score_pass: query rows one wave owns (its MFMA A operands, register-resident)
constexpr int kNarrowRows = 4 * kRowsPerWave;   // window rows of a KV head it takes; more are score_wide's
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;
constexpr float kLazySum = 256.0f;      // a row's reference moves only when the exponentials of a lane's tiles add up to more, so no score is further than 2^8 above it (an exponential's argument is rounded at its own magnitude: here to 2^-22, with references moved at 2^60 to 2^-19)

// The chip's memory-side cache.  The vote pass and the quantizer read keys again: the statistics stream the keys of all but the
// last heads past this cache, whose keys fill it, and the vote pass, which streams, leaves them there for the quantizer.  256
// heads of 32768 keys (2.15 GB), us, statistics + votes + quantizer: all keys through the cache 409 + 370 + 452, none
// 349 + 396 + 506 (what the quantizer has written leaves the cache while it runs), the last 128 MB 393 + 386 + 489, 192 MB
// 405 + 384 + 463, 256 MB 394 + 363 + 452, 448 MB 412 + 367 + 451.  Keys that fit: 8 heads of 32768, votes 15.1 instead of 17.8.
constexpr size_t kSideCache = (size_t)256 << 20;

enum { PASS_STATS = 0, PASS_VOTES = 1 };

struct ScoreArgs {
    const uint16_t* q_obs;  // [B, Hq, W, D]
    const uint16_t* k;      // [B, Hkv, L, D]
    float2* stats_part;     // [heads, n_parts, rows_pad]  (m, Z) in the log2 domain
    float2* stats;          // [heads, rows_pad]           (m, 1/Z)
    double* zsum;           // [heads, rows_pad]           Z
    float* vote;            // [heads, P]
    int L, W, P, gq, n_q_heads, n_kv_heads;
    int rows, rows_pad;     // Gq*W and the rows the waves cover (a multiple of 32 or 64)
    int chunks_per_wg, n_chunks, n_parts;
    int stream_heads;       // STATS: heads below it are streamed past the memory-side cache
    float scale_log2;       // sm_scale * log2(e)
};

// Token counts of the heads, from the host, that the statistics store beside their own work: nothing before the pooling reads
// them, and a launch of its own for them, ahead of everything, costs 1.5 us (whole calls, 32 heads of 20011 tokens, 99.75 -> 98.3; the
// one of other calls does not carry the kilobyte).
struct HeadCounts { int32_t* dst; int32_t v[kCountsInStats]; };
struct NoCounts {};
__device__ __forceinline__ void store_head_count(const HeadCounts& c, int head) {
    if (blockIdx.x == 0 && threadIdx.x == 0) c.dst[head] = c.v[head];
}
__device__ __forceinline__ void store_head_count(const NoCounts&, int) {}

// Up to so many statistics per row the vote pass merges itself while its first keys are on their way, without the launch of
// stats_combine before it: whole calls, us, 8 heads of 2000 keys (16 of them) 26.5 -> 24.9, of 4096 (32) 28.2 -> 26.1, 32 heads of 8192
// (16) 64.5 -> 63.0, 256 heads of 32768 (8) 1276 -> 1261.  More of them take as long as the launch: 8 heads of 32768 (64) 75.3 -> 76.0.
constexpr int kMergeParts = 32;
constexpr int kChunk = 64;              // keys of a chunk
constexpr int kChunkBytes = kChunk * kHeadDim * 2;
constexpr int kPlaces = 2;              // chunks in LDS: the one being computed and the one on its way (place ^ 1 is the other)

// Request 1 KB of a chunk (four key rows) straight into LDS: lane l's 16 bytes from `base + off` land at dst + 16 l.
// Nothing is left in a register, so the only thing to wait for is the counter (arrived()).  The statement overwrites m0, a reserved register
// that a clobber list cannot name: the compiler sets it right before an instruction of its own that reads it, and has none in these kernels.
template <bool STREAM>
__device__ __forceinline__ void request_rows(uint32_t dst, uint32_t off, const void* base) {
    if (STREAM) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(dst), "v"(off), "s"(base) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(base) : "memory");
}
// Wait until this wave's memory and LDS operations are done; BARRIER: meet the other waves.
template <bool BARRIER>
__device__ __forceinline__ void arrived() {
    if (BARRIER) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

// Request a chunk.  Its rows lie unpadded in LDS; the 16-byte piece p of row r is stored at place p ^ (r % 16), so that
// the operand reads meet every bank equally.  Wave w requests rows 16 w .. 16 w + 15.
// DIRECT: keys at multiples of 16 bytes.  Others (no form of the requests is documented for them) pass through registers to the same places.
constexpr int kLoads = 4;               // requests of a wave per chunk
template <int PASS, bool DIRECT>
__device__ __forceinline__ void request_chunk(const ScoreArgs& a, int head, const void* kh, unsigned char* sk, int chunk, int place) {
    const uint32_t sk_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)sk;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kb = lane >> 4;
    auto from = [&](int i) {
        const int key = min(chunk * kChunk + 16 * wave + 4 * i + kb, a.L - 1);      // rows past the end are masked
        return (uint32_t)key * (2u * kHeadDim) + 16u * (uint32_t)(n ^ ((4 * i + kb) & 15));
    };
    auto to = [&](int i) { return place * kChunkBytes + (16 * wave + 4 * i) * (2 * kHeadDim); };
    if constexpr (!DIRECT) {
        u4v v[kLoads];
#pragma unroll
        for (int i = 0; i < kLoads; ++i) v[i] = *reinterpret_cast<const u4any*>(static_cast<const char*>(kh) + from(i));
#pragma unroll
        for (int i = 0; i < kLoads; ++i) *reinterpret_cast<u4v*>(sk + to(i) + 16 * lane) = v[i];
        return;
    }
    auto rows = [&](auto stream) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) request_rows<decltype(stream)::value>(sk_at + to(i), from(i), kh);
    };
    if (PASS == PASS_VOTES || head < a.stream_heads) rows(BoolC<true>{});
    else rows(BoolC<false>{});
}

// Up to 128 window rows.  The four waves are NRW row slabs x KS key strips.  What bounds a pass is memory (K once per
// pass) as long as requests stay in flight while a chunk is computed.  So chunks go from memory into LDS without
// passing through registers, two places deep, and the waves meet once per chunk: behind that barrier the chunk has
// arrived for all of them and the place of the one before it is free for the next request.  A wave forms all its
// scores of a chunk before it uses any (sixteen independent matrix chains), and the one rare branch of the
// statistics stands per chunk.  The statistics take keys as the first operand, so that a lane's scores belong to one row
// (one reference and one sum to keep, two lane exchanges at the end); the votes take queries first: a key's rows are added up
// in the lane, and two exchanges per chunk merge its four tiles.  Before (chunks through registers, two
// barriers per chunk, a branch per 16 keys) -> now, us, statistics + votes: 8 heads of 4096 keys 10.0 + 7.2 -> 6.5 + 5.2,
// 8 of 32768 23.2 + 19.2 -> 18.3 + 15.1, 32 of 16384 37 + 34 -> 29 + 26, 256 of 32768 425 + 414 -> 394 + 363 (2.15 GB:
// 5.5 and 5.9 TB/s), 32 of 20011 with 32 rows 32.6 + 25.4 -> 31.6 + 24.6.  Three and four places in LDS are slower
// (8 heads of 32768: 19.2 + 15.9 and 20.2 + 17.0; not explained: two workgroups per CU, which is all the launch has, still fit).
// MERGE (VOTES): the pass merges the row statistics itself.
template <int NRW, int PASS, bool MERGE = false, bool DIRECT = true, class Counts = NoCounts>
__global__ __launch_bounds__(kThreads, 4) void score_pass(const ScoreArgs a, const Counts counts) {
    constexpr int kMT = kRowsPerWave / 16;
    constexpr int KS = 4 / NRW, KT = 4 / KS;          // key strips; 16-key tiles of a wave per chunk
    constexpr bool SHARED = NRW > 1;                  // a wave reads keys that other waves have requested
    __shared__ __align__(16) unsigned char sk[kPlaces * kChunkBytes];
    __shared__ float svote[(PASS == PASS_VOTES && NRW > 1) ? 2 * NRW * kChunk : 1];

    const int head = blockIdx.y;
    const int b = head / a.n_kv_heads, g = head % a.n_kv_heads;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar: tile positions stay uniform
    const int n = lane & 15, kb = lane >> 4;
    const int rw = wave % NRW, ks = wave / NRW;
    const uint16_t* kh = a.k + (size_t)head * a.L * kHeadDim;
    const int c_begin = blockIdx.x * a.chunks_per_wg;
    const int c_end = min(a.n_chunks, c_begin + a.chunks_per_wg);
    store_head_count(counts, head);

    // Query operand: rows 32*rw + 16*mt + (lane & 15), channels 32*s + 8*kb .. +8.
    Frag qf[kMT][4];
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) {
        const int r = kRowsPerWave * rw + 16 * mt + n;
        const bool live = r < a.rows;
        const int hl = live ? r / a.W : 0, i = live ? r % a.W : 0;
        const uint16_t* qp = a.q_obs + (((size_t)b * a.n_q_heads + g * a.gq + hl) * a.W + i) * kHeadDim + 8 * kb;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            qf[mt][s].q = live ? *reinterpret_cast<const uint4*>(qp + 32 * s) : make_uint4(0, 0, 0, 0);
        }
    }
    // STATS: a lane's scores belong to row 16 mt + n: reference (log2 domain) and sum of exp2(score - reference).
    // VOTES: to rows 16 mt + 4 kb + i: m and 1/Z.
    constexpr int NR = PASS == PASS_STATS ? 1 : 4;
    using Sum = std::conditional_t<PASS == PASS_STATS && (KS > 1), double, float>;
    float m_run[kMT][NR];
    Sum z_run[kMT][NR];
    auto request = [&](int chunk, int place) { request_chunk<PASS, DIRECT>(a, head, kh, sk, chunk, place); };
    // (the first chunk and the query rows arrive together; the compiler's wait for the latter stands here, not in the loop)
    auto settle = [&] {
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
            for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(qf[mt][s].u));
    };
    if constexpr (PASS == PASS_STATS) {
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt) { m_run[mt][0] = kNegBig; z_run[mt][0] = 0.f; }
        request(c_begin, 0);
        settle();
    } else if constexpr (MERGE) {
        // The two halves of the wave take every other part of the slab's 32 rows, all of them on their way at once.
        auto merge = [&](auto count) {
            constexpr int N = decltype(count)::value;
            const int half = lane >> 5, row = kRowsPerWave * rw + (lane & 31);
            const float2* p = a.stats_part + (size_t)head * a.n_parts * a.rows_pad + row;
            float2 v[N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                v[u] = p[(size_t)min(2 * u + half, a.n_parts - 1) * a.rows_pad];
                if (2 * u + half >= a.n_parts) v[u].y = 0.f;
            }
            request(c_begin, 0);
            settle();
            float M = v[0].x;
#pragma unroll
            for (int u = 1; u < N; ++u) M = fmaxf(M, v[u].x);
            M = fmaxf(M, __shfl_xor(M, 32));
            double Z = 0.0;
#pragma unroll
            for (int u = 0; u < N; ++u) Z += (double)v[u].y * (double)__builtin_amdgcn_exp2f(v[u].x - M);
            Z += __shfl_xor(Z, 32);
            const float inv = Z > 0.0 && row < a.rows ? (float)(1.0 / Z) : 0.f;
            if (blockIdx.x == 0 && ks == 0 && half == 0) {                // for the binary64 re-scoring
                a.stats[(size_t)head * a.rows_pad + row] = make_float2(M, inv);
                a.zsum[(size_t)head * a.rows_pad + row] = Z;
            }
#pragma unroll
            for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
                for (int i = 0; i < NR; ++i) {
                    m_run[mt][i] = __shfl(M, 16 * mt + 4 * kb + i);
                    z_run[mt][i] = __shfl(inv, 16 * mt + 4 * kb + i);
                }
        };
        if (a.n_parts <= 8) merge(IntC<4>{});
        else merge(IntC<kMergeParts / 2>{});
    } else {
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int r = kRowsPerWave * rw + 16 * mt + 4 * kb + i;
                const float2 st = a.stats[(size_t)head * a.rows_pad + r];
                m_run[mt][i] = st.x; z_run[mt][i] = (r < a.rows) ? st.y : 0.f;
            }
        request(c_begin, 0);
        settle();
    }
    if (PASS == PASS_VOTES)
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
            for (int i = 0; i < NR; ++i) asm volatile("" : "+v"(m_run[mt][i]), "+v"(z_run[mt][i]));

    const uint32_t kp0 = (uint32_t)(n * 2 * kHeadDim + ((kb ^ n) << 4));  // contraction step 0 of key n; step s: ^ (s << 6)
    int place = 0;
    auto store_votes = [&](int chunk) {               // the chunk's votes over all slabs (one wave's work)
        float v = 0.f;
#pragma unroll
        for (int r = 0; r < NRW; ++r) v += svote[((chunk & 1) * NRW + r) * kChunk + lane];
        const int key = chunk * kChunk + lane;
        if (key < a.P) a.vote[(size_t)head * a.P + key] = v;
    };
    for (int chunk = c_begin; chunk < c_end; ++chunk) {
        // this chunk has arrived, every wave is done with the one before it
        arrived<SHARED>();
        if (chunk + 1 < c_end) request(chunk + 1, place ^ 1);
        if (PASS == PASS_VOTES && NRW > 1)
            if (chunk > c_begin && wave == (chunk & 3)) store_votes(chunk - 1);

        const unsigned char* kp = sk + place * kChunkBytes + 16 * KT * ks * (2 * kHeadDim);
        f4v acc[KT][kMT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            Frag kf[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) kf[s].q = *reinterpret_cast<const uint4*>(kp + 16 * kt * (2 * kHeadDim) + (kp0 ^ (s << 6)));
#pragma unroll
            for (int mt = 0; mt < kMT; ++mt) {
                f4v c = (f4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    c = PASS == PASS_STATS ? __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[s].v, qf[mt][s].v, c, 0, 0, 0)
                                           : __builtin_amdgcn_mfma_f32_16x16x32_f16(qf[mt][s].v, kf[s].v, c, 0, 0, 0);
                acc[kt][mt] = c;
            }
        }
        float col[KT];
        if constexpr (PASS == PASS_STATS) {
            // causal mask only where the chunk reaches the window (raw scores; the scale is positive)
            if ((chunk + 1) * kChunk > a.P) {
                int w = a.W;
                asm volatile("" : "+s"(w));   // keeps the window positions out of the loop's live registers
#pragma unroll
                for (int mt = 0; mt < kMT; ++mt) {
                    const int r = kRowsPerWave * rw + 16 * mt + n;
                    const int last = min(a.P + (r < a.rows ? r % w : -1), a.L - 1) - (chunk * kChunk + 16 * KT * ks + 4 * kb);   // padding rows see the prefix only
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (16 * kt + i > last) acc[kt][mt][i] = -INFINITY;
                }
            }
            // m_run is a reference, not the exact maximum: it moves only when a score beats it by
            // 2^8 or several come near (the sum of the chunk's exponentials tells), so the common path
            // is one fused multiply-add, one exp2 and one add
            float t[kMT];
            auto sums = [&] {
#pragma unroll
                for (int mt = 0; mt < kMT; ++mt) {
                    float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[kt][mt][i], a.scale_log2, -m_run[mt][0]));
                            x[i] = kt == 0 ? e : x[i] + e;
                        }
                    t[mt] = (x[0] + x[1]) + (x[2] + x[3]);
                }
            };
            // (the first chunk always moves it)
            const bool first = chunk == c_begin;
            if (!first) sums();
            if (first || __builtin_amdgcn_ballot_w64(fmaxf(t[0], t[1]) > kLazySum) != 0ull) {   // rare after the first chunks
#pragma unroll
                for (int mt = 0; mt < kMT; ++mt) {
                    float top = acc[0][mt][0];
#pragma unroll
                    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                        for (int i = 0; i < 4; ++i) top = fmaxf(top, acc[kt][mt][i]);
                    top *= a.scale_log2;
                    if (top > m_run[mt][0]) {
                        z_run[mt][0] *= __builtin_amdgcn_exp2f(m_run[mt][0] - top);
                        m_run[mt][0] = top;
                    }
                }
                sums();
            }
#pragma unroll
            for (int mt = 0; mt < kMT; ++mt) z_run[mt][0] += t[mt];
        } else {
            // normalised probabilities summed over this lane's rows, per key (the window's own keys get votes nobody reads)
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                float c0 = 0.f, c1 = 0.f;
#pragma unroll
                for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; i += 2) {
                        c0 = __builtin_fmaf(__builtin_amdgcn_exp2f(__builtin_fmaf(acc[kt][mt][i], a.scale_log2, -m_run[mt][i])),
                                            z_run[mt][i], c0);
                        c1 = __builtin_fmaf(__builtin_amdgcn_exp2f(__builtin_fmaf(acc[kt][mt][i + 1], a.scale_log2, -m_run[mt][i + 1])),
                                            z_run[mt][i + 1], c1);
                    }
                col[kt] = c0 + c1;
            }
        }
        if constexpr (PASS == PASS_VOTES) {
            // sum over the four rows of 16 lanes; an exchange merges two tiles into one register
            auto swap16 = [](float x, float y) {
                const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
                return __uint_as_float(s[0]) + __uint_as_float(s[1]);
            };
            auto swap32 = [](float x, float y) {
                const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
                return __uint_as_float(s[0]) + __uint_as_float(s[1]);
            };
            if constexpr (KT == 4) {          // row q of lanes: tile q
                svote[((chunk & 1) * NRW + rw) * kChunk + lane] = swap32(swap16(col[0], col[1]), swap16(col[2], col[3]));
            } else if constexpr (KT == 2) {   // rows 0 and 1: tiles 0 and 1; rows 2 and 3 the same again
                const float x = swap16(col[0], col[1]), v = swap32(x, x);
                if (lane < 32) svote[((chunk & 1) * NRW + rw) * kChunk + 32 * ks + lane] = v;
            } else {
                const float x = swap16(col[0], col[0]), v = swap32(x, x);
                const int key = chunk * kChunk + 16 * ks + n;
                if (kb == 0 && key < a.P) a.vote[(size_t)head * a.P + key] = v;
            }
        }
        place ^= 1;
    }
    if (PASS == PASS_VOTES && NRW > 1) {
        arrived<SHARED>();
        if (wave == 0) store_votes(c_end - 1);
    }

    if (PASS == PASS_STATS) {
        if constexpr (KS > 1) {
            // The four lanes of every key strip that share a row meet in LDS, and one thread per row adds their sums, which are
            // binary64 since the chunk, and stores the total: rounded once, however many strips and chunks the workgroup has.  Row sums of
            // 64 heads of 8192 keys, 32 rows, against 64 bits, rms: every strip on its own 1.72e-8, strips added in binary32
            // 2.23e-8, this 1.64e-8; whole calls as long as with binary32 (8 heads of 4096 keys 22.9 us, 64 of 8192 80.3).
            constexpr int ROWS = NRW * kRowsPerWave;
            double* s_z = reinterpret_cast<double*>(sk);                 // [strip][lane of the row][row]
            float* s_m = reinterpret_cast<float*>(s_z + 4 * KS * ROWS);
            static_assert(4 * KS * ROWS * (sizeof(double) + sizeof(float)) <= sizeof(sk), "the sums fit the keys' place");
            __syncthreads();                                             // (every wave is done with its keys)
#pragma unroll
            for (int mt = 0; mt < kMT; ++mt) {
                const int at = (4 * ks + kb) * ROWS + kRowsPerWave * rw + 16 * mt + n;
                s_m[at] = m_run[mt][0]; s_z[at] = z_run[mt][0];
            }
            __syncthreads();
            if ((int)threadIdx.x < ROWS) {
                float m_of[4 * KS], m = kNegBig;
                double z = 0.0;
#pragma unroll
                for (int u = 0; u < 4 * KS; ++u) { m_of[u] = s_m[u * ROWS + threadIdx.x]; m = fmaxf(m, m_of[u]); }
#pragma unroll
                for (int u = 0; u < 4 * KS; ++u) z += s_z[u * ROWS + threadIdx.x] * (double)__builtin_amdgcn_exp2f(m_of[u] - m);
                a.stats_part[((size_t)head * a.n_parts + blockIdx.x) * a.rows_pad + threadIdx.x] = make_float2(m, (float)z);
            }
        } else {
            // merge the four lanes that share a row
#pragma unroll
            for (int mt = 0; mt < kMT; ++mt) {
                float m = m_run[mt][0], z = z_run[mt][0];
#pragma unroll
                for (int off = 16; off < 64; off <<= 1) {
                    const float mo = __shfl_xor(m, off), zo = __shfl_xor(z, off);
                    const float mn = fmaxf(m, mo);
                    z = z * __builtin_amdgcn_exp2f(m - mn) + zo * __builtin_amdgcn_exp2f(mo - mn);
                    m = mn;
                }
                if (kb == 0) a.stats_part[((size_t)head * a.n_parts + blockIdx.x) * a.rows_pad + kRowsPerWave * rw + 16 * mt + n] = make_float2(m, z);
            }
        }
    }
}

// 129 to 256 window rows: four waves of 64 rows.  Here the matrix cores and the exponentials bound a pass: 67 us for the
// products of 8 heads, 131072 keys and 256 rows at the rate of a large matrix product, and the vector unit stands still for
// most of a 16x16x32 instruction (two of them with 8 fused multiply-adds and 4 exponentials: 33.9 ns, the latter
// alone 27.5; 8 multiply-adds 26.1 and 10.0).  One 32x32x16 instruction does the same work and lets more of it
// through (31.1 and 20.1 ns).  So tiles are 32 keys x 32 rows, and the product of a tile runs while the scores of the one
// before it are exponentiated, across chunks too: the waves meet when all have a chunk's last keys in registers.  Keys arrive as in
// score_pass.  131072 keys, 8 heads, 256 rows, us, statistics + votes: keys in registers, queries in LDS, 16x16x32, a
// reference moved by selects in every step: 95 + 83; score_pass with 64 rows per wave 94 + 78; 32x32x16 without the next tile's product
// 82 + 78; this 82 + 76.  (The matrix cores are busy for half of that; the clock falls to 1.8 GHz.  Three or four chunks in
// LDS 87 + 79 and 87 + 82; a fixed mixture of matrix and vector instructions 84 + 77.)  What the references cost where
// strong outlier channels make them move: 5 us; a moved reference is shared by the two lanes of a row.
typedef float f16v __attribute__((ext_vector_type(16)));
constexpr int kWideRows = 256;
template <int PASS, bool DIRECT = true, class Counts = NoCounts>
__global__ __launch_bounds__(kThreads, 2) void score_wide(const ScoreArgs a, const Counts counts) {
    constexpr int MT = 2;                             // row tiles of a wave
    constexpr int kWaveRows = 32 * MT;
    constexpr int kSteps = kHeadDim / 16;             // contraction steps
    __shared__ __align__(16) unsigned char sk[kPlaces * kChunkBytes];
    __shared__ float svote[PASS == PASS_VOTES ? 2 * 4 * kChunk : 1];

    const int head = blockIdx.y;
    const int b = head / a.n_kv_heads, g = head % a.n_kv_heads;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hi = lane >> 5;
    const uint16_t* kh = a.k + (size_t)head * a.L * kHeadDim;
    const int c_begin = blockIdx.x * a.chunks_per_wg;
    const int c_end = min(a.n_chunks, c_begin + a.chunks_per_wg);
    store_head_count(counts, head);

    // Query operand: row kWaveRows * wave + 32 * mt + n, channels 16 * s + 8 * hi .. +8.
    Frag qf[MT][kSteps];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int r = kWaveRows * wave + 32 * mt + n;
        const bool live = r < a.rows;
        const int hl = live ? r / a.W : 0, i = live ? r % a.W : 0;
        const uint16_t* qp = a.q_obs + (((size_t)b * a.n_q_heads + g * a.gq + hl) * a.W + i) * kHeadDim + 8 * hi;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            qf[mt][s].q = live ? *reinterpret_cast<const uint4*>(qp + 16 * s) : make_uint4(0, 0, 0, 0);
        }
    }
    // STATS: a lane's scores belong to row 32 mt + n.  VOTES: to rows 32 mt + 8 (i / 4) + 4 hi + i % 4.
    constexpr int NR = PASS == PASS_STATS ? 1 : 16;
    float m_run[MT][NR], z_run[MT][NR];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if (PASS == PASS_STATS) {
                m_run[mt][i] = kNegBig; z_run[mt][i] = 0.f;
            } else {
                const int r = kWaveRows * wave + 32 * mt + 8 * (i >> 2) + 4 * hi + (i & 3);
                const float2 st = a.stats[(size_t)head * a.rows_pad + r];
                m_run[mt][i] = st.x; z_run[mt][i] = (r < a.rows) ? st.y : 0.f;
            }
        }

    auto request = [&](int chunk, int place) { request_chunk<PASS, DIRECT>(a, head, kh, sk, chunk, place); };
    request(c_begin, 0);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s) asm volatile("" : "+v"(qf[mt][s].u));
        if (PASS == PASS_VOTES)
#pragma unroll
            for (int i = 0; i < NR; ++i) asm volatile("" : "+v"(m_run[mt][i]), "+v"(z_run[mt][i]));
    }

    const uint32_t kp0 = (uint32_t)(n * 2 * kHeadDim + ((hi ^ (n & 15)) << 4));  // contraction step 0 of key n; step s: ^ (s << 5)
    struct Tile { f16v f[MT]; };
    auto product = [&](Tile& acc, int place, int kt) {
        const unsigned char* kp = sk + place * kChunkBytes + 32 * kt * (2 * kHeadDim);
        Frag kf[kSteps];
#pragma unroll
        for (int s = 0; s < kSteps; ++s) kf[s].q = *reinterpret_cast<const uint4*>(kp + (kp0 ^ (s << 5)));
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc.f[mt][i] = 0.f;
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc.f[mt] = PASS == PASS_STATS ? __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[s].v, qf[mt][s].v, acc.f[mt], 0, 0, 0)
                                               : __builtin_amdgcn_mfma_f32_32x32x16_f16(qf[mt][s].v, kf[s].v, acc.f[mt], 0, 0, 0);
    };
    // STATS: the tile's scores enter the lane's sums
    auto sums = [&](const Tile& acc, float (&t)[MT]) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float x[4];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(acc.f[mt][i], a.scale_log2, -m_run[mt][0]));
                x[i & 3] = i < 4 ? e : x[i & 3] + e;
            }
            t[mt] = (x[0] + x[1]) + (x[2] + x[3]);
        }
    };
    // causal mask, only where the tile reaches the window
    auto mask = [&](Tile& acc, int tile0) {
        if (tile0 + 32 > a.P) {
            int w = a.W;
            asm volatile("" : "+s"(w));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int r = kWaveRows * wave + 32 * mt + n;
                const int last = min(a.P + (r < a.rows ? r % w : -1), a.L - 1) - (tile0 + 4 * hi);
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (8 * (i >> 2) + (i & 3) > last) acc.f[mt][i] = -INFINITY;
            }
        }
    };
    // (references move as in score_pass)
    auto count = [&](const Tile& acc, float (&t)[MT]) {
        float peak = t[0];
#pragma unroll
        for (int mt = 1; mt < MT; ++mt) peak = fmaxf(peak, t[mt]);
        if (__builtin_amdgcn_ballot_w64(peak > kLazySum) != 0ull) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                float top = acc.f[mt][0];
#pragma unroll
                for (int i = 1; i < 16; ++i) top = fmaxf(top, acc.f[mt][i]);
                top = fmaxf(top, __shfl_xor(top, 32)) * a.scale_log2;
                if (top > m_run[mt][0]) {
                    z_run[mt][0] *= __builtin_amdgcn_exp2f(m_run[mt][0] - top);
                    m_run[mt][0] = top;
                }
            }
            sums(acc, t);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) z_run[mt][0] += t[mt];
    };
    // VOTES: the key's probabilities summed over the lane's rows
    auto column = [&](const Tile& acc) {
        float c0 = 0.f, c1 = 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; i += 2) {
                c0 = __builtin_fmaf(__builtin_amdgcn_exp2f(__builtin_fmaf(acc.f[mt][i], a.scale_log2, -m_run[mt][i])),
                                    z_run[mt][i], c0);
                c1 = __builtin_fmaf(__builtin_amdgcn_exp2f(__builtin_fmaf(acc.f[mt][i + 1], a.scale_log2, -m_run[mt][i + 1])),
                                    z_run[mt][i + 1], c1);
            }
        return c0 + c1;
    };
    int place = 0;
    auto store_votes = [&](int chunk) {
        float v = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) v += svote[((chunk & 1) * 4 + r) * kChunk + lane];
        const int key = chunk * kChunk + lane;
        if (key < a.P) a.vote[(size_t)head * a.P + key] = v;
    };
    Tile even, odd;                              // scores of a chunk's two tiles
    arrived<true>();
    if (c_begin + 1 < c_end) request(c_begin + 1, 1);
    product(even, 0, 0);
    for (int chunk = c_begin; chunk < c_end; ++chunk) {
        float t[MT], col0, col1;
        if (PASS == PASS_STATS) mask(even, chunk * kChunk);
        __builtin_amdgcn_sched_barrier(0);
        product(odd, place, 1);
        if (PASS == PASS_STATS) sums(even, t); else col0 = column(even);
        if (PASS == PASS_STATS) count(even, t);
        arrived<true>();                       // the next chunk is there; every wave has this one in registers
        if (chunk + 2 < c_end) request(chunk + 2, place);
        if (PASS == PASS_VOTES)
            if (chunk > c_begin && wave == (chunk & 3)) store_votes(chunk - 1);
        place ^= 1;
        if (PASS == PASS_STATS) mask(odd, chunk * kChunk + 32);
        __builtin_amdgcn_sched_barrier(0);
        product(even, place, 0);               // (past the last chunk: not used)
        if (PASS == PASS_STATS) sums(odd, t); else col1 = column(odd);
        if (PASS == PASS_STATS) count(odd, t);
        if constexpr (PASS == PASS_VOTES) {   // halves of the wave: tiles 0 and 1
            const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(col0), __float_as_uint(col1), false, false);
            svote[((chunk & 1) * 4 + wave) * kChunk + lane] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
        }
    }
    if (PASS == PASS_VOTES) {
        arrived<true>();
        if (wave == 0) store_votes(c_end - 1);
    }
    if (PASS == PASS_STATS) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float m = m_run[mt][0], z = z_run[mt][0];
            const float mo = __shfl_xor(m, 32), zo = __shfl_xor(z, 32);
            const float mn = fmaxf(m, mo);
            z = z * __builtin_amdgcn_exp2f(m - mn) + zo * __builtin_amdgcn_exp2f(mo - mn);
            if (hi == 0) {
                const int r = kWaveRows * wave + 32 * mt + n;
                a.stats_part[((size_t)head * a.n_parts + blockIdx.x) * a.rows_pad + r] = make_float2(mn, z);
            }
        }
    }
}

// Merge the per-part row statistics; Z is accumulated in binary64.  One wave per row (four rows
// per workgroup): lanes stride over the parts, then a fixed-order butterfly.
__global__ __launch_bounds__(256) void stats_combine(const float2* __restrict__ part, float2* __restrict__ stats,
                                                     double* __restrict__ zsum, int n_parts, int rows_pad) {
    const int head = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int r = 4 * blockIdx.y + (threadIdx.x >> 6);
    if (r >= rows_pad) return;
    const float2* p = part + (size_t)head * n_parts * rows_pad + r;
    float M = kNegBig;
    for (int s = lane; s < n_parts; s += 64) M = fmaxf(M, p[(size_t)s * rows_pad].x);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    double Z = 0.0;
    for (int s = lane; s < n_parts; s += 64) {
        const float2 v = p[(size_t)s * rows_pad];
        Z += (double)v.y * (double)exp2f(v.x - M);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) Z += __shfl_xor(Z, off);
    if (lane == 0) {
        stats[(size_t)head * rows_pad + r] = make_float2(M, Z > 0.0 ? (float)(1.0 / Z) : 0.f);
        zsum[(size_t)head * rows_pad + r] = Z;
    }
}

// ---------------------------------------------------------------------------
// Selection: pool, find the cut, refine the candidates next to it in binary64,
// compact in position order.
//
// What bounds it is a chain of dependent waits (memory, LDS) on few
// workgroups and what one CU can issue, never bandwidth: a head's scores are at most half a megabyte.  The
// work is therefore cut so that the part that grows with the prefix is spread
// over many workgroups and the rest touches each score once:
//   pool_scores  several workgroups per head: max-pool the votes, store the upper 16
//                bits of each pooled score, and count the scores in 4032 bins of equal
//                bit-pattern width (64 per factor of two: at most 1.6 % wide) and the
//                bins' counts in groups of 64
//   select_topk  one workgroup per head, or several where a long prefix leaves CUs idle: the counts give the bin of the cut; ONE
//                sweep over the 16-bit codes leaves a mask bit per sure survivor and
//                collects the few candidates of that bin, whose scores are pooled
//                again and give the exact cut; survivors leave through the mask.
// Prefixes of up to three pooling tiles (4096) do both in the second kernel.  Measured on one CU with sixteen waves: an
// instruction of all of them 8 ns, of one wave 2, a barrier 12, a dependent access to LDS 31, an exchange of lanes through it 35 (by
// DPP 5), a branch that is taken 25, an access to memory 400 to 1000.  So the list around the cut is finished by one wave, one
// candidate per lane and unrolled (before, by all of them, with a barrier after every step), sums go along the lanes by DPP, only
// the counts of the cut's group are read besides the groups', and the sweep lists groups of eight codes instead of candidates.  select_topk, us, before ->
// now (averages over three prompts, a call at a time; one prompt and the next differ by up to 40 %, with the positions that are scored in 64 bits):
// 8 heads of 4064 candidates 9.4 -> 7.7, of 32736 19.4 -> 15.5, of 131008 41.6 -> 29.0 (sixteen workgroups per head), 32 of 20003 15.3 -> 13.3.
// ---------------------------------------------------------------------------
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kMaxPrefix = 131072;
constexpr int kMaxShares = kMaxPrefix / (8 * kSelThreads);   // workgroups of a head that sweep codes, one group of eight candidates per thread
constexpr int kPoolTile = 4 * kSelThreads;   // candidates of one pooling step, four consecutive ones per thread
constexpr int kMaxPoolRadius = 31;    // pool_kernel <= 63
constexpr int kStage = kPoolTile + 2 * kMaxPoolRadius + 2;   // votes of a step with the halo on either side (whole 16-byte pieces)
constexpr int kBinShift = 17;
constexpr int kGroups = 63, kGroupBins = 64;      // score bins in groups: one group per factor of two
constexpr int kBins = kGroups * kGroupBins;       // score bins: the bit pattern >> kBinShift, 2^-54 .. 2^9, clamped at both ends
constexpr int kBinRow = 4096;         // 16-bit words of a pooling workgroup's counts: the bins', then the groups', then (row 0 of a head) the arrivals of the sweeping workgroups
constexpr int kCodeShift = 15;        // the stored code of a score: its pattern's upper 16 bits below the sign
constexpr int kBinBase = ((136 << 23) >> kBinShift) - kBins;   // 2^9 is the first pattern past the last bin (votes stay below 256 rows)
constexpr int kOwnTiles = 3;          // prefixes of up to so many tiles select_topk pools itself; longer ones are pool_scores'
// Prefixes of up to so many shares (32768 candidates) are swept by one workgroup per head, longer ones by one per share, of
// heads that leave each a CU of its own.  One CU takes in about 25 bytes a nanosecond (2 bytes a candidate); the others' masks and
// groups cost a trip through memory, 3 us with the counter.  Whole calls, us, one workgroup -> several: 8 heads of 32736
// candidates 67.4 -> 67.1, of 65504 106.2 -> 102.6, of 131040 165.6 -> 157.7, 32 heads of 16352 95.6 -> 96.2, of 65504 297.1 -> 294.8,
// 128 heads of 32736 547.9 -> 559.0.
constexpr int kAloneShares = 4, kMostShares = 256;
constexpr int kMaxSegs = 16;          // pooling workgroups per head
constexpr int kMaxSegTiles = 15;      // (a workgroup's bin counts are stored in 16 bits)
constexpr int kListCap = 3840;        // candidates around the cut held in LDS; more are swept from memory
constexpr int kFew = 64;              // candidates around the cut that one wave finishes
constexpr int kDigit = 10;            // bits per pass of the radix select
constexpr int kMaxBand = 512;         // candidates re-scored per head; beyond that binary32 decides (and the caller is told)
constexpr int kVoteSlots = 2048;      // binary64 votes (distinct positions) held in LDS during the re-scoring
constexpr int kPartSlots = 1792;      // ... and partial votes of a batch of positions
constexpr float kBandRel = 2.0e-5f;   // >> the binary32 error of a vote (a few 1e-7 relative)

struct SelectArgs {
    const float* vote;      // [heads, P]
    uint16_t* code;         // [heads, p_stride] codes of the pooled scores, in groups of eight (codes_above)
    uint16_t* bins;         // [heads, n_seg, kBinRow] counts of every pooling workgroup
    float* exact;           // [heads, p_stride] pooled scores, only where the candidates around the cut don't fit the list; or NULL
    int32_t* idx;           // [heads, n_kept], in the workspace: the list that the quantizer reads
    int32_t* list;          // the caller's, written beside it and never read; or NULL
    int32_t* unrefined;     // [heads] or NULL: candidates near the cut that binary32 decided (0: all re-scored)
    const int32_t* head_n;  // a head's own cut (<= n_kept), or NULL for n_kept everywhere
    const uint16_t* q_obs;
    const uint16_t* k;
    const float2* stats;    // (m, 1/Z) binary32
    const double* zsum;     // Z binary64
    int P, p_stride, L, W, n_kept, pool, gq, n_q_heads, n_kv_heads, rows, rows_pad;
    int n_seg, seg_tiles;   // pooling workgroups per head and their pooling tiles
    int share_oct;          // groups of eight codes that a sweeping workgroup takes (whole mask words)
    uint32_t w_recip;       // 2^16 / W, rounded up: the quotient of a row number by W (both at most 256) without a division
    float sm_scale;
};

// Pooling ends with a maximum with 0, which no vote is below: a vote that is not a number counts as 0, so a score's pattern is 0 ..
// 0x7f800000 whatever the inputs hold.  Its code fits 16 bits, the bins and the sweep over the codes agree, and every
// head gets exactly as many survivors as it is to have, all of them positions of the prefix.
__device__ __forceinline__ uint32_t score_key(float v) { return __float_as_uint(v); }  // scores are >= 0: bits order like values
__device__ __forceinline__ int score_bin(uint32_t key) { return min(max((int)(key >> kBinShift) - kBinBase, 0), kBins - 1); }

// Eight consecutive candidates share 16 bytes, candidates q and q + 4 the 32-bit word q (so that a
// comparison of both halves of the four words yields their mask byte in order).
typedef unsigned short us2v __attribute__((ext_vector_type(2)));
// mask byte: bit i set where the code of candidate i exceeds t
__device__ __forceinline__ uint32_t codes_above(const uint4& w4, uint32_t t) {
    const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
    const us2v tt = {(unsigned short)t, (unsigned short)t}, one = {1, 1};
    uint32_t m = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        union { uint32_t u; us2v v; } x; x.u = w[q];
        x.v = __builtin_elementwise_min(__builtin_elementwise_sub_sat(x.v, tt), one);
        m |= x.u << q;
    }
    return (m | (m >> 12)) & 0xffu;
}

// Sum of c over the lanes up to this one; the wave's total is lane 63's.  (Lanes passed along a row and the rows' sums
// along the wave, without LDS: an exchange through it takes 50 ns, six of them on a path that is all latency.)
template <int CTRL, int ROWS> __device__ __forceinline__ int dpp_from(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false); }
__device__ __forceinline__ int lanes_up_to(int c) {
    c += dpp_from<0x111, 0xf>(c);   // row_shr 1, 2, 4, 8
    c += dpp_from<0x112, 0xf>(c);
    c += dpp_from<0x114, 0xf>(c);
    c += dpp_from<0x118, 0xf>(c);
    c += dpp_from<0x142, 0xa>(c);   // row_bcast 15: the row before, into rows 1 and 3
    c += dpp_from<0x143, 0xc>(c);   // row_bcast 31: the first half, into the second
    return c;
}
__device__ __forceinline__ int wave_sum(int c) { return __builtin_amdgcn_readlane(lanes_up_to(c), 63); }
__device__ __forceinline__ uint32_t wave_min(uint32_t c) {
    auto low = [&](auto ctrl, auto rows) { c = min(c, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)c, decltype(ctrl)::value, decltype(rows)::value, 0xf, false)); };
    low(IntC<0x111>{}, IntC<0xf>{}); low(IntC<0x112>{}, IntC<0xf>{}); low(IntC<0x114>{}, IntC<0xf>{}); low(IntC<0x118>{}, IntC<0xf>{});
    low(IntC<0x142>{}, IntC<0xa>{}); low(IntC<0x143>{}, IntC<0xc>{});
    return (uint32_t)__builtin_amdgcn_readlane((int)c, 63);
}
// visit(i) for the lanes 0 .. n - 1 (n <= 64) and possibly a few more, eight at a time: a branch that is taken costs 25 ns,
// a lane's value read and compared 3.
template <class Visit>
__device__ __forceinline__ void each_lane(int n, Visit visit) {
    n = __builtin_amdgcn_readfirstlane(n);
    for (int i = 0; i < n; i += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) visit(i + u);
    }
}

// Sum of c over the threads before this one (the caller puts a barrier between two uses of swave).
__device__ __forceinline__ int sum_before(int c, int* swave) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int inc = lanes_up_to(c);
    if (lane == 63) swave[w] = inc;
    __syncthreads();
    int before = inc - c;
#pragma unroll
    for (int i = 0; i < kSelWaves; ++i)
        if (i < w) before += swave[i];
    return before;
}
// Sum of c over the threads after this one (the caller puts a barrier between two uses of swave).
__device__ __forceinline__ int sum_after(int c, int* swave) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int inc = lanes_up_to(c), all = __builtin_amdgcn_readlane(inc, 63);
    if (lane == 63) swave[w] = all;
    __syncthreads();
    int after = all - inc;
#pragma unroll
    for (int i = 0; i < kSelWaves; ++i)
        if (i > w) after += swave[i];
    return after;
}

__device__ __forceinline__ float half_lo(uint32_t w) { return __half2float(__ushort_as_half((uint16_t)(w & 0xffffu))); }
__device__ __forceinline__ float half_hi(uint32_t w) { return __half2float(__ushort_as_half((uint16_t)(w >> 16))); }

// Part of the binary64 vote of one prefix key, computed by one wave: the sum over kPartRows of the group's
// window rows (row_base + lane / 4; the four lanes of a row split the channels) of
// exp2(logit - m_r) / Z_r with the pass-1 statistics.  A product of two binary16 values is exact in
// binary32; the products are summed in binary64.  (It is all latency: few positions are scored, so the rows are spread over as many
// waves as there are and lanes meet without LDS.)
constexpr int kPartRows = 16;
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v) {     // (0 where a row has no such lane)
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double lane_f64(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)b, lane), hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ double vote_f64_part(const SelectArgs& a, int head, int key, int row_base) {
    const int b = head / a.n_kv_heads, g = head % a.n_kv_heads;
    const int lane = threadIdx.x & 63, quarter = lane & 3;
    const int r = row_base + (lane >> 2);
    const bool live = r < a.rows;
    const int rc = live ? r : 0;
    const int hl = (int)(((uint32_t)rc * a.w_recip) >> 16), i = rc - hl * a.W;
    const uint4* kr = reinterpret_cast<const uint4*>(a.k + ((size_t)head * a.L + key) * kHeadDim) + 4 * quarter;
    const uint4* qr = reinterpret_cast<const uint4*>(a.q_obs + (((size_t)b * a.n_q_heads + g * a.gq + hl) * a.W + i) * kHeadDim) + 4 * quarter;
    const double m = (double)a.stats[(size_t)head * a.rows_pad + rc].x;
    const double z = a.zsum[(size_t)head * a.rows_pad + rc];
    double s0 = 0.0, s1 = 0.0;
    uint4 qv[4], kv[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) { qv[c] = qr[c]; kv[c] = kr[c]; }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t qw[4] = {qv[c].x, qv[c].y, qv[c].z, qv[c].w}, kw[4] = {kv[c].x, kv[c].y, kv[c].z, kv[c].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s0 += (double)__builtin_fmaf(half_lo(qw[e]), half_lo(kw[e]), 0.0f);       // (v_fma_mix_f32: no conversions)
            s1 += (double)__builtin_fmaf(half_hi(qw[e]), half_hi(kw[e]), 0.0f);
        }
    }
    double s = s0 + s1;
    s += dpp_f64<0xB1>(s);                        // quad_perm [1,0,3,2]
    s += dpp_f64<0x4E>(s);                        // quad_perm [2,3,0,1]
    double acc = (live && quarter == 0) ? exp2(s * ((double)a.sm_scale * 1.4426950408889634074) - m) / z : 0.0;
    acc += dpp_f64<0x114>(acc);                   // row_shr 4, 8: lane 12 of a row of 16 has its four window rows
    acc += dpp_f64<0x118>(acc);
    return (lane_f64(acc, 12) + lane_f64(acc, 28)) + (lane_f64(acc, 44) + lane_f64(acc, 60));
}

// Max-pooling of one tile: the votes of candidates j0 - r .. j0 + kPoolTile + r go through LDS (0
// outside the prefix) and every thread pools four consecutive candidates, reading
// the votes its windows share once (10 votes for a pool of 7, in three 16-byte reads).
// (The votes are read through a buffer descriptor over the prefix: what lies outside reads as 0 without a test, which on sixteen
// waves are 8 ns an instruction: whole calls, us, 8 heads of 4096 tokens 23.06 -> 22.93, of 32768 68.4 -> 67.9.  The last 64 places
// of the stage are the first wave's.)
struct VoteTile { float v[5]; };
__device__ __forceinline__ __amdgpu_buffer_rsrc_t vote_rsrc(const float* vote, int P) {
    // stride 0 (raw byte offsets), the prefix as the range that is checked, 32-bit data format, no swizzle
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(vote), 0, 4 * P, 0x00020000);
}
__device__ __forceinline__ VoteTile fetch_votes(__amdgpu_buffer_rsrc_t votes, int r, int j0) {
    static_assert(kStage - kPoolTile == 64, "the first wave's");
    VoteTile t;
    const int at = 4 * (j0 - r + (int)threadIdx.x);
#pragma unroll
    for (int u = 0; u < 4; ++u) t.v[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(votes, at + 4 * u * kSelThreads, 0, 0));
    t.v[4] = threadIdx.x < 64 ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(votes, at + 16 * kSelThreads, 0, 0)) : 0.0f;
    return t;
}
__device__ __forceinline__ void stage_votes(const VoteTile& t, float* stage) {
#pragma unroll
    for (int u = 0; u < 4; ++u) stage[threadIdx.x + u * kSelThreads] = t.v[u];
    if (threadIdx.x < 64) stage[threadIdx.x + 4 * kSelThreads] = t.v[4];
}
// Votes 3 .. 2 r of the thread's 2 r + 4 lie in all four windows; the votes before them leave the windows one by one,
// those after them enter.  (Branches on r alone, the same for the whole launch.  256 heads of 32736 candidates, pool 7:
// pool_scores 12 us; with every vote tested against every window 17.)
__device__ __forceinline__ float4 pool_four(const float* stage, int r) {
    const float4* s = reinterpret_cast<const float4*>(stage) + threadIdx.x;
    const float4 a = s[0];
    float4 o;
    if (r >= 2) {
        const int m = r >> 1;                          // 2 r = 4 m or 4 m + 2
        float mid = a.w;
        for (int q = 1; q < m; ++q) {
            const float4 x = s[q];
            mid = fmaxf(mid, fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w)));
        }
        const float4 b = s[m];
        float t0 = b.y, t1 = b.z, t2 = b.w;
        mid = fmaxf(mid, b.x);
        if (r & 1) {
            const float4 c = s[m + 1];
            mid = fmaxf(mid, fmaxf(b.y, b.z));
            t0 = b.w; t1 = c.x; t2 = c.y;
        }
        o.x = fmaxf(fmaxf(a.x, a.y), fmaxf(a.z, mid));
        o.y = fmaxf(fmaxf(a.y, a.z), fmaxf(mid, t0));
        o.z = fmaxf(fmaxf(a.z, mid), fmaxf(t0, t1));
        o.w = fmaxf(fmaxf(mid, t0), fmaxf(t1, t2));
    } else if (r == 1) {
        const float4 c = s[1];
        o.x = fmaxf(fmaxf(a.x, a.y), a.z);
        o.y = fmaxf(fmaxf(a.y, a.z), a.w);
        o.z = fmaxf(fmaxf(a.z, a.w), c.x);
        o.w = fmaxf(fmaxf(a.w, c.x), c.y);
    } else {
        o = a;
    }
    return make_float4(fmaxf(o.x, 0.0f), fmaxf(o.y, 0.0f), fmaxf(o.z, 0.0f), fmaxf(o.w, 0.0f));
}

// Pooled scores and their bin counts; workgroup x of a head takes seg_tiles consecutive tiles.
__global__ __launch_bounds__(kSelThreads) void pool_scores(const SelectArgs a) {
    __shared__ __align__(16) float stage[kStage];
    __shared__ __align__(16) int hist[kBinRow];
    const int head = blockIdx.y;
    const int P = a.P, k = a.head_n ? a.head_n[head] : a.n_kept;
    if (k <= 0 || k >= P) return;               // (nothing of this head is cut)
    const float* vote = a.vote + (size_t)head * P;
    uint32_t* code = reinterpret_cast<uint32_t*>(a.code + (size_t)head * a.p_stride);
    const int r = (a.pool - 1) / 2;
    const int t_begin = blockIdx.x * a.seg_tiles, t_end = min((P + kPoolTile - 1) / kPoolTile, t_begin + a.seg_tiles);
    const __amdgpu_buffer_rsrc_t votes = vote_rsrc(vote, P);
    VoteTile next = fetch_votes(votes, r, t_begin * kPoolTile);
    *reinterpret_cast<int4*>(hist + 4 * threadIdx.x) = make_int4(0, 0, 0, 0);
    for (int t = t_begin; t < t_end; ++t) {
        stage_votes(next, stage);
        __syncthreads();
        if (t + 1 < t_end) next = fetch_votes(votes, r, (t + 1) * kPoolTile);   // in flight while this tile is pooled
        const float4 o = pool_four(stage, r);
        const int j = t * kPoolTile + 4 * (int)threadIdx.x;
        const uint32_t key[4] = {score_key(o.x), score_key(o.y), score_key(o.z), score_key(o.w)};
        const bool whole = (t + 1) * kPoolTile <= P;              // (all tiles but a head's last)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (whole || j + i < P) atomicAdd(&hist[score_bin(key[i])], 1);
        // codes of the thread's four candidates (0 past the end), then the octet's words: the even
        // thread stores words 0 and 1, the odd one words 2 and 3
        uint32_t cd[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) cd[i] = whole || j + i < P ? key[i] >> kCodeShift : 0u;
        const bool odd = threadIdx.x & 1;
        const uint32_t give0 = odd ? cd[0] : cd[2], give1 = odd ? cd[1] : cd[3];
        const uint32_t got0 = __builtin_amdgcn_mov_dpp(give0, 0xB1 /*quad_perm [1,0,3,2]*/, 0xf, 0xf, true);
        const uint32_t got1 = __builtin_amdgcn_mov_dpp(give1, 0xB1, 0xf, 0xf, true);
        if ((j & ~7) < P)
            *reinterpret_cast<uint2*>(code + (j >> 1)) = odd ? make_uint2(got0 | (cd[2] << 16), got1 | (cd[3] << 16))
                                                             : make_uint2(cd[0] | (got0 << 16), cd[1] | (got1 << 16));
        __syncthreads();
    }
    // (the words behind the bins' counts stay 0 here: the places of the groups' counts)
    const int4 c = *reinterpret_cast<const int4*>(hist + 4 * threadIdx.x);
    uint16_t* row = a.bins + ((size_t)head * a.n_seg + blockIdx.x) * kBinRow;
    if (4 * (int)threadIdx.x < kBins)
        reinterpret_cast<uint2*>(row)[threadIdx.x] = make_uint2((uint32_t)c.x | ((uint32_t)c.y << 16), (uint32_t)c.z | ((uint32_t)c.w << 16));
    int sum = (c.x + c.y) + (c.z + c.w);        // a group is the bins of sixteen threads
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    if ((threadIdx.x & 15) == 0) row[kBins + (threadIdx.x >> 4)] = (uint16_t)sum;
}

// The bin of the k-th largest score: its group by the groups' counts, then by the counts of that group's bins
// (two round trips, but a few KB per workgroup instead of all counts).  One wave's work.
__device__ __forceinline__ int bin_of_cut(const uint16_t* bins, int n_seg, int k) {
    const int lane = threadIdx.x & 63;
    auto find = [&](const uint16_t* row, int n, int& above) {
        uint16_t x[kMaxSegs];
#pragma unroll
        for (int s = 0; s < kMaxSegs; ++s) x[s] = s < n_seg && lane < n ? row[(size_t)s * kBinRow + lane] : (uint16_t)0;
        int c = 0;
#pragma unroll
        for (int s = 0; s < kMaxSegs; ++s) c += x[s];
        const int inc = lanes_up_to(c), before = above + __builtin_amdgcn_readlane(inc, 63) - inc;
        const unsigned long long here = __builtin_amdgcn_ballot_w64(before < k && before + c >= k);   // exactly one lane
        const int at = here ? __builtin_ctzll(here) : 0;
        above = __builtin_amdgcn_readlane(before, at);
        return at;
    };
    int above = 0;
    const int group = find(bins + kBins, kGroups, above);
    return kGroupBins * group + find(bins + kGroupBins * group, kGroupBins, above);
}

// T > 0: the prefix is at most T pooling tiles, pooled and counted here by one workgroup per (batch, kv head); of every tile
// thread t keeps the scores of candidates 4 t .. 4 t + 3.
// kAlone: pool_scores has left codes and counts; one workgroup per head sweeps them.
// kSpread: the same by several workgroups of a head.  Each finds the bin of the cut and sweeps the codes of its
// share, one group of eight per thread; mask and list of the share then take the place of the codes that they came from,
// and the workgroup that arrives last goes on with all of them.
// keep: the survivor mask, bit j % 8 of byte j / 8.
enum { kAlone = 0, kSpread = -1 };
template <int T>
__global__ __launch_bounds__(kSelThreads) void select_topk(const SelectArgs a) {
    constexpr bool OWN = T > 0, SPREAD = T == kSpread;
    __shared__ __align__(16) uint32_t keep[(OWN ? T * kPoolTile : kMaxPrefix) / 32];
    __shared__ __align__(16) int tab[2 * kSelThreads + kVoteSlots];      // the counts of the bins (OWN); later the band, then:
    int* hist = tab + 2 * kSelThreads;                            // radix digits and the candidates of the last; later the positions to re-score
    uint32_t* ties = reinterpret_cast<uint32_t*>(tab);            // where binary32 decides: the mask of the candidates equal to the cut
    __shared__ __align__(16) unsigned char big[T > 1 ? 2 * kStage * 4 : kListCap * 8];     // candidates around the cut, or (too many) the pooling stage; before that the pooling stage (OWN); later the binary64 votes
    __shared__ int swave[kSelWaves];
    __shared__ int s_bin, s_list, s_listed, s_sure, s_last, s_digit, s_above, s_few, s_take, s_band, s_hot;
    __shared__ uint32_t s_cut;
    static_assert(kListCap * 8 >= kStage * 4 && sizeof(tab) >= kBinRow * 4 && sizeof(tab) >= (2 * kSelWaves + kListCap) * 4 && kListCap * 8 >= (kPartSlots + kVoteSlots) * 8 &&
                  sizeof(tab) >= kMaxPrefix / 8 && (1 << kDigit) == kSelThreads && kVoteSlots >= (1 << kDigit) + 2 * kFew, "aliases fit");

    const int head = blockIdx.y;
    const int P = a.P, k = a.head_n ? a.head_n[head] : a.n_kept;
    const float* vote = a.vote + (size_t)head * P;
    int32_t* idx = a.idx + (size_t)head * a.n_kept;
    int32_t* list = a.list ? a.list + (size_t)head * a.n_kept : idx;      // (the same words twice where there is none)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = (a.pool - 1) / 2;

    if (k <= 0 || k >= P) {   // (a head-level count may be zero; one that covers the prefix: identity, the scores are not looked at)
        if (a.unrefined && blockIdx.x == 0 && threadIdx.x == 0) a.unrefined[head] = 0;
        for (int j = blockIdx.x * kSelThreads + threadIdx.x; j < k; j += gridDim.x * kSelThreads) { idx[j] = j; list[j] = j; }
        return;
    }
    if (threadIdx.x == 0) { s_list = 0; s_sure = 0; s_listed = 0; s_few = 0; s_band = 0; s_hot = 0; }

    // ---- the bin of the k-th largest score ----
    uint32_t own[OWN ? 4 * T : 1];                 // OWN: the thread's scores (all ones past the end: neither above nor around the cut)
    auto own_at = [&](int i) { return (i >> 2) * kPoolTile + 4 * (int)threadIdx.x + (i & 3); };   // ... and their candidates
    constexpr int OCTS = SPREAD ? 1 : kMaxShares;  // groups of eight codes per thread (not OWN): thread + 1024 i of the share
    const int n_oct = (P + 7) / 8, oct0 = SPREAD ? blockIdx.x * a.share_oct : 0, own_oct = SPREAD ? min(a.share_oct, n_oct - oct0) : n_oct;
    char* codes = OWN ? nullptr : reinterpret_cast<char*>(a.code + (size_t)head * a.p_stride);
    uint4 oct[OWN ? 1 : OCTS];
    if constexpr (OWN) {
        const int n_tiles = (P + kPoolTile - 1) / kPoolTile;
        // (two places for a tile's votes, one barrier per tile; two tiles' votes on their way while one is pooled)
        const __amdgpu_buffer_rsrc_t votes = vote_rsrc(vote, P);
        VoteTile next[2] = {fetch_votes(votes, r, 0), {}};
        if (T > 1 && n_tiles > 1) next[1] = fetch_votes(votes, r, kPoolTile);
        for (int i = threadIdx.x; i < T * kPoolTile / 32; i += kSelThreads) keep[i] = 0u;
        *reinterpret_cast<int4*>(tab + 4 * threadIdx.x) = make_int4(0, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < T; ++q) {
            if (q < n_tiles) {
                float* stage = reinterpret_cast<float*>(big) + (q & 1) * kStage;
                stage_votes(next[q & 1], stage);
                __syncthreads();
                if (q + 2 < T && q + 2 < n_tiles) next[q & 1] = fetch_votes(votes, r, (q + 2) * kPoolTile);
                const float4 o = pool_four(stage, r);
                const float ov[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool in = (q + 1) * kPoolTile <= P || own_at(4 * q + i) < P;      // (whole tiles without a test)
                    own[4 * q + i] = in ? score_key(ov[i]) : 0xffffffffu;
                    if (in) atomicAdd(&tab[score_bin(own[4 * q + i])], 1);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) own[4 * q + i] = 0xffffffffu;
            }
        }
        __syncthreads();
        const int4 b = *reinterpret_cast<const int4*>(tab + 4 * threadIdx.x);
        const int c[4] = {b.x, b.y, b.z, b.w};         // counts of bins 4 thread .. 4 thread + 3
        // every wave its 256 bins; the wave that has the cut looks closer
        const int inc = lanes_up_to((c[0] + c[1]) + (c[2] + c[3])), all = __builtin_amdgcn_readlane(inc, 63);
        if (lane == 0) swave[wave] = all;
        __syncthreads();
        const int up_to = lanes_up_to(lane < kSelWaves ? swave[lane] : 0);
        int above = __builtin_amdgcn_readlane(up_to, kSelWaves - 1) - __builtin_amdgcn_readlane(up_to, wave);
        if (above < k && above + all >= k) {
            above += all - inc;
#pragma unroll
            for (int i = 3; i >= 0; --i) {
                if (above < k && above + c[i] >= k) s_bin = 4 * (int)threadIdx.x + i;    // exactly one bin
                above += c[i];
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < OCTS; ++i) {
            const int o = (int)threadIdx.x + i * kSelThreads;
            oct[i] = o < own_oct ? reinterpret_cast<const uint4*>(codes)[oct0 + o] : make_uint4(0u, 0u, 0u, 0u);
        }
        if (wave == 0) {
            const int bin = bin_of_cut(a.bins + (size_t)head * a.n_seg * kBinRow, a.n_seg, k);
            if (lane == 0) s_bin = bin;
        }
    }
    __syncthreads();                                   // (the counters in LDS are set, too)
    const int cb = __builtin_amdgcn_readfirstlane(s_bin);
    // Candidates of that bin and one code on either side (32768 patterns; the band around the cut
    // reaches at most 2e-5 * 2^24 = 336): codes clo .. chi, patterns klo .. khi.  Everything above survives.
    constexpr uint32_t kCodesPerBin = 1u << (kBinShift - kCodeShift);
    const uint32_t clo = cb == 0 ? 0u : (uint32_t)(cb + kBinBase) * kCodesPerBin - 1u;
    const uint32_t chi = cb == kBins - 1 ? 0xffffu : (uint32_t)(cb + 1 + kBinBase) * kCodesPerBin;
    const uint32_t klo = clo << kCodeShift, khi = (chi << kCodeShift) | ((1u << kCodeShift) - 1u);

    // ---- one sweep: the mask of what lies above, the list of what lies around the cut ----
    uint32_t* list_key = reinterpret_cast<uint32_t*>(big);
    int* list_pos = reinterpret_cast<int*>(big + kListCap * 4);
    uint32_t* groups = reinterpret_cast<uint32_t*>(tab) + 2 * kSelWaves;        // [kListCap], not OWN: groups with candidates around the cut, until these are listed
    // s_list, not OWN: groups above this bit, candidates below.  131072 of these fit.  16384 groups, all that there are, wrap to 0 once the last
    // is counted; no earlier one reads that, and with that many the candidates are beyond the list, which is then not used.
    constexpr int kGroupCount = 18;
    static_assert(kMaxPrefix < (1 << kGroupCount) && kMaxPrefix / 8 <= (1 << (32 - kGroupCount)) && (1 << (32 - kGroupCount)) > kListCap, "the counts fit, or do not count");
    int sure = 0;
    if constexpr (OWN) {
#pragma unroll
        for (int q = 0; q < T; ++q) {
            uint32_t bits = 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) bits |= (int)own[4 * q + i] > (int)khi ? 1u << i : 0u;
            sure += __popc(bits);
            if (bits) atomicOr(&keep[q * (kPoolTile / 32) + (threadIdx.x >> 3)], bits << (4 * (threadIdx.x & 7)));
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (own[4 * q + i] >= klo && own[4 * q + i] <= khi) {
                    const int e = atomicAdd(&s_list, 1);
                    if (e < kListCap) { list_key[e] = own[4 * q + i]; list_pos[e] = own_at(4 * q + i); }
                }
        }
    } else {
        // (a group with candidates around the cut is listed whole, {group, which of its eight}: the sweep is bound by what it
        // issues, and a write per candidate was most of it)
#pragma unroll
        for (int i = 0; i < OCTS; ++i) {
            const int o = (int)threadIdx.x + i * kSelThreads;
            if (!SPREAD && o >= own_oct) break;
            const uint32_t above = codes_above(oct[i], chi);                    // (past the share or the end the codes are 0)
            uint32_t around = clo ? codes_above(oct[i], clo - 1u) & ~above : 0xffu & ~above;
            if (8 * (oct0 + o) + 8 > P) around &= (1u << max(P - 8 * (oct0 + o), 0)) - 1u;
            if (SPREAD && o >= own_oct) around = 0u;
            reinterpret_cast<unsigned char*>(keep)[o] = (unsigned char)above;
            sure += __popc(above);
            if (around) {
                const uint32_t e = (uint32_t)atomicAdd(&s_list, (1 << kGroupCount) + __popc(around)) >> kGroupCount;
                if (e < kListCap) groups[e] = ((uint32_t)(oct0 + o) << 8) | around;
            }
        }
        if (!SPREAD)
            for (int o = n_oct + (int)threadIdx.x; o < (n_oct + 3) / 4 * 4; o += kSelThreads) reinterpret_cast<unsigned char*>(keep)[o] = 0;
    }
    sure = wave_sum(sure);
    if (lane == 0 && sure) atomicAdd(&s_sure, sure);
    __syncthreads();
    int n_list = __builtin_amdgcn_readfirstlane(s_list), n_groups = 0;
    int n_sure = __builtin_amdgcn_readfirstlane(s_sure);
    if constexpr (!OWN) { n_groups = (int)((uint32_t)n_list >> kGroupCount); n_list &= (1 << kGroupCount) - 1; }
    if constexpr (SPREAD) {
        // {survivors, candidates, groups}, mask and groups of the share go where its codes were (the barrier: all of them are in
        // registers; 16 bytes a group of codes, one and four a group here), with device-scope
        // stores: the workgroup that arrives last may be on another XCD.
        constexpr int kSlotHead = 16;
        auto octs_of = [&](int share) { return min(a.share_oct, n_oct - share * a.share_oct); };
        auto words_of = [&](int octs) { return (octs + 3) / 4; };              // 32-bit mask words
        char* slot = codes + (size_t)oct0 * 16;
        const int mask_words = words_of(own_oct);
        auto put = [](void* p, uint32_t v) { __hip_atomic_store(reinterpret_cast<uint32_t*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        auto get = [](const void* p) { return __hip_atomic_load(reinterpret_cast<const uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        if (threadIdx.x < 3) put(slot + 4 * threadIdx.x, (uint32_t)(threadIdx.x == 0 ? n_sure : threadIdx.x == 1 ? n_list : n_groups));
        if ((int)threadIdx.x < mask_words) put(slot + kSlotHead + 4 * threadIdx.x, keep[threadIdx.x]);
        if ((int)threadIdx.x < n_groups) put(slot + kSlotHead + 4 * (mask_words + threadIdx.x), groups[threadIdx.x]);
        // Every store is acknowledged at the device's coherence point before the workgroup's arrival is counted there.
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const int n_shares = gridDim.x;
        if (threadIdx.x == 0) {
            uint32_t* arrivals = reinterpret_cast<uint32_t*>(a.bins + (size_t)head * a.n_seg * kBinRow + kBinRow - 2);   // (upper half of the word)
            s_last = (int)(__hip_atomic_fetch_add(arrivals, 1u << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 16) == n_shares - 1;
        }
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(s_last)) return;
        // Masks and groups of all shares into LDS: a share's by sixteen / n_shares waves, one round trip (but for many groups).
        {
            const int per = kSelWaves / n_shares, share = wave % n_shares, sub = wave / n_shares;
            const bool part = sub < per;
            const int octs = octs_of(share), words = part ? words_of(octs) : 0, at = part ? 64 * sub + lane : 0, step = 64 * per;
            const char* from = codes + (size_t)share * a.share_oct * 16;
            constexpr int kMaskLoads = kSelThreads / 4 / 64;              // mask words per lane of a wave that has a share to itself
            const uint32_t some = get(from), count = get(from + 4), mine = get(from + 8);
            uint32_t m[kMaskLoads], group = 0u;
#pragma unroll
            for (int u = 0; u < kMaskLoads; ++u) m[u] = at + u * step < words ? get(from + kSlotHead + 4 * (at + u * step)) : 0u;
            if (part && at < octs) group = get(from + kSlotHead + 4 * (words + at));      // (one group at least lies behind the mask's place)
            if (sub == 0 && lane == 0) { swave[share] = (int)mine; tab[share] = (int)some; tab[kSelWaves + share] = (int)count; }
#pragma unroll
            for (int u = 0; u < kMaskLoads; ++u)
                if (at + u * step < words) keep[share * (a.share_oct / 4) + at + u * step] = m[u];
            __syncthreads();
            const int up_to = lanes_up_to(lane < n_shares ? swave[lane] : 0), before = share > 0 ? __builtin_amdgcn_readlane(up_to, share - 1) : 0;
            n_groups = __builtin_amdgcn_readlane(up_to, 63);
            n_sure = wave_sum(lane < n_shares ? tab[lane] : 0);
            n_list = wave_sum(lane < n_shares ? tab[kSelWaves + lane] : 0);
            if (part && n_groups <= kListCap)
                for (int e = at; e < (int)mine; e += step) groups[before + e] = e == at ? group : get(from + kSlotHead + 4 * (words + e));
            __syncthreads();
        }
    }
    if (a.unrefined && threadIdx.x == 0) a.unrefined[head] = 0;   // (overwritten below by the same thread if binary32 decides)
    const int need_around = k - n_sure;   // how many of the candidates around the cut survive
    // the pooled score of a candidate, from the votes
    auto pooled_key = [&](int j) -> uint32_t {
        const int t1 = min(j + r, P - 1);
        float best = 0.0f;
        for (int t = max(j - r, 0); t <= t1; t += 8) {      // (eight votes in flight; past the window its last one again)
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = vote[min(t + u, t1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) best = fmaxf(best, x[u]);
        }
        return score_key(best);
    };
    if constexpr (!OWN) {
        // the listed groups' candidates and their scores, eight threads a group
        if (n_list <= kListCap)
            for (int i = threadIdx.x; i < 8 * n_groups; i += kSelThreads) {
                const uint32_t group = groups[i >> 3];
                if (group >> (i & 7) & 1u) {
                    const int j = 8 * (int)(group >> 8) + (i & 7);
                    const uint32_t key = pooled_key(j);
                    const int e = atomicAdd(&s_listed, 1);
                    list_key[e] = key; list_pos[e] = j;
                }
            }
    }
    // Where the list is too short (thousands of scores within two percent of the cut), the whole prefix is
    // pooled once more, tile by tile, into memory; a thread reads back only what it has stored itself.  (In a
    // workspace without that room every visit pools every candidate.)
    // (Whole calls with 8 heads, pool 7: all keys alike, 32736 / 131008 candidates, 127 / 388 us, where
    // pooling every candidate by itself on every visit took 214 / 726; scores spread evenly over 0.1 %,
    // 125 / 379 against 184 / 613.)
    float* exact = a.exact ? a.exact + (size_t)head * a.p_stride : nullptr;
    if constexpr (!OWN) {
        if (__builtin_expect(n_list > kListCap && exact, 0)) {
            float* stage = reinterpret_cast<float*>(big);
            const __amdgpu_buffer_rsrc_t votes = vote_rsrc(vote, P);
            VoteTile next = fetch_votes(votes, r, 0);
            for (int j0 = 0; j0 < P; j0 += kPoolTile) {
                __syncthreads();
                stage_votes(next, stage);
                __syncthreads();
                if (j0 + kPoolTile < P) next = fetch_votes(votes, r, j0 + kPoolTile);
                const float4 o = pool_four(stage, r);
                if (j0 + 4 * (int)threadIdx.x < P) *reinterpret_cast<float4*>(exact + j0 + 4 * threadIdx.x) = o;
            }
        }
    }
    __syncthreads();                            // (the list and its scores are there)
    // every candidate around the cut: from the list (in no particular order), from the thread's own scores (OWN) or
    // from all pooled scores
    auto each_around = [&](auto visit) {
        if (__builtin_expect(n_list <= kListCap, 1)) {
            for (int e = threadIdx.x; e < n_list; e += kSelThreads) visit(list_key[e], list_pos[e]);
        } else if constexpr (OWN) {
#pragma unroll
            for (int i = 0; i < 4 * T; ++i)
                if (own[i] >= klo && own[i] <= khi) visit(own[i], own_at(i));
        } else if (!exact) {
            for (int j = threadIdx.x; j < P; j += kSelThreads) {
                const uint32_t key = pooled_key(j);
                if (key >= klo && key <= khi) visit(key, j);
            }
        } else {
            const int last = (P - 1) & ~3;
            int j = 4 * (int)threadIdx.x;
            float4 next = *reinterpret_cast<const float4*>(exact + min(j, last));
#pragma unroll 1
            for (; j < P; j += kPoolTile) {
                float4 o = next;
                next = *reinterpret_cast<const float4*>(exact + min(j + kPoolTile, last));
#pragma unroll 1
                for (int i = 0; i < 4; ++i) {
                    const uint32_t key = score_key(o.x);
                    if (j + i < P && key >= klo && key <= khi) visit(key, j + i);
                    o.x = o.y; o.y = o.z; o.z = o.w;
                }
            }
        }
    };
    auto set_keep = [&](int j) { atomicOr(&keep[j >> 5], 1u << (j & 31)); };

    // ---- the cut, the survivors above its band, and the band in position order ----
    // Every instruction of the workgroup's sixteen waves costs 8 ns here, one of a single wave 2, a barrier 12 and a
    // branch that is taken 25.  So few candidates are one wave's work, one per lane, in straight lines; of more candidates
    // a radix pass leaves those whose digit is near the cut's (plateaus of the max-pool make several of them alike).
    int* band_raw = tab;                                                   // [kMaxBand] as found
    int* band_pos = tab + kMaxBand;                                        // [kMaxBand] ascending
    double* band_score = reinterpret_cast<double*>(tab + 2 * kMaxBand);    // [kMaxBand]
    static_assert(4 * kMaxBand <= 2 * kSelThreads, "the band fits the table");
    // One pass: counts the digits of the candidates that share the prefix and finds the need-th largest's.
    uint32_t prefix = 0u;
    int need = need_around;                     // the cut is the need-th largest of the candidates that share the prefix
    int fixed = 32 - __builtin_clz(khi - klo), shift = fixed;
    auto radix_pass = [&] {
        hist[threadIdx.x] = 0;
        __syncthreads();
        shift = fixed > kDigit ? fixed - kDigit : 0;
        each_around([&](uint32_t key, int) {
            const uint32_t rel = key - klo;
            if (fixed >= 32 || (rel >> fixed) == (prefix >> fixed)) {
                const int digit = (int)((rel >> shift) & ((1u << (fixed - shift)) - 1u)), some = __builtin_amdgcn_readfirstlane(digit);
                const unsigned long long alike = __builtin_amdgcn_ballot_w64(digit == some);     // (ties: one of the lanes counts them all)
                if (digit != some) atomicAdd(&hist[digit], 1);
                else if (lane == __builtin_ctzll(alike)) atomicAdd(&hist[some], __popcll(alike));
            }
        });
        __syncthreads();
        if (wave == 0) {                        // lane l: digits 256 u + 4 l .. + 3
            int4 c[4];
            int inc[4], all[4], above[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = reinterpret_cast<const int4*>(hist)[64 * u + lane];
                inc[u] = lanes_up_to((c[u].x + c[u].y) + (c[u].z + c[u].w));
                all[u] = __builtin_amdgcn_readlane(inc[u], 63);
            }
#pragma unroll
            for (int u = 3; u >= 0; --u) above[u] = u == 3 ? 0 : above[u + 1] + all[u + 1];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int four[4] = {c[u].x, c[u].y, c[u].z, c[u].w};
                int before = above[u] + all[u] - inc[u];
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    if (before < need && before + four[q] >= need) { s_digit = 256 * u + 4 * lane + q; s_above = before; }     // exactly one digit
                    before += four[q];
                }
            }
        }
        __syncthreads();
        prefix |= __builtin_amdgcn_readfirstlane(s_digit) << shift;
        need -= __builtin_amdgcn_readfirstlane(s_above);
        fixed = shift;
    };
    const uint32_t* few_key = list_key;
    const int* few_pos = list_pos;
    int n_few = n_list;                         // candidates that one wave may go on with, and ...
    int need_few = need_around;                 // ... how many of them survive
    if (__builtin_expect(n_list > kFew && n_list <= kListCap, 0)) {
        radix_pass();
        // the digits that the band can reach: it is narrower than two of them (336 patterns; a digit has 256 and more)
        uint32_t* key_to = reinterpret_cast<uint32_t*>(hist) + (1 << kDigit);
        int* pos_to = hist + (1 << kDigit) + kFew;
        const uint32_t digit = prefix >> shift, last = (1u << kDigit) - 1u;
        const uint32_t d_hi = min(digit + 2u, last), d_lo = digit > 2u ? digit - 2u : 0u;
        need_few = need;
        if (digit + 1u <= last) need_few += hist[digit + 1u];
        if (digit + 2u <= last) need_few += hist[digit + 2u];
        each_around([&](uint32_t key, int j) {
            const uint32_t d = (key - klo) >> shift;
            if (d > d_hi) set_keep(j);
            else if (d >= d_lo) {
                const int e = atomicAdd(&s_few, 1);
                if (e < kFew) { key_to[e] = key; pos_to[e] = j; }
            }
        });
        __syncthreads();
        n_few = __builtin_amdgcn_readfirstlane(s_few);
        few_key = key_to; few_pos = pos_to;
    }
    if (__builtin_expect(n_few <= kFew, 1)) {
        if (wave == 0) {
            const uint32_t key = lane < n_few ? few_key[lane] : 0u;
            const int j = lane < n_few ? few_pos[lane] : 0x7fffffff;
            int above = 0;
            each_lane(n_few, [&](int i) { above += (uint32_t)__builtin_amdgcn_readlane((int)key, i) > key; });     // (lanes past them: 0)
            // the cut is the lowest score that fewer than need_few are above
            const uint32_t at_cut = wave_min(lane < n_few && above < need_few ? key : 0xffffffffu);
            const float low = __uint_as_float(at_cut) * (1.0f - kBandRel), high = __uint_as_float(at_cut) * (1.0f + kBandRel), v = __uint_as_float(key);
            const bool over = lane < n_few && v > high, in = lane < n_few && v <= high && v >= low;
            if (over) set_keep(j);
            const unsigned long long band = __builtin_amdgcn_ballot_w64(in);
            const int n_over = __popcll(__builtin_amdgcn_ballot_w64(over)), n_band = __popcll(band);
            if (in) band_raw[__builtin_amdgcn_mbcnt_hi((uint32_t)(band >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)band, 0u))] = j;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // (LDS serves a wave in order; this only pins the compiler)
            const int mine = lane < n_band ? band_raw[lane] : 0x7fffffff;
            int rank = 0;
            each_lane(n_band, [&](int i) { rank += __builtin_amdgcn_readlane(mine, i) < mine; });
            if (lane < n_band) band_pos[rank] = mine;
            const int n_above = __builtin_amdgcn_readlane(above, __builtin_ctzll(__builtin_amdgcn_ballot_w64(lane < n_few && key == at_cut)));
            if (lane == 0) { s_cut = at_cut; s_band = n_band; s_take = need_few - n_over; s_above = need_few - n_above; }
        }
    } else {
        if (n_list > kListCap) radix_pass();
        while (shift > 0) { __syncthreads(); radix_pass(); }
        if (threadIdx.x == 0) { s_cut = klo + prefix; s_sure = 0; }
        __syncthreads();
        const float at_cut = __uint_as_float(klo + prefix), low = at_cut * (1.0f - kBandRel), high = at_cut * (1.0f + kBandRel);
        each_around([&](uint32_t key, int j) {
            const float v = __uint_as_float(key);
            if (v > high) { set_keep(j); atomicAdd(&s_sure, 1); }
            else if (v >= low) {
                const int e = atomicAdd(&s_band, 1);
                if (e < kMaxBand) band_raw[e] = j;
            }
        });
        __syncthreads();
        if (threadIdx.x == 0) { s_take = need_around - s_sure; s_above = need; }
        if (s_band <= kMaxBand)
            for (int e = threadIdx.x; e < s_band; e += kSelThreads) {
                const int j = band_raw[e];
                int rank = 0;
                for (int o = 0; o < s_band; ++o) rank += band_raw[o] < j;
                band_pos[rank] = j;
            }
    }
    __syncthreads();
    const uint32_t cut_key = __builtin_amdgcn_readfirstlane(s_cut);
    const float cut = __uint_as_float(cut_key);
    const float lo = cut * (1.0f - kBandRel), hi = cut * (1.0f + kBandRel);    // scores that binary32 rounding could move across the cut
    const int tot_band = __builtin_amdgcn_readfirstlane(s_band);
    const int take = __builtin_amdgcn_readfirstlane(s_take);                   // members of the band that survive
    const int need_at_cut = __builtin_amdgcn_readfirstlane(s_above);           // how many candidates equal to the cut are taken (binary32 rule)
    bool refine = tot_band <= kMaxBand;
    int* hot_pos = hist;                                                   // [kVoteSlots]
    int n_hot = 0;
    if (refine && take < tot_band) {
        // ---- the positions whose votes decide: a member's pooled score is the vote of a position in its
        // window that lies in the band itself (with a margin for the edge), so only such votes are
        // scored again, each once -- by the member whose window no earlier member's window covers.  If
        // one position stands behind the whole band (the usual case: a plateau of the max-pool), its
        // members are equal in any precision and nothing needs to be scored.
        const float lo2 = lo * (1.0f - 1.0e-6f), hi2 = hi * (1.0f + 1.0e-6f);
        const int span = 2 * r + 1;
        for (int item = threadIdx.x; item < tot_band * span; item += kSelThreads) {
            const int m = item / span, j = band_pos[m] - r + item % span;
            if (j < 0 || j >= P || (m > 0 && j <= band_pos[m - 1] + r)) continue;
            const float v = vote[j];
            if (v >= lo2 && v <= hi2) {
                const int e = atomicAdd(&s_hot, 1);
                if (e < kVoteSlots) hot_pos[e] = j;
            }
        }
        __syncthreads();
        n_hot = __builtin_amdgcn_readfirstlane(s_hot);
        refine = n_hot <= kVoteSlots;
    }
    if (__builtin_expect(refine, 1)) {
        if (n_hot > 1) {
            // ---- binary64 re-scoring: one wave per (position, kPartRows window rows); the parts of a position are
            // summed in ascending order.  Positions go in batches that fit the parts. ----
            double* part_vote = reinterpret_cast<double*>(big);                      // [kPartSlots]
            double* pos_vote = reinterpret_cast<double*>(big) + kPartSlots;          // [kVoteSlots]
            const int n_parts = (a.rows + kPartRows - 1) / kPartRows;           // (at most 16)
            const int batch = kPartSlots / n_parts;
            for (int p0 = 0; p0 < n_hot; p0 += batch) {
                const int np = min(batch, n_hot - p0);
                for (int item = wave; item < np * n_parts; item += kSelWaves) {
                    const double v = vote_f64_part(a, head, hot_pos[p0 + item / n_parts], kPartRows * (item % n_parts));
                    if (lane == 0) part_vote[item] = v;
                }
                __syncthreads();
                for (int i = threadIdx.x; i < np; i += kSelThreads) {
                    double sum = 0.0;
#pragma unroll
                    for (int q = 0; q < kWideRows / kPartRows; ++q) sum += q < n_parts ? part_vote[i * n_parts + q] : 0.0;
                    pos_vote[p0 + i] = sum;
                }
                __syncthreads();
            }
            // ---- pooled binary64 score of each member, and its rank by (score desc, position asc) ----
            if (tot_band <= 64 && n_hot <= 64) {              // (the usual case: one wave, a member and a position per lane)
                if (wave == 0) {
                    const int j = lane < tot_band ? band_pos[lane] : -1, hot = lane < n_hot ? hot_pos[lane] : -0x40000000;
                    const double hot_vote = lane < n_hot ? pos_vote[lane] : 0.0;
                    double best = 0.0;                        // votes are >= 0
                    each_lane(n_hot, [&](int i) {
                        const double v = lane_f64(hot_vote, i);
                        if (abs(__builtin_amdgcn_readlane(hot, i) - j) <= r) best = fmax(best, v);
                    });
                    if (lane >= tot_band) best = -1.0;
                    int rank = 0;
                    each_lane(tot_band, [&](int i) {
                        const double o = lane_f64(best, i);
                        rank += (o > best) || (o == best && i < lane);
                    });
                    if (lane < tot_band && rank < take) set_keep(j);
                }
            } else {
            for (int m = threadIdx.x; m < tot_band; m += kSelThreads) {
                const int j = band_pos[m];
                double best = 0.0;                            // votes are >= 0
                for (int i = 0; i < n_hot; ++i)
                    if (abs(hot_pos[i] - j) <= r) best = fmax(best, pos_vote[i]);
                band_score[m] = best;
            }
            __syncthreads();
            for (int m = threadIdx.x; m < tot_band; m += kSelThreads) {
                const double sc = band_score[m];
                int rank = 0;
                for (int o = 0; o < tot_band; ++o) rank += (band_score[o] > sc) || (band_score[o] == sc && o < m);
                if (rank < take) set_keep(band_pos[m]);
            }
            }
        } else {                                              // all taken, or all equal: by position
            for (int m = threadIdx.x; m < min(take, tot_band); m += kSelThreads) set_keep(band_pos[m]);
        }
        __syncthreads();
    } else {
        // binary32 decides: everything above the cut, then the first need_at_cut equal to it
        if (a.unrefined && threadIdx.x == 0) a.unrefined[head] = tot_band;
        const int n_words = (P + 31) / 32;
        for (int i = threadIdx.x; i < n_words; i += kSelThreads) ties[i] = 0u;
        __syncthreads();
        each_around([&](uint32_t key, int j) {
            if (key > cut_key) set_keep(j);
            else if (key == cut_key) atomicOr(&ties[j >> 5], 1u << (j & 31));
        });
        __syncthreads();
        const int per = (n_words + kSelThreads - 1) / kSelThreads;   // mask words of a thread, in position order
        int mine = 0;
        for (int i = 0; i < per; ++i) {
            const int w = (int)threadIdx.x * per + i;
            if (w < n_words) mine += __popc(ties[w]);
        }
        int left = need_at_cut - sum_before(mine, swave);
        for (int i = 0; i < per && left > 0; ++i) {
            const int w = (int)threadIdx.x * per + i;
            if (w >= n_words) break;
            for (uint32_t m = ties[w]; m && left > 0; m &= m - 1u, --left) set_keep(32 * w + __builtin_ctz(m));
        }
        __syncthreads();
    }

    // ---- ordered compaction: a wave owns consecutive 64-bit mask words and stores the positions of one
    // at a time, side by side (a thread that walks the bits of its own mask bytes writes every line
    // in many pieces: 17 instead of 5 us when 256 heads do it at once; collecting positions in LDS
    // for 16-byte stores gains nothing: the loop issues instructions, it does not wait for stores; so both stores of a
    // position share a 32-bit offset: 8 heads of 131072 keys take as long as with one list; with two 64-bit addresses 1.8 us more) ----
    const int n_words = (P + 63) / 64, per = (n_words + kSelWaves - 1) / kSelWaves;      // (per <= 128)
    const int w0 = wave * per, w1 = min(w0 + per, n_words);
    uint32_t word[4] = {0u, 0u, 0u, 0u};                     // lane l: words w0 + l and w0 + 64 + l
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int w = w0 + 64 * h + lane;
        if (w < w1) { word[2 * h] = keep[2 * w]; word[2 * h + 1] = 2 * w + 1 < (P + 31) / 32 ? keep[2 * w + 1] : 0u; }
    }
    int at = __builtin_amdgcn_readfirstlane(sum_before(__popc(word[0]) + __popc(word[1]) + __popc(word[2]) + __popc(word[3]), swave));
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int n = min(w1 - w0 - 64 * h, 64);
        for (int u0 = 0; u0 < n; u0 += 4) {                  // four words at a time: a word's chain of scalar and vector steps is all latency
            uint32_t lo[4], hi[4];
            int e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                lo[u] = __builtin_amdgcn_readlane(word[2 * h], (u0 + u) & 63);
                hi[u] = __builtin_amdgcn_readlane(word[2 * h + 1], (u0 + u) & 63);     // (words past the last are 0)
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                e[u] = at + (int)__builtin_amdgcn_mbcnt_hi(hi[u], __builtin_amdgcn_mbcnt_lo(lo[u], 0u));
                at += __popc(lo[u]) + __popc(hi[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (__builtin_amdgcn_inverse_ballot_w64(lo[u] | ((unsigned long long)hi[u] << 32))) {
                    const uint32_t j = 64u * (uint32_t)(w0 + 64 * h + u0 + u) + (uint32_t)lane, off = 4u * (uint32_t)e[u];
                    *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(idx) + off) = j;
                    *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(list) + off) = j;
                }
        }
    }
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Slabs of 32 window rows score_pass covers: 1, 2 or 4.  0: more rows than it takes.
int n_row_slabs(int rows) {
    const int slabs = (rows + kRowsPerWave - 1) / kRowsPerWave;
    return rows > kNarrowRows ? 0 : slabs <= 1 ? 1 : slabs == 2 ? 2 : 4;
}

// merging: the vote pass that merges the row statistics itself, or NULL
template <class Counts>
hipError_t launch_scores(void (*stats_pass)(const ScoreArgs, const Counts), void (*vote_pass)(const ScoreArgs, const NoCounts), void (*merging)(const ScoreArgs, const NoCounts),
                         const ScoreArgs& a, const Counts& counts, int n_wg, int heads, hipStream_t stream) {
    hipLaunchKernelGGL(stats_pass, dim3(n_wg, heads), dim3(kThreads), 0, stream, a, counts);
    const bool merge = merging && a.n_parts <= kMergeParts;
    if (!merge)
        hipLaunchKernelGGL(stats_combine, dim3(heads, (a.rows_pad + 3) / 4), dim3(256), 0, stream, (const float2*)a.stats_part, a.stats, a.zsum,
                           a.n_parts, a.rows_pad);
    hipLaunchKernelGGL((merge ? merging : vote_pass), dim3(n_wg, heads), dim3(kThreads), 0, stream, a, NoCounts{});
    return hipGetLastError();
}

}  // namespace

CompressPlan plan_compress(const kvqp_cfg& cfg) {
    CompressPlan p{};
    p.P = cfg.seq_len - cfg.window;
    p.n_kept = cfg.budget < p.P ? cfg.budget : p.P;
    p.rows = (cfg.n_q_heads / cfg.n_kv_heads) * cfg.window;
    const int nrw = n_row_slabs(p.rows), heads = cfg.batch * cfg.n_kv_heads;
    const bool wide = nrw == 0;
    p.rows_pad = wide ? kWideRows : nrw * kRowsPerWave;
    p.n_chunks = (cfg.seq_len + 63) / 64;                // keys per chunk: 64
    // A workgroup pays for staging its query rows and waits for its first keys alone, so it should have
    // sixteen chunks (64 where the wave holds more rows), as long as that leaves two workgroups per CU;
    // beyond eight per CU more only cost.  Statistics + votes, us, with 512 / 1024 / 2048 workgroups: 8
    // heads of 32768 keys 18.4 + 14.8 / 19.5 + 16.2 / 22.0 + 17.3; 32 heads of 16384 29 + 26, 64 heads 55 + 46 and
    // 128 heads 100 + 92 with any of them; with 256 rows 8 heads of 131072 keys 87 + 78 / 88 + 79.
    auto workgroups = [&](int n_chunks, int& share) {
        const int total = (int)std::min(2048LL, std::max(512LL, (long long)heads * n_chunks / (wide ? 64 : 16)));
        const int least = wide ? 4 : 2;
        int n_wg = (total + heads - 1) / heads;
        if (n_wg > (n_chunks + least - 1) / least) n_wg = (n_chunks + least - 1) / least;
        if (n_wg < 1) n_wg = 1;
        share = (n_chunks + n_wg - 1) / n_wg;
        return (n_chunks + share - 1) / share;
    };
    p.n_wg = workgroups(p.n_chunks, p.chunks_per_wg);
    if (nrw == 1 || nrw == 2) {
        // (Never more statistics than chunks of 128 keys with one per key strip, four or two to a workgroup, would leave: a
        // workspace of the size that was once stated for those is taken.)
        int share;
        const int most = 4 / nrw * workgroups((cfg.seq_len + 127) / 128, share);
        while (p.n_wg > most) { ++p.chunks_per_wg; p.n_wg = (p.n_chunks + p.chunks_per_wg - 1) / p.chunks_per_wg; }
    }
    p.n_parts = p.n_wg;
    p.takes_counts = heads <= kCountsInStats;
    const int rows_pad = p.rows_pad;
    const size_t n_parts = (size_t)p.n_parts;
    size_t off = 0;
    // pooling workgroups per head: enough to fill the chip, whole pooling tiles each
    const int tiles = p.P > 0 ? (p.P + kPoolTile - 1) / kPoolTile : 1;
    const bool apart = tiles > kOwnTiles;                // pooled by pool_scores: codes, counts and pooled scores pass through memory
    int segs = (512 + heads - 1) / heads;
    if (segs > kMaxSegs) segs = kMaxSegs;
    if (segs > tiles) segs = tiles;
    p.seg_tiles = (tiles + segs - 1) / segs;
    if (p.seg_tiles > kMaxSegTiles) p.seg_tiles = kMaxSegTiles;
    p.n_seg = (tiles + p.seg_tiles - 1) / p.seg_tiles;
    p.p_stride = p.P > 0 ? (p.P + 7) / 8 * 8 : 8;
    // (the row statistics of the scoring workgroups are dead when the pooled scores are counted)
    const size_t part_bytes = (size_t)heads * n_parts * rows_pad * sizeof(float2);
    const size_t bins_bytes = apart ? (size_t)heads * p.n_seg * kBinRow * sizeof(uint16_t) : 0;
    p.off_stats_part = off; off = align_up(off + (part_bytes > bins_bytes ? part_bytes : bins_bytes), 256);
    p.off_stats = off;      off = align_up(off + (size_t)heads * rows_pad * (sizeof(float2) + sizeof(double)), 256);
    p.off_vote = off;       off = align_up(off + (size_t)heads * (p.P > 0 ? p.P : 1) * sizeof(float), 256);
    p.off_pooled = off;     off = align_up(off + (apart ? (size_t)heads * p.p_stride * sizeof(uint16_t) : 0), 256);
    p.off_idx = off;        off = align_up(off + (size_t)heads * (p.n_kept > 0 ? p.n_kept : 1) * sizeof(int32_t), 256);
    p.total = off;
    p.exact_bytes = apart ? (size_t)heads * p.p_stride * sizeof(float) : 0;
    return p;
}

hipError_t launch_select(const kvqp_cfg& cfg, const void* q_obs, const void* k, int32_t* idx, int32_t* list, int32_t* unrefined, void* ws,
                         const CompressPlan& plan, const int32_t* head_n, bool score, hipStream_t stream) {
    char* base = static_cast<char*>(ws);
    const int heads = cfg.batch * cfg.n_kv_heads;
    const int n_wg = plan.n_wg;

    ScoreArgs a;
    a.q_obs = (const uint16_t*)q_obs; a.k = (const uint16_t*)k;
    a.stats_part = reinterpret_cast<float2*>(base + plan.off_stats_part);
    float2* stats = reinterpret_cast<float2*>(base + plan.off_stats);
    a.rows = plan.rows; a.rows_pad = plan.rows_pad;
    double* zsum = reinterpret_cast<double*>(base + plan.off_stats + (size_t)heads * a.rows_pad * sizeof(float2));
    a.stats = stats; a.zsum = zsum;
    a.vote = reinterpret_cast<float*>(base + plan.off_vote);
    a.L = cfg.seq_len; a.W = cfg.window; a.P = plan.P; a.gq = cfg.n_q_heads / cfg.n_kv_heads;
    a.n_q_heads = cfg.n_q_heads; a.n_kv_heads = cfg.n_kv_heads;
    a.chunks_per_wg = plan.chunks_per_wg; a.n_chunks = plan.n_chunks; a.n_parts = plan.n_parts;
    a.scale_log2 = cfg.sm_scale * kLog2e;
    a.stream_heads = std::max(0, heads - (int)(kSideCache / ((size_t)cfg.seq_len * kHeadDim * 2)));

    hipError_t e;
    if (score) {   // scores are needed only when something is dropped
        constexpr void (*none)(const ScoreArgs, const NoCounts) = nullptr;
        const int slabs = n_row_slabs(plan.rows);
        auto aligned = [&](const auto& counts) {
            using Counts = std::decay_t<decltype(counts)>;
            switch (slabs) {
                case 1: return launch_scores(score_pass<1, PASS_STATS, false, true, Counts>, score_pass<1, PASS_VOTES>, score_pass<1, PASS_VOTES, true>, a, counts, n_wg, heads, stream);
                case 2: return launch_scores(score_pass<2, PASS_STATS, false, true, Counts>, score_pass<2, PASS_VOTES>, score_pass<2, PASS_VOTES, true>, a, counts, n_wg, heads, stream);
                case 4: return launch_scores(score_pass<4, PASS_STATS, false, true, Counts>, score_pass<4, PASS_VOTES>, score_pass<4, PASS_VOTES, true>, a, counts, n_wg, heads, stream);
                default: return launch_scores(score_wide<PASS_STATS, true, Counts>, score_wide<PASS_VOTES>, none, a, counts, n_wg, heads, stream);
            }
        };
        if ((uintptr_t)k & 15) {      // (whole calls, us, 8 heads: 4096 keys 28.5 instead of 25.5, 32768 75.7 / 76.0, 131072 with 256 rows 239.6 / 237.1)
            if (plan.counts && (e = upload_counts(plan.counts_dst, plan.counts, heads, stream)) != hipSuccess) return e;
            switch (slabs) {
                case 1: e = launch_scores(score_pass<1, PASS_STATS, false, false>, score_pass<1, PASS_VOTES, false, false>, none, a, NoCounts{}, n_wg, heads, stream); break;
                case 2: e = launch_scores(score_pass<2, PASS_STATS, false, false>, score_pass<2, PASS_VOTES, false, false>, none, a, NoCounts{}, n_wg, heads, stream); break;
                case 4: e = launch_scores(score_pass<4, PASS_STATS, false, false>, score_pass<4, PASS_VOTES, false, false>, none, a, NoCounts{}, n_wg, heads, stream); break;
                default: e = launch_scores(score_wide<PASS_STATS, false>, score_wide<PASS_VOTES, false>, none, a, NoCounts{}, n_wg, heads, stream); break;
            }
        } else if (plan.counts) {
            HeadCounts counts;
            counts.dst = plan.counts_dst;
            for (int i = 0; i < kCountsInStats; ++i) counts.v[i] = i < heads ? plan.counts[i] : 0;
            e = aligned(counts);
        } else {
            e = aligned(NoCounts{});
        }
        if (e != hipSuccess) return e;
    }
    SelectArgs s;
    s.vote = a.vote; s.code = reinterpret_cast<uint16_t*>(base + plan.off_pooled); s.idx = idx; s.list = list; s.unrefined = unrefined; s.head_n = head_n;
    s.q_obs = a.q_obs; s.k = a.k; s.stats = stats; s.zsum = zsum;
    s.P = plan.P; s.L = cfg.seq_len; s.W = cfg.window; s.n_kept = plan.n_kept; s.pool = cfg.pool_kernel;
    s.gq = a.gq; s.n_q_heads = cfg.n_q_heads; s.n_kv_heads = cfg.n_kv_heads; s.rows = a.rows; s.rows_pad = a.rows_pad;
    s.sm_scale = cfg.sm_scale; s.w_recip = (65536u + (uint32_t)cfg.window - 1u) / (uint32_t)cfg.window;
    s.bins = reinterpret_cast<uint16_t*>(base + plan.off_stats_part);
    s.exact = plan.exact_bytes > 0 ? reinterpret_cast<float*>(base + plan.total) : nullptr;
    s.p_stride = plan.p_stride; s.n_seg = plan.n_seg; s.seg_tiles = plan.seg_tiles;
    const int octs = (plan.P + 7) / 8, shares = (octs + kSelThreads - 1) / kSelThreads;       // (sweeping workgroups of a head, kSpread)
    s.share_oct = ((octs + shares - 1) / std::max(shares, 1) + 7) / 8 * 8;
    auto own = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(1, heads), dim3(kSelThreads), 0, stream, s); };
    // Up to three pooling tiles per workgroup: the launch before it and the codes' way through memory are worth more than
    // the workgroups that pool side by side (whole calls, us, two kernels -> one: 8 heads of 8192 keys 41.3 -> 35.1, of 12000 43.7 ->
    // 38.9, 32 heads 68.8 -> 62.1 and 88.5 -> 84.5, 128 heads 184.6 -> 177.5 and 241.7 -> 239.2).  From four on the votes, four
    // bytes each through one CU, take longer: 8 heads of 16384 keys 51.1 -> 52.3, of 20000 60.3 -> 65.7, 32 heads 117.4 -> 118.9.
    static_assert(kOwnTiles == 3, "a kernel for each");
    if (plan.P <= kPoolTile) own(select_topk<1>);
    else if (plan.P <= 2 * kPoolTile) own(select_topk<2>);
    else if (plan.P <= kOwnTiles * kPoolTile) own(select_topk<kOwnTiles>);
    else {
        if (score) hipLaunchKernelGGL(pool_scores, dim3(plan.n_seg, heads), dim3(kSelThreads), 0, stream, s);
        if (shares > kAloneShares && heads * shares <= kMostShares) hipLaunchKernelGGL(select_topk<kSpread>, dim3(shares, heads), dim3(kSelThreads), 0, stream, s);
        else own(select_topk<kAlone>);
    }
    return hipGetLastError();
}

}  // namespace kvqp
