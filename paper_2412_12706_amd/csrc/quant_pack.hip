// Gather the surviving tokens, quantize them group by group and write the
// packed cache (paper Section 3, "KV Quantization": z = min, m = max,
// s = (m - z)/(2^B - 1), Q(G) = round((G - z)/s); grouping axes of Section 2 /
// Section 6.3).  Every survivor row is read once (2 x 256 B, scattered) and
// k*bpt bytes are written; there is no reuse to exploit.  What bounds it on
// the MI355X: vector-instruction issue at 2 and 4 bits (the vector ALUs were
// busy all the time at 1090 instructions per thread for 64 elements), then
// memory.  So an element costs five: v_fma_mix_f32 (widen and subtract z),
// multiply, round, clamp, and a multiply-add that puts its field into the word
// as a whole number in binary32; order keys take two instructions per pair, and
// every lane exchange merges two registers into one.  256 heads, 16384 of 32768
// tokens at 2 bits: 510 -> 453 us (2.55 GB: 5.6 TB/s); 8 heads, 8192 tokens at
// 4 bits: 15.7 -> 12.5 us; 16384 tokens at 2 bits in groups of 64: 22 -> 19 us.
//
// One workgroup owns TB consecutive kept tokens of one (batch, kv head): whole
// key groups (G | TB) and whole value superblocks (SB | TB).  Thread
// (r = tid / 16, c8 = tid % 16) keeps channels 8 c8 .. 8 c8 + 7 of rows
// r, r + 16, r + 32, ... in registers from the gather to the packed words:
//   * minima / maxima are taken on packed 16-bit order keys (two channels per
//     register), across lanes with DPP / permlane exchanges and across waves
//     through a few KB of LDS;
//   * key words are assembled in registers and stored straight from them
//     (a word holds consecutive channels of one token);
//   * value words hold one channel of several tokens (the tile-transposed
//     layout of kvqp.h): wave kb owns tokens 4 kb + i, lanes OR their fields
//     together, and the finished superblocks leave through LDS as 16-byte
//     coalesced stores.
#include "kvqp_internal.h"

namespace kvqp {
namespace {

constexpr int kThreads = 256;
constexpr uint32_t kBlockCount = 0x80000000u;   // overflow prefix array, until ovf_fill has been there: a block's own count

// One launch of the quantize-and-pack kernel: n_tok rows per head of (k, v) -- rows idx[...] or, with
// idx == NULL, rows 0 .. n_tok-1 -- land at tokens dst_base .. of a cache laid out for n_cap tokens.
struct QuantPackJob {
    const kvqp_cache& c;
    const void* k; const void* v; const int32_t* idx;
    const int32_t* head_n;   // device: rows of each head (<= n_tok, whole groups), or NULL for n_tok everywhere
    uint32_t tau_bits;       // outlier filtering: |x| is above the threshold iff its binary16 pattern exceeds this
    bool outliers;
    int heads, src_rows, window, n_tok, dst_base, n_cap, bits, group_size, key_axis;
    bool copy_tail;
    const int32_t* head_base = nullptr;   // device: first destination token of each head in place of dst_base, or NULL
    int base_quantum = 1;                 // what every head_base entry is a multiple of
    int ovf_cap = 0;                      // outlier filtering: entries of a head's overflow list
    int tail_len = 0;                     // > 0: the rows come from the front of a tail of that many, which is to close up
};

// Whether the quantizer itself closes the tail up: one workgroup has all of a head's rows and nothing reads them after it.
constexpr int quant_tokens(int bits, int group) { return (bits != 16 && group == 128) ? 128 : 64; }   // per workgroup
bool closes_tail(const QuantPackJob& j) { return j.n_tok <= quant_tokens(j.bits, j.group_size) && !j.outliers; }

typedef unsigned short us2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
    union { uint32_t u; us2v v; } x, y, z; x.u = a; y.u = b; z.v = __builtin_elementwise_min(x.v, y.v); return z.u;
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
    union { uint32_t u; us2v v; } x, y, z; x.u = a; y.u = b; z.v = __builtin_elementwise_max(x.v, y.v); return z.u;
}

// 1 in the half-words of a that exceed b's
__device__ __forceinline__ uint32_t pk_above(uint32_t a, uint32_t b) {
    union { uint32_t u; us2v v; } x, y; x.u = a; y.u = b;
    x.v = __builtin_elementwise_min(__builtin_elementwise_sub_sat(x.v, y.v), us2v{1, 1});
    return x.u;
}

// binary16 bit patterns -> keys that order like the values (-0 below +0), on both halves of a word:
// negative halves inverted, the others with the sign bit set (two instructions)
typedef short ss2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t order_key2(uint32_t w) {
    union { uint32_t u; ss2v v; } t;
    t.u = w;
    t.v = t.v >> (short)15;
    return w ^ (t.u | 0x80008000u);
}
__device__ __forceinline__ uint16_t key_to_half(uint32_t key) { return (key & 0x8000u) ? (uint16_t)(key & 0x7fffu) : (uint16_t)~key; }
__device__ __forceinline__ float half_bits_to_float(uint16_t h) { return __half2float(__ushort_as_half(h)); }

// The quantizer's binary32 sequence; every operation individually rounded.
struct GroupParams {
    uint16_t scale_h, zero_h;
    float zf, inv;   // inv == 0 marks the degenerate group (all codes 0)
};
template <int BITS>
__device__ __forceinline__ GroupParams group_params(uint32_t kmin, uint32_t kmax) {
    GroupParams g;
    g.zero_h = key_to_half(kmin);
    const uint16_t mh = key_to_half(kmax);
    g.zf = half_bits_to_float(g.zero_h);
    const float r = __fsub_rn(half_bits_to_float(mh), g.zf);
    const float s32 = __fdiv_rn(r, (float)((1 << BITS) - 1));
    const __half sh = __float2half_rn(s32);
    g.scale_h = __half_as_ushort(sh);
    const float sf = __half2float(sh);
    g.inv = (sf == 0.0f) ? 0.0f : __fdiv_rn(1.0f, sf);
    return g;
}
// The code of one element, as a float: the words are put together by multiply-adds (field_sum).
// one is 1.0f that the compiler does not know: x * one - z is the widening and the subtraction in one
// instruction (v_fma_mix_f32; the product is exact, so the difference is rounded once, as a subtraction is).
template <int BITS>
__device__ __forceinline__ float encode(uint16_t xh, float zf, float inv, float one) {
    // a degenerate group needs no branch: (x - z) * 0 rounds and clamps to code 0
    const float c = rintf(__fmul_rn(__builtin_fmaf(half_bits_to_float(xh), one, -zf), inv));
    return fminf(fmaxf(c, 0.0f), (float)((1 << BITS) - 1));
}
// c + 2^SHIFT * hi: fields of whole numbers side by side, exact while the sum stays below 2^24
template <int SHIFT> __device__ __forceinline__ float field_sum(float c, float hi) { return __builtin_fmaf(hi, (float)(1 << SHIFT), c); }

template <int CTRL> __device__ __forceinline__ uint32_t dpp(uint32_t v) { return __builtin_amdgcn_update_dpp(0u, v, CTRL, 0xF, 0xF, true); }
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kRowHalfMirror = 0x141, kRowMirror = 0x140;

// one of four values by a lane's number 0 .. 3 (by value: a choice among array elements becomes branches)
__device__ __forceinline__ uint32_t pick(int i, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    asm("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
    const uint32_t lo = (i & 1) ? b : a, hi = (i & 1) ? d : c;
    return (i & 2) ? hi : lo;
}

// min / max over the LANES consecutive lanes (4, 8 or 16) that share a per-token group
template <int LANES> __device__ __forceinline__ void group_minmax(uint32_t& mn, uint32_t& mx) {
    mn = min(mn, dpp<kQuadXor1>(mn)); mx = max(mx, dpp<kQuadXor1>(mx));
    mn = min(mn, dpp<kQuadXor2>(mn)); mx = max(mx, dpp<kQuadXor2>(mx));
    if (LANES >= 8) { mn = min(mn, dpp<kRowHalfMirror>(mn)); mx = max(mx, dpp<kRowHalfMirror>(mx)); }
    if (LANES >= 16) { mn = min(mn, dpp<kRowMirror>(mn)); mx = max(mx, dpp<kRowMirror>(mx)); }
}

// c, or 0 where the mask is set
__device__ __forceinline__ float without(float c, uint32_t mask) { return __uint_as_float(__float_as_uint(c) & ~mask); }

// codes of a thread's eight channels of one row
template <int BITS>
__device__ __forceinline__ void encode8(const uint32_t (&w)[4], const float (&zf)[8], const float (&inv)[8], float one, float (&c)[8]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        c[2 * q] = encode<BITS>((uint16_t)(w[q] & 0xffffu), zf[2 * q], inv[2 * q], one);
        c[2 * q + 1] = encode<BITS>((uint16_t)(w[q] >> 16), zf[2 * q + 1], inv[2 * q + 1], one);
    }
}

// the same when all eight channels share one group
template <int BITS>
__device__ __forceinline__ void encode8(const uint32_t (&w)[4], float zf, float inv, float one, float (&c)[8]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        c[2 * q] = encode<BITS>((uint16_t)(w[q] & 0xffffu), zf, inv, one);
        c[2 * q + 1] = encode<BITS>((uint16_t)(w[q] >> 16), zf, inv, one);
    }
}

// Key words of one row from the thread's eight codes (row-major layout of kvqp.h: channel d sits in
// word d / E at half-word r % 2, field r / 2, r = d % E) and their store, at words row .. of kc.
// keep: all ones, or 0 for a padding row (its words are stored as zeros).
template <int BITS>
__device__ __forceinline__ void store_key_words(uint32_t* kc, uint32_t row, int c8, const float (&c)[8], uint32_t keep = 0xFFFFFFFFu) {
    constexpr int E = 32 / BITS;
    if constexpr (E == 8) {   // four fields per half-word
        float half[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) half[h] = field_sum<8>(field_sum<4>(c[h], c[2 + h]), field_sum<4>(c[4 + h], c[6 + h]));
        kc[row + (uint32_t)c8] = ((uint32_t)half[0] | ((uint32_t)half[1] << 16)) & keep;
    } else if constexpr (E == 4) {   // two fields per half-word, two words
        uint32_t w[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
            w[u] = ((uint32_t)field_sum<8>(c[4 * u], c[4 * u + 2]) | ((uint32_t)field_sum<8>(c[4 * u + 1], c[4 * u + 3]) << 16)) & keep;
        *reinterpret_cast<uint2*>(kc + (row + 2u * (uint32_t)c8)) = make_uint2(w[0], w[1]);
    } else {   // E == 16: the word spans this lane's channels and its neighbour's; four of eight fields per half-word, sum < 2^24
        float half[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) half[h] = field_sum<4>(field_sum<2>(c[h], c[2 + h]), field_sum<2>(c[4 + h], c[6 + h]));
        uint32_t w = (uint32_t)field_sum<16>(half[0], half[1]);
        // odd lanes hold channels 8..15 of the word: fields 4..7 of each half-word
        if (c8 & 1) w <<= 4 * BITS;
        w |= dpp<kQuadXor1>(w);
        if (!(c8 & 1)) kc[row + (uint32_t)(c8 >> 1)] = w & keep;
    }
}

// sum over the 16 lanes of a row, in every lane; and the sum over the lanes before this one
__device__ __forceinline__ uint32_t row16_sum(uint32_t v) {
    v += dpp<kQuadXor1>(v); v += dpp<kQuadXor2>(v); v += dpp<kRowHalfMirror>(v); v += dpp<kRowMirror>(v);
    return v;
}
__device__ __forceinline__ uint32_t row16_before(uint32_t v) {
    uint32_t s = v;
    s += dpp<0x111>(s); s += dpp<0x112>(s); s += dpp<0x114>(s); s += dpp<0x118>(s);   // row_shr 1, 2, 4, 8 (zeros shifted in)
    return s - v;
}
// all ones where the bit is set
__device__ __forceinline__ uint32_t bit_mask(uint32_t bits, int bit) { return (uint32_t)__builtin_amdgcn_sbfe((int)bits, (unsigned)bit, 1u); }
// 0xFFFF in the half-words whose bit (bit: low half, bit + 1: high half) is set
__device__ __forceinline__ uint32_t half_mask(uint32_t bits, int bit) { return (bit_mask(bits, bit) & 0xFFFFu) | (bit_mask(bits, bit + 1) & 0xFFFF0000u); }

// Rows [n_shift, tail_len) of both tail tensors of a head move down to [0, tail_len - n_shift).  One
// workgroup; 16 rows per round go through registers (all reads of a round before its writes, rounds
// in ascending order, so overlapping ranges are safe).
__device__ __forceinline__ void close_tail(uint16_t* tail_k, uint16_t* tail_v, int head, int tail_cap, int n_shift, int tail_len) {
    uint16_t* tk = tail_k + (size_t)head * tail_cap * kHeadDim;
    uint16_t* tv = tail_v + (size_t)head * tail_cap * kHeadDim;
    const int r = threadIdx.x >> 4, c8 = threadIdx.x & 15;
    for (int r0 = n_shift; r0 < tail_len; r0 += 16) {
        const int row = r0 + r;
        const bool live = row < tail_len;
        uint4 a = make_uint4(0, 0, 0, 0), b = a;
        if (live) {
            a = *reinterpret_cast<const uint4*>(tk + (size_t)row * kHeadDim + 8 * c8);
            b = *reinterpret_cast<const uint4*>(tv + (size_t)row * kHeadDim + 8 * c8);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (the barrier alone does not wait for loads in flight)
        __syncthreads();
        if (live) {
            *reinterpret_cast<uint4*>(tk + (size_t)(row - n_shift) * kHeadDim + 8 * c8) = a;
            *reinterpret_cast<uint4*>(tv + (size_t)(row - n_shift) * kHeadDim + 8 * c8) = b;
        }
        __syncthreads();
    }
}

// Waves per SIMD the registers have to allow: as many as they do without spilling (other workgroups hide
// one's waits: at three waves instead of six the former code was 35 % slower).
constexpr int quant_waves(int bits, int group, bool out) {
    return out ? (group == 128 ? 3 : 5) : group == 128 ? 4 : bits == 2 && group == 32 ? 7 : 8;
}

template <int BITS, int G, bool OUT>
__global__ __launch_bounds__(kThreads, quant_waves(BITS, G, OUT)) void gather_quant_pack(
    const uint16_t* k, const uint16_t* v, const int32_t* __restrict__ idx,
    uint32_t* __restrict__ k_codes, uint32_t* __restrict__ v_codes, uint16_t* __restrict__ k_scale,
    uint16_t* __restrict__ k_zero, uint16_t* __restrict__ v_scale, uint16_t* __restrict__ v_zero,
    uint16_t* tail_k, uint16_t* tail_v, int L, int W, int n_kept, int key_axis,
    int tail_cap, int n_tok_blocks, int n_cap, int dst_base, const int32_t* __restrict__ head_n,
    uint32_t* __restrict__ k_out, uint32_t* __restrict__ v_out, uint32_t tau_bits,
    const int32_t* __restrict__ head_base, int base_quantum, uint32_t* __restrict__ k_ovf,
    uint32_t* __restrict__ v_ovf, int ovf_cap, int tail_len) {
    // (k / v may be the tail itself: neither is a restrict pointer.)
    // L: rows per head of the source tensors.  idx: source row of every token of this call
    // ([heads, n_kept]), or NULL for rows 0 .. n_kept-1.  The tokens land at positions dst_base ..
    // dst_base + n_kept - 1 of a cache whose buffers are laid out for n_cap tokens per head.
    // head_n: a head's own token count in place of n_kept (idx keeps its stride of n_kept), or NULL.
    // head_base: a head's own first position in place of dst_base, or NULL; it is cut to dst_base and
    // rounded down to a multiple of base_quantum, so whatever the array holds the stores stay inside
    // the buffers and on group and superblock boundaries.
    // tail_len > 0: the source rows are the oldest of tail_len tail rows and one workgroup takes all of a
    // head's; it closes the tail up when it is done with them.
    // OUT: outlier filtering; k_out / v_out receive four slot words per token row, and the number of
    // a block's further outliers is left at entry (block + 1) of the head's overflow prefix array
    // (k_ovf / v_ovf), which ovf_fill turns into prefix counts before it writes the entries.
    constexpr bool QUANT = BITS != 16;
    constexpr int TB = quant_tokens(BITS, G);            // tokens per workgroup
    constexpr int R = TB / 16;                            // rows per thread
    constexpr int NG = TB / G > 0 ? TB / G : 1;           // per-channel key groups per workgroup
    constexpr int JPG = G / 16;                           // a thread's rows per key group
    constexpr int CPT = kHeadDim / G;                     // per-token groups per row
    constexpr int GL = G / 8;                             // lanes per per-token group
    constexpr int E = 32 / BITS;
    constexpr int SB = v_superblock(BITS);
    constexpr int WPT = v_words_per_tile(BITS);
    constexpr int SBW = v_superblock_words(BITS);
    constexpr int NSB = TB / SB;
    __shared__ __align__(16) uint32_t s_words[NSB * SBW];                 // finished value superblocks
    __shared__ __align__(16) uint16_t s_min[QUANT ? 4 * NG * kHeadDim : 8];   // per wave: channel minima (order keys) / maxima (inverted)
    __shared__ __align__(16) uint16_t s_max[QUANT ? 4 * NG * kHeadDim : 8];
    __shared__ __align__(16) float2 s_par[QUANT ? NG * kHeadDim : 1];     // (z, 1/s) per (key group, channel)
    __shared__ int s_cnt[2][OUT ? TB / 32 : 1];                           // OUT: outliers beyond the slots per 32-token block (keys, values)

    const int head = blockIdx.y;
    const uint16_t* kh = k + (size_t)head * L * kHeadDim;
    const uint16_t* vh = v + (size_t)head * L * kHeadDim;

    if ((int)blockIdx.x >= n_tok_blocks) {
        // Tail: the last W prompt rows stay at full precision.
        const int P = L - W;
        for (int item = threadIdx.x; item < W * 16; item += kThreads) {
            const int t = item >> 4, c = item & 15;
            const size_t src = (size_t)(P + t) * kHeadDim + c * 8, dst = ((size_t)head * tail_cap + t) * kHeadDim + c * 8;
            *reinterpret_cast<uint4*>(tail_k + dst) = *reinterpret_cast<const uint4*>(kh + src);
            *reinterpret_cast<uint4*>(tail_v + dst) = *reinterpret_cast<const uint4*>(vh + src);
        }
        return;
    }

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c8 = threadIdx.x & 15, r = threadIdx.x >> 4, i4 = (threadIdx.x >> 4) & 3;
    const int t0 = blockIdx.x * TB;
    int base = dst_base;
    if (head_base) {
        base = min(max(head_base[head], 0), dst_base);
        base -= base % base_quantum;
    }
    const int d0 = base + t0;                // first destination token: a multiple of the group and superblock sizes
    const int n_head = head_n ? head_n[head] : n_kept;
    if (t0 >= n_head) return;                // (the whole workgroup: nothing of this head left)
    const int ntok = min(TB, n_head - t0);   // any count: the head's last block and last key group may be partly filled
    const int ntok_pad = rows32(ntok);       // rows of the last block past the count are written as zeros
    if constexpr (OUT) {
        if (threadIdx.x < 2 * (TB / 32)) (&s_cnt[0][0])[threadIdx.x] = 0;
        __syncthreads();
    }

    // ---- gather: all of the thread's rows of both tensors are requested before anything is used.
    // The row numbers come first, all of them, and then every row load leaves without waiting for
    // another (two round trips to memory instead of one per row); a row past the count reads the
    // block's last row instead, so no load depends on a branch, and is cleared afterwards. ----
    // (Addresses here and below: a base that is the same for the workgroup and 32 bits per lane.)
    uint32_t kw[R][4], vw[R][4];
    bool live[R];
    uint32_t pos[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        live[j] = r + 16 * j < ntok;      // (the same for the 16 lanes of a token row)
        pos[j] = (uint32_t)min(r + 16 * j, ntok - 1);
    }
    const uint16_t *kb = kh, *vb = vh;
    if (idx) {                            // (uniform; rows of a prompt: below 2^18)
        const int32_t* rows = idx + (size_t)head * n_kept + t0;
#pragma unroll
        for (int j = 0; j < R; ++j) pos[j] = (uint32_t)rows[pos[j]];
    } else {
        kb += (size_t)t0 * kHeadDim;
        vb += (size_t)t0 * kHeadDim;
    }
    // (Keys first, all of them: they are worked on while the values are on their way; whole calls, us, keys and values in turn -> this:
    // 8 heads of 4096 tokens 23.6 -> 23.25, of 32768 65.1 -> 64.7, 131072 213.0 -> 212.3.  Prompt rows are read once: non-temporal.)
    auto gather = [&](const uint16_t* base, uint32_t (&w)[R][4]) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            typedef uint32_t u4v __attribute__((ext_vector_type(4)));
            const u4v a = __builtin_nontemporal_load(reinterpret_cast<const u4v*>(base + (pos[j] * kHeadDim + 8u * c8)));
            w[j][0] = a[0]; w[j][1] = a[1]; w[j][2] = a[2]; w[j][3] = a[3];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    gather(kb, kw);
    gather(vb, vw);
    if (ntok < TB) {                      // (uniform) the head's last block: rows past the count are zeros
        // (but a copy of the last row leaves the minima and maxima of per-channel groups alone)
        const bool clear_k = !QUANT || OUT || key_axis != KVQP_KEY_PER_CHANNEL;
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (!live[j]) {
#pragma unroll
                for (int q = 0; q < 4; ++q) { kw[j][q] = clear_k ? 0u : kw[j][q]; vw[j][q] = 0u; }
            }
    }

    // Outlier marking (OUT): om gets a bit per own element whose magnitude is above the threshold --
    // every such element of the row is an outlier (Section 6.3 item (1): no limit per row).
    auto mark = [&](const uint32_t (&w)[R][4], uint32_t (&om)[R]) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            uint32_t cand = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) cand |= pk_above(w[j][q] & 0x7fff7fffu, tau_bits * 0x10001u) << (2 * q);
            om[j] = (cand | (cand >> 15)) & 0xffu;
        }
    };
    // slot word of element x (binary16 pattern) in channel ch given its group's zero
    auto slot_word = [](uint32_t xh, uint32_t ch, float zf) -> uint32_t {
        const float diff = __fsub_rn(half_bits_to_float((uint16_t)xh), zf);
        return (__float_as_uint(diff) & 0xFFFFFF00u) | 0x80u | ch;
    };
    // Slot words of the rows: an outlier's index is the number of outliers before it in the row
    // (lanes before this one, then the lane's own earlier elements); the first four go to the row's
    // slots in that (ascending channel) order, lanes 0-3 of the row clear the unused slots.  Outliers
    // beyond the fourth belong to the head's overflow list, which a later kernel fills; here they are
    // only counted per block of 32 tokens (cnt, in LDS).  zero_of(j, e): the zero of element e's group in row j.
    auto store_slots = [&](uint32_t* out, int* cnt, const uint32_t (&w)[R][4], const uint32_t (&om)[R], auto zero_of) {
        // (The counts of four rows go along the lanes together, a byte each: a row has 128 elements.  An outlier per lane and
        // round: lanes seldom have more than one.  With the eight elements tested in turn, and marks formed one element at a
        // time, 32 heads of 20011 tokens took 101.1 us in all instead of 99.8; the outliers of four rows in one loop 0.5 more.)
        uint32_t* rows = out + ((size_t)head * n_cap + d0) * 4;      // (one base for the workgroup, 32 bits per lane)
#pragma unroll
        for (int j4 = 0; j4 < R; j4 += 4) {
            uint32_t mine = 0u;
#pragma unroll
            for (int u = 0; u < 4; ++u) mine |= (uint32_t)__builtin_popcount(om[j4 + u]) << (8 * u);
            const uint32_t totals = row16_sum(mine), before = row16_before(mine);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = j4 + u;
                const uint32_t row = (uint32_t)(r + 16 * j) * 4u, total = (totals >> (8 * u)) & 0xffu;
                // slots without an outlier, and a padding row's
                if (c8 < 4 && r + 16 * j < ntok_pad && (!live[j] || (uint32_t)c8 >= total)) rows[row + c8] = 0u;
                if (c8 == 0 && live[j] && total > 4u) atomicAdd(&cnt[j >> 1], (int)(total - 4u));
                uint32_t at = (before >> (8 * u)) & 0xffu;
                for (uint32_t m = live[j] ? om[j] : 0u; __builtin_amdgcn_ballot_w64(m != 0u) != 0ull; m &= m - 1u)
                    if (m) {
                        const int e = __builtin_ctz(m);
                        const uint32_t xh = (pick(e >> 1, w[j][0], w[j][1], w[j][2], w[j][3]) >> (16 * (e & 1))) & 0xffffu;
                        if (at < 4u) rows[row + at] = slot_word(xh, (uint32_t)(8 * c8 + e), zero_of(j, e));
                        ++at;
                    }
            }
        }
    };

    float one = 1.0f;                     // (see encode)
    asm("" : "+s"(one));
    // Per-token groups (values always, keys on that axis): every row is complete inside GL lanes.
    // Hands the codes of every row to sink(row, codes) and stores scale / zero.  Lane q of a quad derives the parameters
    // of rows q, q + 4, ... and hands them to the other three.  om: outlier bits (OUT); zrow: float
    // bits of the zero of the lane's own group, per row.
    auto per_token = [&](const uint32_t (&w)[R][4], uint16_t* scale, uint16_t* zero, const uint32_t (&om)[R],
                         uint32_t (&zrow)[R], auto sink) {
        uint32_t mn[R], mx[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t a = order_key2(w[j][q]);
                const uint32_t ex = OUT ? half_mask(om[j], 2 * q) : 0u;   // excluded halves: neutral for min and max
                lo = pk_min(lo, a | ex); hi = pk_max(hi, a & ~ex);
            }
            mn[j] = min(lo & 0xffffu, lo >> 16); mx[j] = max(hi & 0xffffu, hi >> 16);
            group_minmax<GL>(mn[j], mx[j]);
            if (OUT && mn[j] > mx[j]) { mn[j] = 0x8000u; mx[j] = 0x8000u; }   // nothing left in the group: zero +0, scale 0
        }
        const int q4 = c8 & 3;
#pragma unroll
        for (int jj = 0; jj < R / 4; ++jj) {
            const uint32_t a = pick(q4, mn[4 * jj], mn[4 * jj + 1], mn[4 * jj + 2], mn[4 * jj + 3]);
            const uint32_t b = pick(q4, mx[4 * jj], mx[4 * jj + 1], mx[4 * jj + 2], mx[4 * jj + 3]);
            const GroupParams gp = group_params<BITS>(a, b);
            const int t = r + 16 * (4 * jj + q4);
            if (t < ntok_pad && (c8 & (GL - 1)) < 4) {               // (a padding row of the last block was loaded as zeros: scale 0, zero +0)
                const size_t first = ((size_t)head * n_cap + d0) * CPT;
                const uint32_t m = (uint32_t)(t * CPT + c8 / GL);
                (scale + first)[m] = gp.scale_h; (zero + first)[m] = gp.zero_h;
            }
            const uint32_t zb = __float_as_uint(gp.zf), ib = __float_as_uint(gp.inv);
            const uint32_t zq[4] = {dpp<0x00>(zb), dpp<0x55>(zb), dpp<0xAA>(zb), dpp<0xFF>(zb)};
            const uint32_t iq[4] = {dpp<0x00>(ib), dpp<0x55>(ib), dpp<0xAA>(ib), dpp<0xFF>(ib)};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float c[8];
                encode8<BITS>(w[4 * jj + u], __uint_as_float(zq[u]), __uint_as_float(iq[u]), one, c);
                zrow[4 * jj + u] = zq[u];
                if constexpr (OUT) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) c[e] = without(c[e], bit_mask(om[4 * jj + u], e));   // outliers: code 0
                }
                sink(4 * jj + u, c);
            }
        }
    };
    // ---------------- keys ----------------
    uint32_t* kc = k_codes + ((size_t)head * n_cap + d0) * (kHeadDim / E);   // first row of this workgroup
    uint32_t om[R], zrow[R];   // outlier bits of the tensor at hand (OUT); zero of the lane's own per-token group
#pragma unroll
    for (int j = 0; j < R; ++j) om[j] = 0u;
    if constexpr (OUT) mark(kw, om);
    if constexpr (!QUANT) {
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (r + 16 * j < ntok_pad)     // (rows past the count were loaded as zeros)
                *reinterpret_cast<uint4*>(kc + (uint32_t)((r + 16 * j) * (kHeadDim / 2) + 4 * c8)) = make_uint4(kw[j][0], kw[j][1], kw[j][2], kw[j][3]);
    } else if (key_axis == KVQP_KEY_PER_CHANNEL) {
        // minima / maxima per channel over the G tokens of a group: own rows, the four row lanes of
        // the wave (lane ^ 16, ^ 32), then the four waves through LDS
        // (the empty asm keeps the compiler from forming every word's order key ahead of the branch, for both axes)
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) asm("" : "+v"(kw[j][q]));
        uint32_t pmin[NG][4], pmax[NG][4];
#pragma unroll
        for (int ug = 0; ug < NG; ++ug)
#pragma unroll
            for (int q = 0; q < 4; ++q) { pmin[ug][q] = 0xffffffffu; pmax[ug][q] = 0u; }
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (!OUT || live[j]) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t a = order_key2(kw[j][q]);
                    const uint32_t ex = OUT ? half_mask(om[j], 2 * q) : 0u;
                    pmin[j / JPG][q] = pk_min(pmin[j / JPG][q], a | ex); pmax[j / JPG][q] = pk_max(pmax[j / JPG][q], a & ~ex);
                }
            }
        // Maxima go on as minima of the inverted keys, and every lane exchange merges two registers into one:
        // exchanged between neighbouring rows of 16 lanes, a minimum's and a maximum's register leave the even
        // rows with the one and the odd rows with the other; exchanged between the halves of the wave, the two
        // key groups' (or, with one group, two words') leave one to each half.
        uint32_t red[NG][4];
#pragma unroll
        for (int ug = 0; ug < NG; ++ug)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const auto x = __builtin_amdgcn_permlane16_swap(pmin[ug][q], ~pmax[ug][q], false, false);
                red[ug][q] = pk_min(x[0], x[1]);
            }
        uint16_t* s_red = lane & 16 ? s_max : s_min;
        if constexpr (NG == 2) {
            uint32_t g[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const auto x = __builtin_amdgcn_permlane32_swap(red[0][q], red[1][q], false, false);
                g[q] = pk_min(x[0], x[1]);
            }
            *reinterpret_cast<uint4*>(s_red + (wave * 2 + (lane >> 5)) * kHeadDim + 8 * c8) = make_uint4(g[0], g[1], g[2], g[3]);
        } else {
            uint32_t g[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const auto x = __builtin_amdgcn_permlane32_swap(red[0][q], red[0][2 + q], false, false);
                g[q] = pk_min(x[0], x[1]);
            }
            *reinterpret_cast<uint2*>(s_red + wave * kHeadDim + 8 * c8 + 4 * (lane >> 5)) = make_uint2(g[0], g[1]);
        }
        __syncthreads();
        for (int item = threadIdx.x; item < NG * kHeadDim; item += kThreads) {   // one (group, channel) each
            const int ug = item / kHeadDim, d = item % kHeadDim;
            uint32_t a = 0xffffu, b = 0xffffu;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                a = min(a, (uint32_t)s_min[(w * NG + ug) * kHeadDim + d]);
                b = min(b, (uint32_t)s_max[(w * NG + ug) * kHeadDim + d]);
            }
            b = 0xffffu - b;
            if (OUT && a > b) { a = 0x8000u; b = 0x8000u; }   // every token of the group is an outlier here: zero +0, scale 0
            const GroupParams gp = group_params<BITS>(a, b);
            s_par[item] = make_float2(gp.zf, gp.inv);
            if (ug * G < ntok) {
                const size_t first = ((size_t)head * ((n_cap + G - 1) / G) + d0 / G) * kHeadDim;
                (k_scale + first)[(uint32_t)item] = gp.scale_h; (k_zero + first)[(uint32_t)item] = gp.zero_h;
            }
        }
        __syncthreads();
#pragma unroll
        for (int ug = 0; ug < NG; ++ug) {
            float zf[8], inv[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 pr = *reinterpret_cast<const float4*>(&s_par[ug * kHeadDim + 8 * c8 + 2 * q]);
                zf[2 * q] = pr.x; inv[2 * q] = pr.y; zf[2 * q + 1] = pr.z; inv[2 * q + 1] = pr.w;
            }
#pragma unroll
            for (int jl = 0; jl < JPG && ug * JPG + jl < R; ++jl) {
                const int j = ug * JPG + jl;
                float c[8];
                encode8<BITS>(kw[j], zf, inv, one, c);
                if constexpr (OUT) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) c[e] = without(c[e], bit_mask(om[j], e));
                }
                // (padding rows of the last block hold code 0)
                if (r + 16 * j < ntok_pad) store_key_words<BITS>(kc, (uint32_t)((r + 16 * j) * (kHeadDim / E)), c8, c, live[j] ? 0xFFFFFFFFu : 0u);
            }
        }
        if constexpr (OUT)   // the zero of (row j's key group, own channel 8 c8 + e) from the table the codes were made with
            store_slots(k_out, s_cnt[0], kw, om, [&](int j, int e) { return s_par[(j / JPG) * kHeadDim + 8 * c8 + e].x; });
    } else {
        per_token(kw, k_scale, k_zero, om, zrow, [&](int j, const float (&c)[8]) {   // (a padding row was loaded as zeros: scale 0, all codes 0)
            if (r + 16 * j < ntok_pad) store_key_words<BITS>(kc, (uint32_t)((r + 16 * j) * (kHeadDim / E)), c8, c);
        });
        if constexpr (OUT) store_slots(k_out, s_cnt[0], kw, om, [&](int j, int) { return __uint_as_float(zrow[j]); });
    }

    // ---------------- values ----------------
    // Token t = r + 16 j = 32 (j / 2) + 16 (j % 2) + 4 wave + i4: half-word H = j % 2, 32-token block
    // j / 2, kb = wave, i = i4.  A lane's field of word (superblock, kb, channel, wl) sits at
    // 16 H + BITS p with run = 4 blk + i4 = wl (E/2) + p; lanes of equal wl OR their fields together.
    {
        uint32_t part[NSB][8];
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
            for (int dd = 0; dd < 8; ++dd) part[sb][dd] = 0u;
        if constexpr (QUANT) {
            if constexpr (OUT) mark(vw, om);
            // A lane's fields of a word sit at 16 H + 8 blk + BITS * (its own place), H = j % 2: the rows of a half-word
            // add up as floats (blocks only at 2 bits), the lane's place is one shift at the end.  (A padding row's codes are all 0.)
            float sum[R / 2][8];                       // rows 2 j2 and 2 j2 + 1: below 2^24
            float even[8];
            per_token(vw, v_scale, v_zero, om, zrow, [&](int j, const float (&c)[8]) {
#pragma unroll
                for (int dd = 0; dd < 8; ++dd) {
                    if ((j & 1) == 0) even[dd] = c[dd];
                    else sum[j >> 1][dd] = field_sum<16>(even[dd], c[dd]);
                }
            });
            if constexpr (OUT) store_slots(v_out, s_cnt[1], vw, om, [&](int j, int) { return __uint_as_float(zrow[j]); });
            const uint32_t place = BITS * (i4 % (E / 2));
#pragma unroll
            for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
                for (int dd = 0; dd < 8; ++dd) {
                    if constexpr (SB == 64) part[sb][dd] = ((uint32_t)sum[2 * sb][dd] | ((uint32_t)sum[2 * sb + 1][dd] << 8)) << place;
                    else part[sb][dd] = (uint32_t)sum[sb][dd] << place;
                }
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int sb = j >> 1, H = j & 1;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    part[sb][2 * q] |= (vw[j][q] & 0xffffu) << (16 * H);
                    part[sb][2 * q + 1] |= (vw[j][q] >> 16) << (16 * H);
                }
            }
        }
        // Row lanes whose fields share a word merge them, and every lane exchange merges two registers into one:
        // a lane is left with 8 / LANES_PER_WORD of the channels, first + 0 .. (bit 2 of the channel by the lane's
        // place among the neighbouring rows, bit 1 by the half of the wave).
        constexpr int LANES_PER_WORD = (E / 2 >= 4) ? 4 : E / 2;
        constexpr int NW = 8 / LANES_PER_WORD;
        const int wl = (E / 2 >= 4) ? 0 : i4 / (E / 2);          // run / (E/2) with blk = 0 (SB = 32 whenever E/2 < 4)
        const int tile = c8 >> 1, y = tile * WPT + wl;
        const int first = (LANES_PER_WORD >= 2 ? 4 * (i4 & 1) : 0) + (LANES_PER_WORD >= 4 ? 2 * (i4 >> 1) : 0);
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb) {
            uint32_t m[NW];
            if constexpr (LANES_PER_WORD == 1) {
#pragma unroll
                for (int dd = 0; dd < 8; ++dd) m[dd] = part[sb][dd];
            } else {
                uint32_t h[4];
#pragma unroll
                for (int dd = 0; dd < 4; ++dd) {
                    const auto x = __builtin_amdgcn_permlane16_swap(part[sb][dd], part[sb][4 + dd], false, false);
                    h[dd] = x[0] | x[1];
                }
#pragma unroll
                for (int dd = 0; dd < NW; ++dd) {
                    if constexpr (LANES_PER_WORD == 4) {
                        const auto x = __builtin_amdgcn_permlane32_swap(h[dd], h[2 + dd], false, false);
                        m[dd] = x[0] | x[1];
                    } else {
                        m[dd] = h[dd];
                    }
                }
            }
#pragma unroll
            for (int dd = 0; dd < NW; ++dd) {
                const int n = 8 * (c8 & 1) + first + dd;
                s_words[sb * SBW + ((y >> 2) * 64 + wave * 16 + n) * 4 + (y & 3)] = m[dd];
            }
        }
        __syncthreads();
        const int n_sb = (ntok + SB - 1) / SB;
        uint32_t* vc = v_codes + (size_t)head * SBW * ((n_cap + SB - 1) / SB) + (size_t)(d0 / SB) * SBW;
        for (int item = threadIdx.x; item < n_sb * SBW / 4; item += kThreads)
            reinterpret_cast<uint4*>(vc)[item] = reinterpret_cast<const uint4*>(s_words)[item];
    }
    // (the barrier before the value store: every wave has its rows in registers)
    if (tail_len > 0) close_tail(tail_k, tail_v, head, tail_cap, n_head, tail_len);
    if constexpr (OUT) {   // (the barrier before the value store orders every row's count before this)
        const int tensor = threadIdx.x / (TB / 32), blk = threadIdx.x % (TB / 32);
        if (threadIdx.x < 2 * (TB / 32) && 32 * blk < ntok) {
            uint32_t* ovf = (tensor ? v_ovf : k_ovf) + (size_t)head * ovf_words(n_cap, ovf_cap);
            ovf[d0 / 32 + blk + 1] = (uint32_t)s_cnt[tensor][blk] | kBlockCount;
        }
    }
}

// The prefix counts and overflow entries of one block of 32 tokens (one wave).  The quantizer has left every
// block's own number of overflow outliers, marked by kBlockCount, at the block's entry + 1 of the head's prefix
// array; here the mark goes and the number becomes the prefix count.  An entry of the array is
// one or the other at any time and tells which, so a wave adds up the blocks before its own, backwards
// up to the first prefix count that it meets, without waiting for anyone: a prefix count that was stored
// meanwhile only saves it the rest.  (A kernel of its own for the prefix counts, one wave per head and
// tensor, was a launch between two others and went through a long head 64 blocks at a time.)
// Then the block's rows are read again, the
// outliers beyond a row's fourth found in channel order, and written as (word, token) at the block's
// place in the head's list -- position = prefix count of the block + entries of the block's earlier
// rows -- unless they lie beyond the list's capacity.  Most blocks have none and leave at once.
template <int G>
__global__ __launch_bounds__(64) void ovf_fill(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                               const int32_t* __restrict__ idx, const uint16_t* __restrict__ k_zero,
                                               const uint16_t* __restrict__ v_zero, uint32_t* __restrict__ k_ovf,
                                               uint32_t* __restrict__ v_ovf, int L, int n_kept, int key_axis, int n_cap,
                                               int dst_base, const int32_t* __restrict__ head_n, uint32_t tau_bits,
                                               const int32_t* __restrict__ head_base, int base_quantum, int ovf_cap) {
    const int head = blockIdx.y, lane = threadIdx.x, tensor = blockIdx.z;
    int base = dst_base;
    if (head_base) {
        base = min(max(head_base[head], 0), dst_base);
        base -= base % base_quantum;
    }
    const int n_head = head_n ? min(max(head_n[head], 0), n_kept) : n_kept;
    const int t0 = 32 * blockIdx.x;
    uint32_t* ovf = (tensor ? v_ovf : k_ovf) + (size_t)head * ovf_words(n_cap, ovf_cap);
    const int first = base / 32, blk = first + (int)blockIdx.x;
    if (first == 0 && t0 == 0 && lane == 0) ovf[0] = 0u;
    if (t0 >= n_head) return;
    auto entry = [&](int i) { return __hip_atomic_load(ovf + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    const uint32_t own = entry(blk + 1) & ~kBlockCount;
    uint32_t at = 0u;                                // entries of the blocks before this one
    constexpr int kAhead = 4;                        // entries per lane and step: 256 blocks
    for (int top = blk; ; top -= 64 * kAhead) {      // entries top, top - 1, ...; entry `first` is a prefix count (0 at a head's start)
        uint32_t v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = top - 64 * u - lane;
            const uint32_t x = entry(max(i, first));
            v[u] = i > first ? x : first > 0 ? x & ~kBlockCount : 0u;
        }
        bool known = false;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const unsigned long long done = __builtin_amdgcn_ballot_w64((v[u] & kBlockCount) == 0u);    // prefix counts
            const int last = done ? __builtin_ctzll(done) : 63;
            uint32_t add = known || lane > last ? 0u : v[u] & ~kBlockCount;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) add += __shfl_xor(add, off);
            at += add;
            known = known || done != 0ull;
        }
        if (known) break;
    }
    if (lane == 0) __hip_atomic_store(ovf + blk + 1, at + own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (own == 0u) return;                           // (wave-uniform) nothing beyond the slots in this block
    uint32_t* entries = ovf + ovf_start_words(n_cap);
    const uint16_t* src = (tensor ? v : k) + (size_t)head * L * kHeadDim;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    for (int t = t0; t < min(t0 + 32, n_head); ++t) {
        const int pos = idx ? idx[(size_t)head * n_kept + t] : t;
        const uint32_t w = *reinterpret_cast<const uint32_t*>(src + (size_t)pos * kHeadDim + 2 * lane);   // channels 2 lane, 2 lane + 1
        const bool c0 = (w & 0x7fffu) > tau_bits, c1 = ((w >> 16) & 0x7fffu) > tau_bits;
        const unsigned long long b0 = __builtin_amdgcn_ballot_w64(c0), b1 = __builtin_amdgcn_ballot_w64(c1);
        const uint32_t total = (uint32_t)(__popcll(b0) + __popcll(b1));
        if (total <= 4u) continue;                   // (wave-uniform)
        const uint32_t r0 = (uint32_t)(__popcll(b0 & lt_mask) + __popcll(b1 & lt_mask)), r1 = r0 + (c0 ? 1u : 0u);
        const int tok = base + t;                    // the token's position in the head
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const bool is = e ? c1 : c0;
            const uint32_t rank = e ? r1 : r0;
            if (is && rank >= 4u) {
                const int d = 2 * lane + e;
                const size_t m = (tensor == 0 && key_axis == KVQP_KEY_PER_CHANNEL)
                                     ? ((size_t)head * ((n_cap + G - 1) / G) + tok / G) * kHeadDim + d
                                     : ((size_t)head * n_cap + tok) * (kHeadDim / G) + d / G;
                const float zf = half_bits_to_float((tensor ? v_zero : k_zero)[m]);
                const uint32_t xh = e ? (w >> 16) : (w & 0xffffu);
                const float diff = __fsub_rn(half_bits_to_float((uint16_t)xh), zf);
                const uint32_t e_at = at + rank - 4u;
                if (e_at < (uint32_t)ovf_cap) {
                    entries[2 * (size_t)e_at] = (__float_as_uint(diff) & 0xFFFFFF00u) | 0x80u | (uint32_t)d;
                    entries[2 * (size_t)e_at + 1] = (uint32_t)tok;
                }
            }
        }
        at += total - 4u;
    }
}

template <int BITS, int G, bool OUT>
hipError_t launch_bits_g(const QuantPackJob& j, hipStream_t stream) {
    constexpr int TB = quant_tokens(BITS, G);
    const int nblk = (j.n_tok + TB - 1) / TB;
    dim3 grid(nblk + (j.copy_tail ? 1 : 0), j.heads);
    if (grid.x == 0) return hipSuccess;
    hipLaunchKernelGGL((gather_quant_pack<BITS, G, OUT>), grid, dim3(kThreads), 0, stream, (const uint16_t*)j.k,
                       (const uint16_t*)j.v, j.idx, (uint32_t*)j.c.k_codes, (uint32_t*)j.c.v_codes, (uint16_t*)j.c.k_scale,
                       (uint16_t*)j.c.k_zero, (uint16_t*)j.c.v_scale, (uint16_t*)j.c.v_zero, (uint16_t*)j.c.tail_k,
                       (uint16_t*)j.c.tail_v, j.src_rows, j.window, j.n_tok, j.key_axis, j.c.tail_cap, nblk, j.n_cap,
                       j.dst_base, j.head_n, (uint32_t*)j.c.k_out, (uint32_t*)j.c.v_out, j.tau_bits, j.head_base,
                       j.base_quantum, (uint32_t*)j.c.k_ovf, (uint32_t*)j.c.v_ovf, j.ovf_cap, closes_tail(j) ? j.tail_len : 0);
    hipError_t e = hipGetLastError();
    if constexpr (OUT) {
        if (e != hipSuccess || j.n_tok == 0) return e;
        hipLaunchKernelGGL((ovf_fill<G>), dim3((j.n_tok + 31) / 32, j.heads, 2), dim3(64), 0, stream, (const uint16_t*)j.k,
                           (const uint16_t*)j.v, j.idx, (const uint16_t*)j.c.k_zero, (const uint16_t*)j.c.v_zero,
                           (uint32_t*)j.c.k_ovf, (uint32_t*)j.c.v_ovf, j.src_rows, j.n_tok, j.key_axis, j.n_cap, j.dst_base,
                           j.head_n, j.tau_bits, j.head_base, j.base_quantum, j.ovf_cap);
        e = hipGetLastError();
    }
    return e;
}
template <int BITS>
hipError_t launch_bits(const QuantPackJob& j, hipStream_t stream) {
    if constexpr (BITS == 16) {
        return launch_bits_g<BITS, 32, false>(j, stream);
    } else {
        if (j.outliers) {
            switch (j.group_size) {
                case 32: return launch_bits_g<BITS, 32, true>(j, stream);
                case 64: return launch_bits_g<BITS, 64, true>(j, stream);
                default: return launch_bits_g<BITS, 128, true>(j, stream);
            }
        }
        switch (j.group_size) {
            case 32: return launch_bits_g<BITS, 32, false>(j, stream);
            case 64: return launch_bits_g<BITS, 64, false>(j, stream);
            default: return launch_bits_g<BITS, 128, false>(j, stream);
        }
    }
}

__global__ __launch_bounds__(kThreads) void tail_shift(uint16_t* __restrict__ tail_k, uint16_t* __restrict__ tail_v,
                                                       int tail_cap, int n_shift, int tail_len) {
    close_tail(tail_k, tail_v, blockIdx.x, tail_cap, n_shift, tail_len);
}

hipError_t launch_job(const QuantPackJob& j, hipStream_t stream) {
    switch (j.bits) {
        case 2: return launch_bits<2>(j, stream);
        case 4: return launch_bits<4>(j, stream);
        case 8: return launch_bits<8>(j, stream);
        default: return launch_bits<16>(j, stream);
    }
}

}  // namespace

// Largest binary16 magnitude pattern whose value does not exceed tau (> 0): |x| > tau iff the
// pattern of |x| is greater (patterns of non-negative halves order like their values).
static uint32_t threshold_bits(float tau) {
    auto value = [](uint32_t h) -> double {   // finite non-negative binary16 pattern -> value
        const int e = (int)(h >> 10), m = (int)(h & 0x3ff);
        return e == 0 ? m * (1.0 / 16777216.0) : (double)(1024 + m) * (e >= 25 ? (double)(1 << (e - 25)) : 1.0 / (double)(1 << (25 - e)));
    };
    uint32_t lo = 0, hi = 0x7BFF;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) / 2;
        if (value(mid) <= (double)tau) lo = mid; else hi = mid - 1;
    }
    return lo;
}
static void set_outliers(QuantPackJob& j, const kvqp_cfg& cfg) {
    j.outliers = outliers_on(cfg);
    j.ovf_cap = cfg.outlier_overflow_cap;
    j.tau_bits = j.outliers ? threshold_bits(cfg.outlier_threshold) : 0x7fffu;
}

hipError_t launch_quant_pack(const kvqp_cfg& cfg, const void* k, const void* v, const int32_t* idx, int n_kept,
                             const int32_t* head_n, const kvqp_cache& cache, hipStream_t stream) {
    QuantPackJob j{cache};
    set_outliers(j, cfg);
    j.k = k; j.v = v; j.idx = idx; j.head_n = head_n;
    j.heads = cfg.batch * cfg.n_kv_heads; j.src_rows = cfg.seq_len; j.window = cfg.window;
    j.n_tok = n_kept; j.dst_base = 0; j.n_cap = layout_tokens(cache, n_kept);
    j.bits = cfg.bits; j.group_size = cfg.group_size; j.key_axis = cfg.key_axis; j.copy_tail = true;
    return launch_job(j, stream);
}

// Host counts -> device array, carried in kernel arguments (copied when the launch is enqueued, so
// the caller's array may go away as soon as the call returns; no staging copy, no synchronisation).
struct CountBatch { int32_t v[kCountsPerLaunch]; };
__global__ void store_counts(int32_t* __restrict__ dst, CountBatch b, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = b.v[i];
}
hipError_t upload_counts(int32_t* dst, const int32_t* src_host, int n, hipStream_t stream, int add) {
    for (int i0 = 0; i0 < n; i0 += kCountsPerLaunch) {
        CountBatch b;
        const int m = n - i0 < kCountsPerLaunch ? n - i0 : kCountsPerLaunch;
        for (int i = 0; i < m; ++i) b.v[i] = (src_host ? src_host[i0 + i] : 0) + add;
        for (int i = m; i < kCountsPerLaunch; ++i) b.v[i] = 0;
        hipLaunchKernelGGL(store_counts, dim3((m + 255) / 256), dim3(256), 0, stream, dst + i0, b, m);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The n_tokens oldest tail rows are quantized onto the end of the packed part, then the tail closes up.
// base_quantum > 0: every head at its own count (cache.head_n_kept), counts being multiples of it.
hipError_t launch_append_tail(const kvqp_cfg& cfg, const kvqp_cache& cache, int n_tokens, int base_quantum, hipStream_t stream) {
    QuantPackJob j{cache};
    set_outliers(j, cfg);
    j.k = cache.tail_k; j.v = cache.tail_v; j.idx = nullptr; j.head_n = nullptr;
    if (base_quantum > 0) { j.head_base = cache.head_n_kept; j.base_quantum = base_quantum; }
    j.heads = cfg.batch * cfg.n_kv_heads; j.src_rows = cache.tail_cap; j.window = 0;
    j.n_tok = n_tokens; j.dst_base = cache.n_kept; j.n_cap = layout_tokens(cache, cache.n_kept);
    j.bits = cfg.bits; j.group_size = cfg.group_size; j.key_axis = cfg.key_axis; j.copy_tail = false;
    j.tail_len = cache.tail_len;
    hipError_t e = launch_job(j, stream);
    if (e != hipSuccess || closes_tail(j)) return e;
    hipLaunchKernelGGL(tail_shift, dim3(j.heads), dim3(kThreads), 0, stream, (uint16_t*)cache.tail_k, (uint16_t*)cache.tail_v,
                       cache.tail_cap, n_tokens, cache.tail_len);
    return hipGetLastError();
}

}  // namespace kvqp
