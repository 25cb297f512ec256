// Huffman decode + undifferencing of the pointing streams (section 4.1), and
// of the TOD and flag streams (k_decode1: one stream, same format).
//
// Two kernels per call: k_tables, then a decoder.
//
// k_tables turns every table blob into a DecTab: the canonical limits and a
// 12-bit prefix table giving the code length of every prefix whose codes all
// share one length.  The limit of a length L <= 12 is a multiple of 2^20 and
// never splits a prefix, and each longer length splits at most one, so the
// prefix table resolves the short codes and almost every long one too (the
// psi differences are near-uniform on +-4095: almost all psi codes are longer
// than 12 bits); only codes behind one of the <= 20 split prefixes search the
// limits.
//
// The decoders: k_decode32 and k_decode32_1 for chunks of 32 symbols (the
// default spacing of the side index), k_decode and k_decode1 for longer
// chunks, whose words would not fit a block's LDS, and for streams of 32-symbol
// chunks too dense for it (over 22 bits a sample for both streams of the pointing,
// over 15 for one stream alone).
//
// k_decode: a block owns up to C3_DEC_NT consecutive chunks of one segment; each
// thread parses one chunk of both streams from the side index, G codes per
// round, adds the symbol values to its running value (x_i = x_{i-1} + d_i),
// range-checks, and leaves the samples in an LDS tile; the block then writes
// the tile in rows of 16 consecutive samples of a chunk.
#include <mutex>
#include <type_traits>

#include "common.h"
#include "perdev.h"

namespace {

constexpr int G = 16;          // symbols per thread per round
constexpr int GP = G + 1;      // padded LDS row (no bank conflicts on the column writes)
constexpr int SPLIT = 32 - C3_KLUT;

// smallest L in [from, maxlen] with w < lim[L]; 0 if there is none
__device__ __forceinline__ int code_len(const DecTab &T, unsigned long long w, int from) {
    for (int L = from; L <= T.maxlen; ++L)
        if (w < T.lim[L]) return L;
    return 0;
}
__device__ __forceinline__ int code_len(const DecTab &T, unsigned long long w) { return code_len(T, w, T.minlen); }

// length of the code at the top of win from its prefix-table entry e: e itself
// when the prefix resolves it (0 < e < 64); otherwise a search of the limits
// from the shortest length under the prefix (e = 64 | that length) or from
// minlen (e = 0: no code starts the prefix).  0: invalid code.
__device__ __forceinline__ int resolve_len(const DecTab &T, uint32_t win, int e) {
    if (e > 0 && e < 64) return e;
    return code_len(T, win, e ? (e & 63) : T.minlen);
}

// The decoding table of one blob [nsym, maxlen, count_1 .. count_32, symbols...]
// in LDS, by all NT threads of a block; they meet at a barrier at its end.  The
// 32 counts are loaded by 32 lanes at once and walked in registers, and a
// prefix's two lengths are counts of the limits below it, so nothing in it is
// a chain of loads (one thread walking the blob, and a search per prefix, took
// 14 to 27 us a call: more than the decode itself for a few scans).
template <int NT>
__device__ __forceinline__ void build_table(DecTab &T, const uint32_t *__restrict__ blob) {
    const int tid = threadIdx.x;
    if (tid < 64) {
        const uint32_t mine = tid >= 1 && tid <= 32 ? blob[1 + tid] : 0;
        unsigned long long first = 0, lim = 0;
        int64_t off = 0;
        int32_t delta = 0;
        int ok = 1, minlen = 33, maxlen = 0;
        for (int L = 1; L <= 32; ++L) {
            const uint32_t cnt = __builtin_amdgcn_readlane(mine, L);
            const unsigned long long end = first + cnt;
            if (end > (1ull << L)) ok = 0;  // more codes of length <= L than L bits hold
            if (tid == L) {
                delta = (int32_t)(off - (int64_t)first);
                lim = end << (32 - L);
            }
            if (tid == 33) lim = end << (32 - L);  // ends as lim[32]
            if (cnt) {
                if (minlen > 32) minlen = L;
                maxlen = L;
            }
            off += cnt;
            first = end << 1;
        }
        if (maxlen == 0 || off != (int64_t)blob[0]) ok = 0;
        if (tid <= 33) {
            T.lim[tid] = lim;
            T.delta[tid] = delta;
        }
        if (tid == 0) {
            T.minlen = minlen > 32 ? 32 : minlen;
            T.maxlen = maxlen;
            T.nsym = ok ? (int32_t)off : 0;
            T.ok = ok;
            T.pad[0] = T.pad[1] = 0;
        }
    }
    __syncthreads();
    // Code lengths only grow with the code value, so a prefix's codes have
    // lengths from L0 (its first code's) to L1 (its last code's); the limits
    // grow with the length, so each is minlen plus the limits passed.
    constexpr int PER = (1 << C3_KLUT) / NT;
    static_assert(PER * NT == 1 << C3_KLUT, "prefixes per thread");
    const int e0 = tid * PER;
    const int lo = T.minlen, hi = T.maxlen;
    int n0[PER], n1[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) n0[i] = n1[i] = lo;
    for (int L = lo; L <= hi; ++L) {
        const unsigned long long lim = T.lim[L];
        const int c = (int)((lim + ((1ull << SPLIT) - 1)) >> SPLIT), f = (int)(lim >> SPLIT);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            n0[i] += e0 + i >= c;
            n1[i] += e0 + i >= f;
        }
    }
    const bool ok = T.ok;
#pragma unroll
    for (int i = 0; i < PER; ++i)
        T.lut[e0 + i] = !ok || n0[i] > hi ? 0 : (uint8_t)(n0[i] == n1[i] ? n0[i] : 64 | n0[i]);
    __syncthreads();
}

__global__ __launch_bounds__(1024) void k_tables(HuffDev hp, HuffDev hs, DecTab *tabs) {
    __shared__ DecTab T;
    const int b = blockIdx.x;
    const bool is_p = b < hp.ntable;
    const int t = is_p ? b : b - hp.ntable;
    build_table<1024>(T, is_p ? hp.tables + hp.table_off[t] : hs.tables + hs.table_off[t]);
    const uint4 *src = (const uint4 *)&T;
    uint4 *dst = (uint4 *)(tabs + b);
    for (int i = threadIdx.x; i < (int)(sizeof(DecTab) / 16); i += 1024) dst[i] = src[i];
}

// word 3 of a raw buffer resource on gfx9-family chips (untyped dword access)
#define C3_BUF_WORD3 0x00020000

// block-uniform values (one segment per block) moved to scalar registers, so
// that the buffer resources built from them are scalar
__device__ __forceinline__ int32_t uni(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ const void *uni(const void *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const void *)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void *base, int32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)uni(base), 0, uni(bytes), C3_BUF_WORD3);
}

// dword i of a raw buffer: 0 past its end (the hardware range check)
__device__ __forceinline__ uint32_t buf_word(__amdgpu_buffer_rsrc_t r, uint32_t i) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, (int)(4u * i), 0, 0);
}

// MSB-first bit reader over one segment's stream (a raw buffer, so reads
// past the end give zero bits).  Look-ahead: three pairs of words in stream
// order, kept as loaded (no reordering at load time).  A pair is loaded two
// pair-lengths before its first word is used, so the wait for it falls long
// after the load was issued.
struct BitReader {
    __amdgpu_buffer_rsrc_t rs;
    unsigned long long buf;  // next bits, MSB first; nbits of them valid
    uint2 n0, n1, n2;        // look-ahead words n0.x, n0.y, n1.x, ... in stream order
    uint32_t wp;             // next word to load
    int nbits, nh;           // nh: words of n0 not yet taken (2, 1 or 0)

    __device__ __forceinline__ uint2 load2(uint32_t p) const {
        return make_uint2(buf_word(rs, p), buf_word(rs, p + 1u));
    }
    __device__ void init(__amdgpu_buffer_rsrc_t r, uint32_t bit) {
        rs = r;
        const uint32_t p = bit >> 5;
        const int s = bit & 31;
        const uint2 w = load2(p);
        buf = (((unsigned long long)w.x << 32) | w.y) << s;
        nbits = 64 - s;
        n0 = load2(p + 2u);
        n1 = load2(p + 4u);
        n2 = load2(p + 6u);
        nh = 2;
        wp = p + 8u;
    }
    __device__ __forceinline__ void refill() {
        const bool need = nbits < 32;
        const uint32_t word = nh == 2 ? n0.x : n0.y;
        const int sh = need ? 32 - nbits : 0;
        buf |= need ? (unsigned long long)word << sh : 0ull;
        nbits += need ? 32 : 0;
        nh -= need ? 1 : 0;
        if (nh == 0) {  // every second refill: the pairs move up, one more is loaded
            n0 = n1;
            n1 = n2;
            nh = 2;
            n2 = load2(wp);
            wp += 2u;
        }
    }
    // the next 32 bits, the next code at the top (refilled first)
    __device__ __forceinline__ uint32_t window() {
        refill();
        return (uint32_t)(buf >> 32);
    }
    // drop the Lc bits of the code just read
    __device__ __forceinline__ void consume(int Lc) {
        buf <<= Lc;
        nbits -= Lc;
    }
    // symbol index of the next code; L = its length (0: invalid code)
    __device__ __forceinline__ int32_t next(const DecTab &T, int &L) {
        const uint32_t win = window();
        L = resolve_len(T, win, T.lut[win >> SPLIT]);
        const int Lc = L ? L : 1;
        const int32_t idx = (int32_t)(win >> (32 - Lc)) + T.delta[Lc];
        consume(Lc);
        return L ? idx : -1;
    }
};

__global__ __launch_bounds__(C3_DEC_NT) void k_decode(LayoutDev Ld, HuffDev hp, HuffDev hs,
                                                  const DecTab *__restrict__ tabs,
                                                  const DecodeTask *__restrict__ tasks,
                                                  int32_t *__restrict__ pix_out,
                                                  uint16_t *__restrict__ psi_out, uint32_t *err) {
    __shared__ DecTab cp, cq;
    __shared__ int32_t tp[C3_DEC_NT * GP];
    __shared__ uint16_t tq[C3_DEC_NT * GP];  // psi symbol indices, then psi values
    __shared__ uint32_t blk_err;

    const DecodeTask task = tasks[blockIdx.x];
    const int seg = task.seg;
    const int tid = threadIdx.x;
    const int64_t s0 = Ld.seg_off[seg];
    const int n = (int)(Ld.seg_off[seg + 1] - s0);
    const int C = hp.chunk_len;
    const int band = Ld.seg_band[seg];
    const uint32_t npix = (uint32_t)Ld.band[band].npix;
    const uint32_t npsi = (uint32_t)Ld.band[band].npsi;

    // this segment's two tables (an out-of-range table id is an invalid code)
    const int tpi = hp.seg_table[seg], tqi = hs.seg_table[seg];
    const bool tabs_ok = tpi >= 0 && tpi < hp.ntable && tqi >= 0 && tqi < hs.ntable;
    {
        const uint4 *sp = (const uint4 *)(tabs + (tabs_ok ? tpi : 0));
        const uint4 *sq = (const uint4 *)(tabs + hp.ntable + (tabs_ok ? tqi : 0));
        uint4 *dp = (uint4 *)&cp, *dq = (uint4 *)&cq;
        for (int i = tid; i < (int)(sizeof(DecTab) / 16); i += C3_DEC_NT) {
            dp[i] = sp[i];
            dq[i] = sq[i];
        }
        if (tid == 0) blk_err = 0;
    }
    __syncthreads();
    const bool codes_ok = tabs_ok && cp.ok && cq.ok && cq.nsym < 65535;
    // symbol arrays as raw buffers of nsym entries: an invalid index reads 0
    const __amdgpu_buffer_rsrc_t symp =
        raw_buffer(hp.tables + hp.table_off[tabs_ok ? tpi : 0] + 34, 4 * cp.nsym);
    const __amdgpu_buffer_rsrc_t symq =
        raw_buffer(hs.tables + hs.table_off[tabs_ok ? tqi : 0] + 34, 4 * cq.nsym);

    const int l = tid;
    const int c = task.chunk0 + l;
    // the side index must hold ceil(n / C) chunks for this segment
    const int nch_idx = (int)min(hp.seg_chunk_off[seg + 1] - hp.seg_chunk_off[seg],
                                 hs.seg_chunk_off[seg + 1] - hs.seg_chunk_off[seg]);
    const bool active = l < task.nchunk && c < nch_idx;
    uint32_t bad = codes_ok ? 0u : C3_ERR_CODE;
    if (l < task.nchunk && c >= nch_idx) bad |= C3_ERR_CHUNK;
    BitReader rp, rq;
    int ns = 0;
    int32_t xp = 0, xq = 0;      // running (undifferenced) values
    int32_t bitp = 0, bitq = 0;  // bits consumed by this chunk's codes
    uint32_t start_p = 0, start_q = 0;
    // the two streams of this segment as raw buffers (below 2^29 words each)
    const int64_t wp0 = hp.seg_word_off[seg], wq0 = hs.seg_word_off[seg];
    const int64_t nwp = hp.seg_word_off[seg + 1] - wp0, nwq = hs.seg_word_off[seg + 1] - wq0;
    const bool words_ok = nwp >= 0 && nwq >= 0 && nwp < (1ll << 29) && nwq < (1ll << 29);
    if (!words_ok) bad |= C3_ERR_CHUNK;
    const __amdgpu_buffer_rsrc_t rsp = raw_buffer(hp.words + wp0, words_ok ? (int32_t)(4 * nwp) : 0);
    const __amdgpu_buffer_rsrc_t rsq = raw_buffer(hs.words + wq0, words_ok ? (int32_t)(4 * nwq) : 0);
    if (active) {
        const int64_t gp = hp.seg_chunk_off[seg] + c;
        const int64_t gq = hs.seg_chunk_off[seg] + c;
        start_p = hp.chunk_bit[gp];
        start_q = hs.chunk_bit[gq];
        rp.init(rsp, start_p);
        rq.init(rsq, start_q);
        xp = hp.chunk_prev[gp];
        xq = hs.chunk_prev[gq];
        ns = (codes_ok && words_ok) ? min(C, n - c * C) : 0;
    }
    const int nround = (C + G - 1) / G;

    // one round: parse G codes of both streams per chunk (symbol indices into
    // this thread's tile row; psi tables hold at most 65535 symbols, checked
    // with the table), then their symbol values (gathers issued in groups),
    // running sums and range checks.  Values go to the thread's tile row, or
    // to registers (v0p, v0q) when the caller asks for them there.
    auto round = [&](int k0, bool to_regs, int32_t *v0p, uint16_t *v0q) {
        if (!(active && k0 < ns)) return;
#pragma unroll 4  // full unrolling runs out of scalar registers
        for (int k = 0; k < G; ++k) {
            // the two streams' table reads are issued together: both
            // prefix-table entries, then (after the rare searches) both
            // index offsets
            const uint32_t wp = rp.window(), wq = rq.window();
            const int ep = cp.lut[wp >> SPLIT], eq = cq.lut[wq >> SPLIT];
            const int Lp = resolve_len(cp, wp, ep), Lq = resolve_len(cq, wq, eq);
            const int Lcp = Lp ? Lp : 1, Lcq = Lq ? Lq : 1;
            const int32_t ip = (int32_t)(wp >> (32 - Lcp)) + cp.delta[Lcp];
            const int32_t iq = (int32_t)(wq >> (32 - Lcq)) + cq.delta[Lcq];
            rp.consume(Lcp);
            rq.consume(Lcq);
            const bool v = k0 + k < ns;
            bad |= (v && (Lp == 0 || Lq == 0)) ? C3_ERR_CODE : 0u;
            bitp += v ? Lp : 0;
            bitq += v ? Lq : 0;
            tp[l * GP + k] = Lp ? ip : -1;
            tq[l * GP + k] = (uint16_t)(Lq ? iq : 0xFFFF);
        }
#pragma unroll
        for (int h = 0; h < G; h += G / 2) {
            int32_t gp_[G / 2], gq_[G / 2];
#pragma unroll
            for (int k = 0; k < G / 2; ++k) {
                gp_[k] = (int32_t)buf_word(symp, (uint32_t)tp[l * GP + h + k]);
                gq_[k] = (int32_t)buf_word(symq, (uint32_t)tq[l * GP + h + k]);
            }
#pragma unroll
            for (int k = 0; k < G / 2; ++k) {
                const bool v = k0 + h + k < ns;
                xp += v ? gp_[k] : 0;
                xq += v ? gq_[k] : 0;
                const bool okp = (uint32_t)xp < npix, okq = (uint32_t)xq < npsi;
                bad |= (v && !okp) ? C3_ERR_PIX : 0u;
                bad |= (v && !okq) ? C3_ERR_PSI : 0u;
                if (to_regs) {
                    v0p[h + k] = okp ? xp : 0;
                    v0q[h + k] = (uint16_t)(okq ? xq : 0);
                } else {
                    tp[l * GP + h + k] = okp ? xp : 0;
                    tq[l * GP + h + k] = (uint16_t)(okq ? xq : 0);
                }
            }
        }
    };
    // write the tile of the round at k0: 16-lane rows of consecutive samples
    // of one chunk
    auto write_tile = [&](int k0) {
#pragma unroll 4
        for (int m = 0; m < G; ++m) {
            const int q = m * C3_DEC_NT + tid;
            const int ll = q >> 4, kk = q & 15;
            const int cc = task.chunk0 + ll;
            const int t = cc * C + k0 + kk;
            if (ll < task.nchunk && cc < nch_idx && k0 + kk < C && t < n && codes_ok && words_ok) {
                pix_out[s0 + t] = tp[ll * GP + kk];
                psi_out[s0 + t] = tq[ll * GP + kk];
            }
        }
    };
    if (nround == 2) {
        // a chunk of two rounds: every store after every load.  Stores and
        // loads share one in-order completion counter, so a store followed by
        // a load that is waited on costs the store's whole latency; the first
        // round's values wait in registers until the second round's loads
        // are done.
        int32_t v0p[G];
        uint16_t v0q[G];
        round(0, true, v0p, v0q);
        round(G, false, nullptr, nullptr);
        __syncthreads();
        write_tile(G);
        __syncthreads();
        if (active && ns > 0) {
#pragma unroll
            for (int k = 0; k < G; ++k) {
                tp[l * GP + k] = v0p[k];
                tq[l * GP + k] = v0q[k];
            }
        }
        __syncthreads();
        write_tile(0);
    } else {
        for (int rd = 0; rd < nround; ++rd) {
            round(rd * G, false, nullptr, nullptr);
            __syncthreads();
            write_tile(rd * G);
            __syncthreads();
        }
    }
    // chunk boundary consistency with the side index: the codes of chunk c end
    // where chunk c + 1 starts, and the running value meets its stored one
    if (active && codes_ok && c + 1 < nch_idx) {
        const int64_t gp = hp.seg_chunk_off[seg] + c + 1;
        const int64_t gq = hs.seg_chunk_off[seg] + c + 1;
        if ((int64_t)start_p + bitp != (int64_t)hp.chunk_bit[gp] || xp != hp.chunk_prev[gp]) bad |= C3_ERR_CHUNK;
        if ((int64_t)start_q + bitq != (int64_t)hs.chunk_bit[gq] || xq != hs.chunk_prev[gq]) bad |= C3_ERR_CHUNK;
    }
    if (active && ns > 0) {
        if ((int64_t)start_p + bitp > 32 * nwp) bad |= C3_ERR_CHUNK;
        if ((int64_t)start_q + bitq > 32 * nwq) bad |= C3_ERR_CHUNK;
    }
    if (bad) atomicOr(&blk_err, bad);
    __syncthreads();
    if (tid == 0 && blk_err) atomicOr(err, blk_err);
}

// ------------------------------------------- chunks of 32 symbols, words in LDS
// The decoders for the densest side index (chunk_len = 32, the format's
// default).  Everything a lane's serial code chain reads is in LDS: the
// block's stream words (staged with coalesced loads; its 512 chunks are
// consecutive in the stream), the decoding tables and the symbol values as
// 16-bit integers, most frequent first.  The window of the next 32 bits is one
// two-word LDS read at the lane's bit position, so there is no look-ahead
// state.  A wave whose 64 chunks are whole swaps its samples between lanes and
// stores contiguous lines (store_rows): no LDS tile, no barrier after the staging.
// Short chunks, and blocks whose words do not fit, are stored sample by sample.
// Symbols that do not fit (beyond the table's first KS entries, or wider than
// 16 bits) are marked and read from memory, eight codes' together.
//
// The decoder that gathers its symbols from memory and reads its words per
// lane is bound by the texture path (64 cache lines per gather); this one by
// the code chain (LDS latency, then vector-ALU issue at 0.45).  Pointing, 70
// GHz-like: 9.4e8 samples 5.32 -> 3.20 ms, 1e8 samples 611 -> 356 us; pointing,
// TOD and flags of a 30 GHz-like set of 1.8e7 samples 314 -> 212 us (tables
// included).

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(4))) Store16 {
    u32x4 v;
};
struct __attribute__((packed, aligned(2))) Store16h {
    u32x4 v;
};
struct __attribute__((packed, aligned(1))) Store16b {
    u32x4 v;
};

constexpr int kEsc = -32768;      // marks a symbol that is read from memory
constexpr int kWordsPer = 36;     // words a chunk may touch from its first on: 32 codes of 32 bits, and a window's three

// LDS image of one stream: table, 16-bit symbols (two extra entries: the
// escape, and the zero that an invalid code yields), staged words
template <int KS>
struct StreamLds {
    DecTab T;
    int16_t sym[KS + 2];
};

// Staging, in two halves so that every load of a block is issued before the
// first is waited for: PER dwords a thread, 512 apart, from a raw buffer
// (zeros past its end), then to LDS.
template <int PER>
struct Stage {
    uint32_t v[PER];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t w0) {
#pragma unroll
        for (int r = 0; r < PER; ++r) v[r] = buf_word(rs, w0 + threadIdx.x + (uint32_t)r * C3_DEC_NT);
    }
    __device__ __forceinline__ void words(uint32_t *W, uint32_t n) const {
#pragma unroll
        for (int r = 0; r < PER; ++r)
            if (threadIdx.x + (uint32_t)r * C3_DEC_NT < n) W[threadIdx.x + r * C3_DEC_NT] = v[r];
    }
    // as symbols: 16-bit values, or the escape
    template <int KS>
    __device__ __forceinline__ void symbols(StreamLds<KS> &S) const {
        static_assert(KS == PER * C3_DEC_NT, "symbols per thread");
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const int x = (int)v[r];
            S.sym[threadIdx.x + r * C3_DEC_NT] = (int16_t)(x > kEsc && x <= 32767 ? x : kEsc);
        }
        if (threadIdx.x == 0) {
            S.sym[KS] = (int16_t)kEsc;
            S.sym[KS + 1] = 0;
        }
    }
};
// words beyond the first 16 of a thread
__device__ __forceinline__ void stage_rest(uint32_t *W, __amdgpu_buffer_rsrc_t rs, uint32_t w0, uint32_t n) {
    for (uint32_t i = threadIdx.x + 16 * C3_DEC_NT; i < n; i += C3_DEC_NT) W[i] = buf_word(rs, w0 + i);
}
// a table's symbols as a raw buffer: those its blob has room for
__device__ __forceinline__ __amdgpu_buffer_rsrc_t symbol_buffer(const HuffDev &h, int t) {
    const uint32_t *blob = h.tables + h.table_off[t];
    const int64_t room = max((int64_t)0, min(h.table_off[t + 1] - h.table_off[t] - 34, (int64_t)blob[0]));
    return raw_buffer(blob + 34, (int32_t)(4 * min(room, (int64_t)1 << 28)));
}

// One stream of one lane: bit position (relative to the staged words, or to
// the segment's stream when they are not staged) and running value.
template <int KS, bool STAGED>
struct LaneStream {
    const StreamLds<KS> &S;
    const uint32_t *W;
    __amdgpu_buffer_rsrc_t rs, rsym;
    uint32_t pos;
    int32_t x;
    uint32_t w[3];   // the words under pos and the two after them
    uint32_t at;     // bit within them
    int L;           // length of the current code
    bool inv;        // no code matches: one bit is consumed, the symbol counts as 0

    // one read serves two codes: 31 + 32 + 32 bits at most
    __device__ __forceinline__ void read() {
        const uint32_t i = pos >> 5;
#pragma unroll
        for (int k = 0; k < 3; ++k) w[k] = STAGED ? W[i + k] : buf_word(rs, i + k);
        at = pos & 31;
    }
    __device__ __forceinline__ uint32_t window() const {
        const bool up = at >= 32;
        const uint32_t a = up ? w[1] : w[0], b = up ? w[2] : w[1];
        return (uint32_t)(((((unsigned long long)a << 32) | b) << (at & 31)) >> 32);
    }
    // the prefix does not settle the length: search the limits
    __device__ __forceinline__ void search(uint32_t win, int e) {
        L = resolve_len(S.T, win, e);
        inv = L == 0;
        L = inv ? 1 : L;
    }
    __device__ __forceinline__ uint32_t index(uint32_t win) const {
        return (win >> (32 - L)) + (uint32_t)S.T.delta[L];
    }
    // the zero entry for no code, the escape beyond the symbols held
    __device__ __forceinline__ int value(uint32_t i) const { return S.sym[inv ? KS + 1 : min(i, (uint32_t)KS)]; }
    __device__ __forceinline__ void consume() {
        pos += L;
        at += L;
    }
};

// entry e of the prefix table settles the code length
__device__ __forceinline__ bool settled(int e) { return (uint32_t)(e - 1) < 63u; }

// the marked symbols of eight codes, their reads in flight together (idx: the
// symbols' own indices)
template <typename LS>
__device__ __forceinline__ void escapes(const LS &s, int *v, const uint32_t *idx) {
    bool any = false;
#pragma unroll
    for (int k = 0; k < 8; ++k) any |= v[k] == kEsc;
    if (any) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (v[k] == kEsc) v[k] = (int)buf_word(s.rsym, idx[k]);
    }
}

// A wave's 64 lanes each hold 16 consecutive dwords of their own output (four
// units of 16 bytes); the transposed store makes the four rows of 16 lanes
// write the four units of one lane, so an instruction covers whole 64-byte
// pieces and a wave's few instructions a contiguous stretch of memory.  Lanes
// that store their own units one by one leave 32,768 lines per XCD half
// written, more than its L2 holds, and memory sees 2.3 times the bytes.
// v: the units' dwords; out: the wave's first output; per: bytes of a lane's
// output; off: offset of these units in it.
template <typename St>
__device__ __forceinline__ void store_rows(uint32_t *v, char *out, uint32_t per, uint32_t off) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // dword i of the units 0..3
        uint32_t &a = v[i], &b = v[4 + i], &c = v[8 + i], &d = v[12 + i];
        // rows 2, 3 of the first with rows 0, 1 of the second
        auto x = __builtin_amdgcn_permlane32_swap(a, c, false, false);
        auto y = __builtin_amdgcn_permlane32_swap(b, d, false, false);
        // odd rows of the first with even rows of the second
        auto p = __builtin_amdgcn_permlane16_swap(x[0], y[0], false, false);
        auto q = __builtin_amdgcn_permlane16_swap(x[1], y[1], false, false);
        a = p[0];
        b = p[1];
        c = q[0];
        d = q[1];
    }
    const uint32_t row = (threadIdx.x >> 4) & 3, l = threadIdx.x & 15;
    char *o = out + l * per + row * 16 + off;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        ((St *)(o + (uint32_t)r * 16 * per))->v = u32x4{v[4 * r], v[4 * r + 1], v[4 * r + 2], v[4 * r + 3]};
}

// Dynamic LDS of the two kernels: streams, then the staged words.  Two blocks
// of the pointing decoder share a CU, three of the single-stream decoder.
constexpr int KSP = 4096, KSQ = 8192;  // symbols held: pixel stream, psi (and TOD, flag) stream
constexpr int kPair = (int)(sizeof(StreamLds<KSP>) + sizeof(StreamLds<KSQ>)), kOne = (int)sizeof(StreamLds<KSQ>);
// (LDS is allocated in units of 1280 bytes; 256 are the block votes'.)
constexpr int kPairLds = C3_LDS_MAX / 2 - 256, kOneLds = C3_LDS_MAX / 3 / 1280 * 1280 - 256;
constexpr uint32_t kPairWords = (kPairLds - (kPair + 15) / 16 * 16) / 4, kOneWords = (kOneLds - (kOne + 15) / 16 * 16) / 4;

extern __shared__ __attribute__((aligned(16))) unsigned char c3_dec_lds[];

// a table that k_tables made to LDS (blocks that build their own tables were
// no faster at any size, one launch less included)
template <int KS>
__device__ __forceinline__ void stage_table(StreamLds<KS> &S, const DecTab *tab) {
    constexpr int n = (int)(sizeof(DecTab) / 16);
    static_assert(n <= C3_DEC_NT, "one load a thread");
    if (threadIdx.x < n) ((uint4 *)&S.T)[threadIdx.x] = ((const uint4 *)tab)[threadIdx.x];
}

// first and last bit of the block's chunks in one stream, and whether every
// lane's chunk lies between them (a side index in order)
struct Span {
    uint32_t w0, n;  // first word, words to stage
};
__device__ __forceinline__ Span span_of(uint32_t first, uint32_t last) {
    const uint32_t w0 = first >> 5;
    return Span{w0, last >= first ? (last >> 5) - w0 + kWordsPer : 0xFFFFFFFFu};
}

__global__ __launch_bounds__(C3_DEC_NT, 4) void k_decode32(LayoutDev Ld, HuffDev hp, HuffDev hs,
                                                        const DecTab *__restrict__ tabs,
                                                        const DecodeTask *__restrict__ tasks,
                                                        int32_t *__restrict__ pix_out,
                                                        uint16_t *__restrict__ psi_out, uint32_t *err) {
    StreamLds<KSP> &SP = *(StreamLds<KSP> *)c3_dec_lds;
    StreamLds<KSQ> &SQ = *(StreamLds<KSQ> *)(c3_dec_lds + sizeof(StreamLds<KSP>));
    uint32_t *W = (uint32_t *)(c3_dec_lds + (kPair + 15) / 16 * 16);
    constexpr int C = 32;

    const DecodeTask task = tasks[blockIdx.x];
    const int seg = task.seg;
    const int64_t s0 = Ld.seg_off[seg];
    const int n = (int)(Ld.seg_off[seg + 1] - s0);
    const int band = Ld.seg_band[seg];
    const uint32_t npix = (uint32_t)Ld.band[band].npix;
    const uint32_t npsi = (uint32_t)Ld.band[band].npsi;
    const int tpi = hp.seg_table[seg], tqi = hs.seg_table[seg];
    const bool tabs_ok = tpi >= 0 && tpi < hp.ntable && tqi >= 0 && tqi < hs.ntable;
    const uint32_t *bp = hp.tables + hp.table_off[tabs_ok ? tpi : 0], *bq = hs.tables + hs.table_off[tabs_ok ? tqi : 0];
    const int64_t cp0 = hp.seg_chunk_off[seg], cq0 = hs.seg_chunk_off[seg];
    // the side index must hold ceil(n / C) chunks for this segment
    const int nch_idx = (int)min(hp.seg_chunk_off[seg + 1] - cp0, hs.seg_chunk_off[seg + 1] - cq0);
    const int64_t wp0 = hp.seg_word_off[seg], wq0 = hs.seg_word_off[seg];
    const int64_t nwp = hp.seg_word_off[seg + 1] - wp0, nwq = hs.seg_word_off[seg + 1] - wq0;
    const bool words_ok = nwp >= 0 && nwq >= 0 && nwp < (1ll << 29) && nwq < (1ll << 29);
    const __amdgpu_buffer_rsrc_t rsp = raw_buffer(hp.words + wp0, words_ok ? (int32_t)(4 * nwp) : 0);
    const __amdgpu_buffer_rsrc_t rsq = raw_buffer(hs.words + wq0, words_ok ? (int32_t)(4 * nwq) : 0);

    const int l = threadIdx.x;
    const int c = task.chunk0 + l;
    const bool active = l < task.nchunk && c < nch_idx;
    const int nact = min(task.nchunk, nch_idx - task.chunk0);  // the block's chunks with an index entry
    const __amdgpu_buffer_rsrc_t symp = symbol_buffer(hp, tabs_ok ? tpi : 0), symq = symbol_buffer(hs, tabs_ok ? tqi : 0);
    Stage<KSP / C3_DEC_NT> sp_;
    Stage<KSQ / C3_DEC_NT> sq_;
    sp_.load(symp, 0);
    sq_.load(symq, 0);
    uint32_t start_p = 0, start_q = 0;
    int32_t xp = 0, xq = 0;
    if (active) {
        start_p = hp.chunk_bit[cp0 + c];
        start_q = hs.chunk_bit[cq0 + c];
        xp = hp.chunk_prev[cp0 + c];
        xq = hs.chunk_prev[cq0 + c];
    }
    // stage the words when both streams' spans fit and the index is in order
    Span sp{0, 0}, sq{0, 0};
    bool fits = false;
    if (nact > 0) {
        const uint32_t fp = hp.chunk_bit[cp0 + task.chunk0], lp = hp.chunk_bit[cp0 + task.chunk0 + nact - 1];
        const uint32_t fq = hs.chunk_bit[cq0 + task.chunk0], lq = hs.chunk_bit[cq0 + task.chunk0 + nact - 1];
        sp = span_of(fp, lp);
        sq = span_of(fq, lq);
        fits = sp.n <= kPairWords && sq.n <= kPairWords && sp.n + sq.n <= kPairWords;
        fits = !__syncthreads_or(!fits || (active && (start_p < fp || start_p > lp || start_q < fq || start_q > lq)));
    }
    {
        Stage<16> wq_, wp_;
        if (fits) {
            wp_.load(rsp, sp.w0);
            wq_.load(rsq, sq.w0);
        }
        stage_table(SP, tabs + (tabs_ok ? tpi : 0));
        stage_table(SQ, tabs + hp.ntable + (tabs_ok ? tqi : 0));
        sp_.symbols(SP);
        sq_.symbols(SQ);
        if (fits) {
            wp_.words(W, sp.n);
            wq_.words(W + sp.n, sq.n);
            stage_rest(W, rsp, sp.w0, sp.n);
            stage_rest(W + sp.n, rsq, sq.w0, sq.n);
        }
    }
    __syncthreads();
    const bool codes_ok = tabs_ok && SP.T.ok && SQ.T.ok && SQ.T.nsym < 65535;
    uint32_t bad = codes_ok ? 0u : C3_ERR_CODE;
    if (l < task.nchunk && c >= nch_idx) bad |= C3_ERR_CHUNK;
    if (!words_ok) bad |= C3_ERR_CHUNK;
    // every chunk of the wave is there and whole
    const bool full_wave = __ballot(active && (c + 1) * C <= n) == ~0ull;
    if (active && codes_ok && words_ok) {
        const int ns = min(C, n - c * C);
        int32_t bitp = 0, bitq = 0;  // bits consumed by this chunk's codes
        int32_t *po = pix_out + s0 + (int64_t)c * C;
        uint16_t *qo = psi_out + s0 + (int64_t)c * C;
        // the next eight codes of both streams; FULL: all of them belong to the chunk
        auto eight = [&](auto full, auto &P, auto &Q, int k0, int *vp, int *vq, uint32_t p0, uint32_t q0) {
            constexpr bool FULL = decltype(full)::value;
            uint32_t ip[8], iq[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (!FULL && k0 + k == ns) {  // the segment's last chunk may be short
                    bitp = (int32_t)(P.pos - p0);
                    bitq = (int32_t)(Q.pos - q0);
                }
                // the two streams' reads are issued together
                if (k % 2 == 0) {
                    P.read();
                    Q.read();
                }
                const uint32_t wp = P.window(), wq = Q.window();
                const int ep = SP.T.lut[wp >> SPLIT], eq = SQ.T.lut[wq >> SPLIT];
                P.L = ep;
                Q.L = eq;
                P.inv = Q.inv = false;
                if (!(settled(ep) && settled(eq))) {
                    P.search(wp, ep);
                    Q.search(wq, eq);
                    if ((FULL || k0 + k < ns) && (P.inv || Q.inv)) bad |= C3_ERR_CODE;
                }
                P.consume();
                Q.consume();
                ip[k] = P.index(wp);
                iq[k] = Q.index(wq);
                vp[k] = P.value(ip[k]);
                vq[k] = Q.value(iq[k]);
            }
            escapes(P, vp, ip);
            escapes(Q, vq, iq);
            uint32_t mp = 0, mq = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const bool v = FULL || k0 + k < ns;
                P.x += v ? vp[k] : 0;
                Q.x += v ? vq[k] : 0;
                vp[k] = P.x;
                vq[k] = Q.x;
                mp = max(mp, (uint32_t)P.x);
                mq = max(mq, (uint32_t)Q.x);
            }
            if (mp >= npix || mq >= npsi) {  // out of range: reported, stored as 0
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if ((uint32_t)vp[k] >= npix) {
                        if (FULL || k0 + k < ns) bad |= C3_ERR_PIX;
                        vp[k] = 0;
                    }
                    if ((uint32_t)vq[k] >= npsi) {
                        if (FULL || k0 + k < ns) bad |= C3_ERR_PSI;
                        vq[k] = 0;
                    }
                }
            }
        };
        auto parse = [&](auto staged) {
            constexpr bool ST = decltype(staged)::value;
            LaneStream<KSP, ST> P{SP, W, rsp, symp, ST ? start_p - 32 * sp.w0 : start_p, xp};
            LaneStream<KSQ, ST> Q{SQ, W + sp.n, rsq, symq, ST ? start_q - 32 * sq.w0 : start_q, xq};
            const uint32_t p0 = P.pos, q0 = Q.pos;
            for (int k0 = 0; k0 < ns; k0 += 8) {
                int vp[8], vq[8];
                eight(std::false_type{}, P, Q, k0, vp, vq, p0, q0);
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (k0 + k < ns) {
                        po[k0 + k] = vp[k];
                        qo[k0 + k] = (uint16_t)vq[k];
                    }
            }
            if (ns % 8 == 0) {
                bitp = (int32_t)(P.pos - p0);
                bitq = (int32_t)(Q.pos - q0);
            }
            xp = P.x;
            xq = Q.x;
        };
        if (fits && full_wave) {
            LaneStream<KSP, true> P{SP, W, rsp, symp, start_p - 32 * sp.w0, xp};
            LaneStream<KSQ, true> Q{SQ, W + sp.n, rsq, symq, start_q - 32 * sq.w0, xq};
            uint32_t pv[C], qv[C / 2];
#pragma unroll
            for (int k0 = 0; k0 < C; k0 += 8) {
                int vp[8], vq[8];
                eight(std::true_type{}, P, Q, k0, vp, vq, 0, 0);
#pragma unroll
                for (int k = 0; k < 8; ++k) pv[k0 + k] = (uint32_t)vp[k];
#pragma unroll
                for (int k = 0; k < 8; k += 2) qv[(k0 + k) / 2] = (uint32_t)vq[k] | ((uint32_t)vq[k + 1] << 16);
            }
            bitp = (int32_t)(P.pos - (start_p - 32 * sp.w0));
            bitq = (int32_t)(Q.pos - (start_q - 32 * sq.w0));
            xp = P.x;
            xq = Q.x;
            const int64_t o = s0 + (int64_t)(task.chunk0 + (l & ~63)) * C;  // the wave's first sample
            store_rows<Store16>(pv, (char *)(pix_out + o), 4 * C, 0);
            store_rows<Store16>(pv + 16, (char *)(pix_out + o), 4 * C, 64);
            store_rows<Store16h>(qv, (char *)(psi_out + o), 2 * C, 0);
        } else if (fits) {
            parse(std::true_type{});
        } else {
            parse(std::false_type{});
        }
        // chunk boundary consistency with the side index: the codes of chunk c
        // end where chunk c + 1 starts, and the running value meets its stored one
        if (c + 1 < nch_idx) {
            if ((int64_t)start_p + bitp != (int64_t)hp.chunk_bit[cp0 + c + 1] || xp != hp.chunk_prev[cp0 + c + 1])
                bad |= C3_ERR_CHUNK;
            if ((int64_t)start_q + bitq != (int64_t)hs.chunk_bit[cq0 + c + 1] || xq != hs.chunk_prev[cq0 + c + 1])
                bad |= C3_ERR_CHUNK;
        }
        if (ns > 0) {
            if ((int64_t)start_p + bitp > 32 * nwp) bad |= C3_ERR_CHUNK;
            if ((int64_t)start_q + bitq > 32 * nwq) bad |= C3_ERR_CHUNK;
        }
    }
    if (bad) atomicOr(err, bad);
}

// One integer stream per segment (the TOD or the flag words), without range
// checks; KIND as in k_decode1.
template <int KIND>
__global__ __launch_bounds__(C3_DEC_NT, 6) void k_decode32_1(LayoutDev Ld, HuffDev h, const DecTab *__restrict__ tabs,
                                                          const DecodeTask *__restrict__ tasks, double quantum,
                                                          uint32_t flag_mask, void *__restrict__ out,
                                                          uint8_t *__restrict__ mask_out, uint32_t *err) {
    StreamLds<KSQ> &S = *(StreamLds<KSQ> *)c3_dec_lds;
    uint32_t *W = (uint32_t *)(c3_dec_lds + (kOne + 15) / 16 * 16);
    constexpr int C = 32;
    const DecodeTask task = tasks[blockIdx.x];
    const int seg = task.seg;
    const int64_t s0 = Ld.seg_off[seg];
    const int n = (int)(Ld.seg_off[seg + 1] - s0);
    const int ti = h.seg_table[seg];
    const bool tabs_ok = ti >= 0 && ti < h.ntable;
    const uint32_t *blob = h.tables + h.table_off[tabs_ok ? ti : 0];
    const int64_t c0 = h.seg_chunk_off[seg];
    const int nch_idx = (int)(h.seg_chunk_off[seg + 1] - c0);
    const int64_t w0 = h.seg_word_off[seg];
    const int64_t nw = h.seg_word_off[seg + 1] - w0;
    const bool words_ok = nw >= 0 && nw < (1ll << 29);
    const __amdgpu_buffer_rsrc_t rs = raw_buffer(h.words + w0, words_ok ? (int32_t)(4 * nw) : 0);
    const int l = threadIdx.x;
    const int c = task.chunk0 + l;
    const bool active = l < task.nchunk && c < nch_idx;
    const int nact = min(task.nchunk, nch_idx - task.chunk0);
    const __amdgpu_buffer_rsrc_t sym = symbol_buffer(h, tabs_ok ? ti : 0);
    Stage<KSQ / C3_DEC_NT> s_;
    s_.load(sym, 0);
    uint32_t start = 0;
    int32_t x = 0;
    if (active) {
        start = h.chunk_bit[c0 + c];
        x = h.chunk_prev[c0 + c];
    }
    Span sp{0, 0};
    bool fits = false;
    if (nact > 0) {
        const uint32_t f = h.chunk_bit[c0 + task.chunk0], la = h.chunk_bit[c0 + task.chunk0 + nact - 1];
        sp = span_of(f, la);
        fits = !__syncthreads_or(sp.n > kOneWords || (active && (start < f || start > la)));
    }
    {
        Stage<16> w_;
        if (fits) w_.load(rs, sp.w0);
        stage_table(S, tabs + (tabs_ok ? ti : 0));
        s_.symbols(S);
        if (fits) {
            w_.words(W, sp.n);
            stage_rest(W, rs, sp.w0, sp.n);
        }
    }
    __syncthreads();
    const bool codes_ok = tabs_ok && S.T.ok;
    uint32_t bad = codes_ok ? 0u : C3_ERR_CODE;
    if (l < task.nchunk && c >= nch_idx) bad |= C3_ERR_CHUNK;
    if (!words_ok) bad |= C3_ERR_CHUNK;
    const bool full_wave = __ballot(active && (c + 1) * C <= n) == ~0ull;
    if (active && codes_ok && words_ok) {
        const int ns = min(C, n - c * C);
        int32_t bits = 0;
        const int64_t o0 = s0 + (int64_t)c * C;
        auto eight = [&](auto full, auto &P, int k0, int *v, uint32_t p0) {
            constexpr bool FULL = decltype(full)::value;
            uint32_t ix[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (!FULL && k0 + k == ns) bits = (int32_t)(P.pos - p0);
                if (k % 2 == 0) P.read();
                const uint32_t w = P.window();
                const int e = S.T.lut[w >> SPLIT];
                P.L = e;
                P.inv = false;
                if (!settled(e)) {
                    P.search(w, e);
                    if ((FULL || k0 + k < ns) && P.inv) bad |= C3_ERR_CODE;
                }
                P.consume();
                ix[k] = P.index(w);
                v[k] = P.value(ix[k]);
            }
            escapes(P, v, ix);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                P.x += FULL || k0 + k < ns ? v[k] : 0;
                v[k] = P.x;
            }
        };
        auto parse = [&](auto staged) {
            constexpr bool ST = decltype(staged)::value;
            LaneStream<KSQ, ST> P{S, W, rs, sym, ST ? start - 32 * sp.w0 : start, x};
            const uint32_t p0 = P.pos;
            for (int k0 = 0; k0 < ns; k0 += 8) {
                int v[8];
                eight(std::false_type{}, P, k0, v, p0);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int64_t o = o0 + k0 + k;
                    if (k0 + k >= ns) continue;
                    if constexpr (KIND == 0) {
                        ((float *)out)[o] = (float)(quantum * (double)v[k]);
                    } else if constexpr (KIND == 1) {
                        ((double *)out)[o] = quantum * (double)v[k];
                    } else {
                        if (out) ((uint32_t *)out)[o] = (uint32_t)v[k];
                        if (mask_out) mask_out[o] = ((uint32_t)v[k] & flag_mask) == 0u;
                    }
                }
            }
            if (ns % 8 == 0) bits = (int32_t)(P.pos - p0);
            x = P.x;
        };
        if (fits && full_wave) {
            LaneStream<KSQ, true> P{S, W, rs, sym, start - 32 * sp.w0, x};
            const int64_t o = s0 + (int64_t)(task.chunk0 + (l & ~63)) * C;  // the wave's first sample
            constexpr int SZ = KIND == 1 ? 8 : 4;
            char *ow = (char *)out + o * SZ;
            uint32_t mb[8];  // mask bytes of the chunk
#pragma unroll
            for (int h = 0; h < C; h += 16) {
                uint32_t u[16 * SZ / 4];
#pragma unroll
                for (int k0 = 0; k0 < 16; k0 += 8) {
                    int v[8];
                    eight(std::true_type{}, P, h + k0, v, 0);
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        if constexpr (KIND == 0) {
                            u[k0 + k] = __float_as_uint((float)(quantum * (double)v[k]));
                        } else if constexpr (KIND == 1) {
                            const uint64_t b = (uint64_t)__double_as_longlong(quantum * (double)v[k]);
                            u[2 * (k0 + k)] = (uint32_t)b;
                            u[2 * (k0 + k) + 1] = (uint32_t)(b >> 32);
                        } else {
                            u[k0 + k] = (uint32_t)v[k];
                            const uint32_t m = ((uint32_t)v[k] & flag_mask) == 0u ? 1u << (8 * (k & 3)) : 0u;
                            uint32_t &w = mb[(h + k0 + k) / 4];
                            w = k % 4 ? w | m : m;
                        }
                    }
                }
                if (KIND != 2 || out) {
                    store_rows<Store16>(u, ow, C * SZ, (uint32_t)(h * SZ));
                    if constexpr (KIND == 1) store_rows<Store16>(u + 16, ow, C * SZ, (uint32_t)(h * SZ) + 64);
                }
            }
            if constexpr (KIND == 2) {
                if (mask_out) {  // the lane's 32 bytes, of any alignment
                    ((Store16b *)(mask_out + o0))[0].v = u32x4{mb[0], mb[1], mb[2], mb[3]};
                    ((Store16b *)(mask_out + o0))[1].v = u32x4{mb[4], mb[5], mb[6], mb[7]};
                }
            }
            bits = (int32_t)(P.pos - (start - 32 * sp.w0));
            x = P.x;
        } else if (fits) {
            parse(std::true_type{});
        } else {
            parse(std::false_type{});
        }
        if (c + 1 < nch_idx) {
            if ((int64_t)start + bits != (int64_t)h.chunk_bit[c0 + c + 1] || x != h.chunk_prev[c0 + c + 1])
                bad |= C3_ERR_CHUNK;
        }
        if (ns > 0 && (int64_t)start + bits > 32 * nw) bad |= C3_ERR_CHUNK;
    }
    if (bad) atomicOr(err, bad);
}

// ------------------------------------------------------- allocation-free variant
// Scratch of decode_pointing_noalloc: the decoding tables of both streams,
// then the work list, in one static array per device (held until the process
// ends).  Host code uses only the address hipGetSymbolAddress returns for it.
static __device__ __align__(256) unsigned char scratch[C3_NOALLOC_BYTES];

// The work list of k_decode in segment order: segment s takes
// ceil(ceil(n_s / C) / C3_DEC_NT) tasks, starting at the sum of the counts before
// it.  One block scans the counts 1024 segments at a time.  Exactly ntask
// entries are written: the host counts them from its mirror of the offsets;
// entries the device offsets do not fill are empty tasks (no chunk), and
// none is written past ntask, whatever the device offsets hold.
__global__ __launch_bounds__(1024) void k_decode_tasks(const int64_t *__restrict__ seg_off, int nseg, int C,
                                                       int ntask, DecodeTask *__restrict__ tasks) {
    __shared__ int32_t pre[1024];
    __shared__ int64_t carry;
    const int tid = threadIdx.x;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nseg; base += 1024) {
        const int s = base + tid;
        int nch = 0, cnt = 0;
        if (s < nseg) {
            const int64_t n = seg_off[s + 1] - seg_off[s];
            nch = n > 0 ? (int)((n + C - 1) / C) : 0;
            cnt = (nch + C3_DEC_NT - 1) / C3_DEC_NT;
        }
        pre[tid] = cnt;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {  // inclusive scan
            const int v = tid >= o ? pre[tid - o] : 0;
            __syncthreads();
            pre[tid] += v;
            __syncthreads();
        }
        const int64_t start = carry + pre[tid] - cnt;
        for (int j = 0; j < cnt && start + j < ntask; ++j)
            tasks[start + j] = DecodeTask{s, j * C3_DEC_NT, min(C3_DEC_NT, nch - j * C3_DEC_NT), 0};
        __syncthreads();
        if (tid == 1023) carry += pre[1023];
        __syncthreads();
    }
    for (int64_t i = carry + tid; i < ntask; i += 1024) tasks[i] = DecodeTask{0, 0, 0, 0};
}

// One integer stream per segment (the TOD or the flag words): the same chunk
// parse and undifferencing as k_decode, without range checks; the tile is
// written as KIND 0: FP32 quantum * x, 1: FP64 quantum * x, 2: flag words
// (and, if mask_out, the mask byte (x & flag_mask) == 0).
template <int KIND>
__global__ __launch_bounds__(C3_DEC_NT) void k_decode1(LayoutDev Ld, HuffDev h, const DecTab *__restrict__ tabs,
                                                   const DecodeTask *__restrict__ tasks, double quantum,
                                                   uint32_t flag_mask, void *__restrict__ out,
                                                   uint8_t *__restrict__ mask_out, uint32_t *err) {
    __shared__ DecTab cp;
    __shared__ int32_t tp[C3_DEC_NT * GP];
    __shared__ uint32_t blk_err;

    const DecodeTask task = tasks[blockIdx.x];
    const int seg = task.seg;
    const int tid = threadIdx.x;
    const int64_t s0 = Ld.seg_off[seg];
    const int n = (int)(Ld.seg_off[seg + 1] - s0);
    const int C = h.chunk_len;

    const int ti = h.seg_table[seg];
    const bool tabs_ok = ti >= 0 && ti < h.ntable;
    {
        const uint4 *sp = (const uint4 *)(tabs + (tabs_ok ? ti : 0));
        uint4 *dp = (uint4 *)&cp;
        for (int i = tid; i < (int)(sizeof(DecTab) / 16); i += C3_DEC_NT) dp[i] = sp[i];
        if (tid == 0) blk_err = 0;
    }
    __syncthreads();
    const bool codes_ok = tabs_ok && cp.ok;
    const __amdgpu_buffer_rsrc_t sym = raw_buffer(h.tables + h.table_off[tabs_ok ? ti : 0] + 34, 4 * cp.nsym);

    const int l = tid;
    const int c = task.chunk0 + l;
    const int nch_idx = (int)(h.seg_chunk_off[seg + 1] - h.seg_chunk_off[seg]);
    const bool active = l < task.nchunk && c < nch_idx;
    uint32_t bad = codes_ok ? 0u : C3_ERR_CODE;
    if (l < task.nchunk && c >= nch_idx) bad |= C3_ERR_CHUNK;
    BitReader rd;
    int ns = 0;
    int32_t x = 0, bits = 0;
    uint32_t start = 0;
    const int64_t w0 = h.seg_word_off[seg];
    const int64_t nw = h.seg_word_off[seg + 1] - w0;
    const bool words_ok = nw >= 0 && nw < (1ll << 29);
    if (!words_ok) bad |= C3_ERR_CHUNK;
    const __amdgpu_buffer_rsrc_t rs = raw_buffer(h.words + w0, words_ok ? (int32_t)(4 * nw) : 0);
    if (active) {
        const int64_t g = h.seg_chunk_off[seg] + c;
        start = h.chunk_bit[g];
        rd.init(rs, start);
        x = h.chunk_prev[g];
        ns = (codes_ok && words_ok) ? min(C, n - c * C) : 0;
    }
    const int nround = (C + G - 1) / G;
    for (int r = 0; r < nround; ++r) {
        const int k0 = r * G;
        if (active && k0 < ns) {
#pragma unroll 4
            for (int k = 0; k < G; ++k) {
                int L;
                const int32_t ix = rd.next(cp, L);
                const bool v = k0 + k < ns;
                bad |= (v && L == 0) ? C3_ERR_CODE : 0u;
                bits += v ? L : 0;
                tp[l * GP + k] = ix;
            }
#pragma unroll
            for (int hh = 0; hh < G; hh += G / 2) {
                int32_t gv[G / 2];
#pragma unroll
                for (int k = 0; k < G / 2; ++k) gv[k] = (int32_t)buf_word(sym, (uint32_t)tp[l * GP + hh + k]);
#pragma unroll
                for (int k = 0; k < G / 2; ++k) {
                    x += (k0 + hh + k < ns) ? gv[k] : 0;
                    tp[l * GP + hh + k] = x;
                }
            }
        }
        __syncthreads();
#pragma unroll 4
        for (int m = 0; m < G; ++m) {
            const int q = m * C3_DEC_NT + tid;
            const int ll = q >> 4, kk = q & 15;
            const int cc = task.chunk0 + ll;
            const int t = cc * C + k0 + kk;
            if (ll < task.nchunk && cc < nch_idx && k0 + kk < C && t < n && codes_ok && words_ok) {
                const int32_t v = tp[ll * GP + kk];
                if constexpr (KIND == 0) {
                    ((float *)out)[s0 + t] = (float)(quantum * (double)v);
                } else if constexpr (KIND == 1) {
                    ((double *)out)[s0 + t] = quantum * (double)v;
                } else {
                    if (out) ((uint32_t *)out)[s0 + t] = (uint32_t)v;
                    if (mask_out) mask_out[s0 + t] = ((uint32_t)v & flag_mask) == 0u;
                }
            }
        }
        __syncthreads();
    }
    if (active && codes_ok && c + 1 < nch_idx) {
        const int64_t g = h.seg_chunk_off[seg] + c + 1;
        if ((int64_t)start + bits != (int64_t)h.chunk_bit[g] || x != h.chunk_prev[g]) bad |= C3_ERR_CHUNK;
    }
    if (active && ns > 0 && (int64_t)start + bits > 32 * nw) bad |= C3_ERR_CHUNK;
    if (bad) atomicOr(&blk_err, bad);
    __syncthreads();
    if (tid == 0 && blk_err) atomicOr(err, blk_err);
}

}  // namespace

namespace c3 {

namespace {
// The LDS decoders take streams of 32-symbol chunks whose words usually fit a
// block's LDS (512 chunks of `words` words each on average, with a twentieth
// to spare); blocks whose words do not fit read them from memory.
bool staged_words(int64_t words, int64_t nchunk, uint32_t room) {
    return nchunk > 0 && (double)words / (double)nchunk * C3_DEC_NT * 1.05 + 2 * kWordsPer <= (double)room;
}

template <int KIND>
void launch_decode1(hipStream_t st, const LayoutDev &L, const HuffDev &h, DecTab *tabs, const DecodeTask *tasks,
                    int ntask, double quantum, uint32_t flag_mask, void *out, uint8_t *mask_out, uint32_t *err) {
    const dim3 g(ntask), b(C3_DEC_NT);
    HuffDev none = h;
    none.ntable = 0;
    hipLaunchKernelGGL(k_tables, dim3(h.ntable), dim3(1024), 0, st, h, none, tabs);
    if (h.chunk_len == 32 && staged_words(h.nwords, h.nchunk, kOneWords))
        hipLaunchKernelGGL(k_decode32_1<KIND>, g, b, kOneLds, st, L, h, tabs, tasks, quantum, flag_mask, out, mask_out,
                           err);
    else
        hipLaunchKernelGGL(k_decode1<KIND>, g, b, 0, st, L, h, tabs, tasks, quantum, flag_mask, out, mask_out, err);
}
}  // namespace

hipError_t launch_decode_stream(hipStream_t st, const LayoutDev &L, const HuffDev &h, DecTab *tabs,
                                const DecodeTask *tasks, int ntask, int kind, double quantum,
                                uint32_t flag_mask, void *out, uint8_t *mask_out, uint32_t *err) {
    if (ntask <= 0) return hipSuccess;
    auto *go = kind == 0 ? launch_decode1<0> : kind == 1 ? launch_decode1<1> : launch_decode1<2>;
    go(st, L, h, tabs, tasks, ntask, quantum, flag_mask, out, mask_out, err);
    return hipGetLastError();
}

hipError_t dec_init_attributes() {
    static PerDevice inits;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    return inits.once<hipError_t>(dev, [&] {
        for (const void *f : {(const void *)k_decode32, (const void *)k_decode32_1<0>, (const void *)k_decode32_1<1>,
                              (const void *)k_decode32_1<2>}) {
            const hipError_t r = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, C3_LDS_MAX - 4096);
            if (r != hipSuccess) e = r;
        }
        return e;
    });
}

hipError_t noalloc_scratch(void **ptr) {
    // one address per device, looked up once with that device current
    static std::mutex mu;
    static void *addr[C3_MAX_DEVICES] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= C3_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t launch_decode_noalloc(hipStream_t st, const LayoutDev &L, const HuffDev &hp, const HuffDev &hs,
                                 void *scratch_ptr, int ntask, int32_t *pix_out, uint16_t *psi_out,
                                 uint32_t *err) {
    if (ntask <= 0) return hipSuccess;
    DecTab *tabs = (DecTab *)scratch_ptr;
    DecodeTask *tasks = (DecodeTask *)((char *)scratch_ptr + noalloc_task_offset(hp.ntable + hs.ntable));
    hipLaunchKernelGGL(k_decode_tasks, dim3(1), dim3(1024), 0, st, L.seg_off, L.nseg, hp.chunk_len, ntask, tasks);
    return launch_decode(st, L, hp, hs, tabs, tasks, ntask, pix_out, psi_out, err);
}

hipError_t launch_decode(hipStream_t st, const LayoutDev &L, const HuffDev &hp, const HuffDev &hs,
                         DecTab *tabs, const DecodeTask *tasks, int ntask, int32_t *pix_out,
                         uint16_t *psi_out, uint32_t *err) {
    if (ntask <= 0) return hipSuccess;
    const dim3 g(ntask), b(C3_DEC_NT);
    hipLaunchKernelGGL(k_tables, dim3(hp.ntable + hs.ntable), dim3(1024), 0, st, hp, hs, tabs);
    if (hp.chunk_len == 32 && staged_words(hp.nwords + hs.nwords, hp.nchunk, kPairWords))
        hipLaunchKernelGGL(k_decode32, g, b, kPairLds, st, L, hp, hs, tabs, tasks, pix_out, psi_out, err);
    else
        hipLaunchKernelGGL(k_decode, g, b, 0, st, L, hp, hs, tabs, tasks, pix_out, psi_out, err);
    return hipGetLastError();
}

}  // namespace c3
