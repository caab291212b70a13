// Entropy coding of the quantized coefficients (Sec. 3.4): every channel's coefficient vector,
// in coefficient order, is cut into blocks of B values, and every block is coded on its own by
// the adaptive run-length / Golomb-Rice coder the paper uses, so the blocks code in parallel.
// The paper gives no parameters; the coder follows the published method with these choices:
//   * block b = j * C + c holds coefficients j*B .. j*B + B - 1 of channel c; its code is a
//     whole number of 32-bit words, filled from the most significant bit;
//   * two adaptive parameters with 3 fractional bits, kp (run mode while kp >> 3 > 0) and krp
//     (Golomb-Rice parameter kr = krp >> 3), both starting at 8 and kept within 0..80;
//   * run mode: a 0 bit per 2^k zeros (kp += 4), then a 1 and the remaining count in k bits,
//     then, unless the block ends, the sign bit and GR(|v| - 1) of the value that ends the run
//     (kp -= 6); Golomb-Rice mode: GR(2v) or GR(-2v - 1) (kp += 3 after a zero, -= 3 otherwise);
//   * GR(u): u >> kr ones, a 0, the kr low bits; 24 ones then u in 32 bits when u >> kr >= 24;
//     krp -= 2 when u >> kr = 0, += u >> kr when it is above 1.
// A thread codes one block, and a workgroup is one wave: it takes RPW = floor(64 / C) block rows (one
// for C > 32), thread t the block b = blockIdx RPW C + t, so a step of the wave touches whole matrix
// rows (C consecutive values per block row) and needs no staging.
//
// What bounds it: the blocks are serial chains, so a frame's work is (instructions per value) x
// B x (waves per SIMD) issue slots of four cycles: 1954 waves over 1024 SIMDs for a 1M x 56 matrix
// in blocks of 512. Every value therefore takes one straight-line step in which run mode and
// Golomb-Rice mode are selected, not branched on (lanes of a wave are in different modes almost
// always, so a branch costs both sides), a code of at most 31 (encoder) or 32 (decoder) bits is
// handled as one word, and only longer codes (an escape, or a long quotient after a long run)
// take a branch of their own. 1M x 56, blocks of 512: counting 294 -> 73 us (43 instructions per
// value), writing 557 -> 150 us (about 95), decoding 1326 -> 229 us (about 135), against a coder that
// branched on the mode, kept 64-bit bit buffers and (decoding) waited on a global load per word;
// the matrix
// (224 MB) and its code (22 MB) move at about a fifth of a copy's rate: issue slots bound all three.
#include "gsc_device.h"

namespace gsc {

constexpr int RLGR_THREADS = WAVE;  // one thread per block, one wave per workgroup
constexpr int RLGR_STEP = 16;       // values per thread between two refills
constexpr uint32_t RLGR_FRAC = 3, RLGR_PMAX = 80, RLGR_START = 8;
constexpr int RLGR_RUN_UP = 4, RLGR_RUN_DOWN = 6, RLGR_GR_UP = 3, RLGR_GR_DOWN = 3;
constexpr uint32_t RLGR_ESCAPE = 24;
static_assert(GSC_MAX_CHANNELS <= RLGR_THREADS, "at least one block row per wave");

// Block rows per wave.
__host__ __device__ inline uint32_t rl_rows(uint32_t C) { return (uint32_t)RLGR_THREADS / C; }

// A parameter (kp or krp, 0..80) after an adaptation step.
__device__ inline uint32_t rl_adapt(uint32_t p, int d) { return (uint32_t)min(max((int)p + d, 0), (int)RLGR_PMAX); }
// krp's step after a Golomb-Rice quotient q (bounded, so that it cannot overflow).
__device__ inline int rl_gr_step(uint32_t q) { return q > 1 ? (int)min(q, RLGR_PMAX) : 2 * (int)q - 2; }
__device__ inline uint32_t rl_ones(uint32_t n) { return (1u << n) - 1u; }  // n < 32

// This thread's block: its rows [r0, r0 + L) of channel c, its index b; L = 0 for a thread without one.
// The matrix offset of its first value is split into the wave's uniform part (ubase, values) and the
// thread's (off, bytes; at most 64 x 65536 x 4 for C = 1 and 2 x 65536 x 64 x 4 for the widest).
struct RlBlock {
    uint32_t b, L, off;
    size_t ubase;
    uint32_t lmin, lmax;  // over the wave's blocks
};
__device__ inline RlBlock rl_block(uint32_t nv, uint32_t C, uint32_t B, uint32_t nb)
{
    RlBlock k;
    const uint32_t tid = threadIdx.x, rpw = rl_rows(C), j0 = blockIdx.x * rpw, dj = tid / C;
    const bool on = tid < rpw * C && j0 + dj < nb;
    k.b = blockIdx.x * rpw * C + tid;
    k.L = on ? min(B, nv - (j0 + dj) * B) : 0u;
    k.ubase = (size_t)j0 * B * C;
    k.off = on ? 4u * (dj * B * C + (tid - dj * C)) : 0u;
    k.lmax = wave_umax(k.L);
    k.lmin = wave_umin(on ? k.L : 0xFFFFFFFFu);
    return k;
}

// ------------------------------------------------------------------------------ encoder
// Counts the bits of a block (W = false) or writes its words (W = true) at `out`.
template <bool W>
struct RlgrEnc {
    uint32_t kp = RLGR_START, krp = RLGR_START;
    uint32_t run = 0;    // zeros of the open run segment not yet sent
    bool open = false;   // the last value was a zero in run mode
    uint32_t nbits = 0;  // (W = false)
    uint32_t cur = 0, fill = 0;  // (W = true) the word being filled from its top, bits filled (< 32)
    GAS uint32_t *out = nullptr;

    __device__ void put(uint32_t v, uint32_t n)  // the value v < 2^n, n <= 31
    {
        const uint32_t c = v << ((32u - n) & 31u);  // (n = 0: v = 0)
        cur |= c >> fill;
        fill += n;
        if (fill >= 32) {
            *out++ = cur;
            fill -= 32;
            cur = c << (n - fill);  // (the n - fill bits that went out: 1..31)
        }
    }
    __device__ __attribute__((always_inline)) void value(int32_t v)
    {
        const uint32_t k = kp >> RLGR_FRAC, kr = krp >> RLGR_FRAC;
        const bool rm = k != 0, z = v == 0, in_run = rm && z;  // (run mode while kp >> 3 > 0)
        const uint32_t zz = ((uint32_t)v << 1) ^ (uint32_t)(v >> 31);  // 2v or -2v - 1
        const uint32_t u = rm ? (zz - 1u) >> 1 : zz;                   // |v| - 1 after a run
        // a zero of a run sends nothing but a 0 bit when the segment's 2^k zeros are complete; its
        // quotient is set to 1, the one that leaves krp alone
        const uint32_t q = in_run ? 1u : u >> kr;
        const uint32_t run1 = run + 1u;
        const bool full = (run1 >> k) != 0;
        const uint32_t n1 = rm ? k + 2u : 0u, n2 = q + 1u + kr;
        if (W) {
            uint32_t n = n1 + n2;
            if (q >= RLGR_ESCAPE || n > 31u) {  // (a zero of a run has n <= 24)
                const uint32_t s = (uint32_t)v >> 31;
                if (rm) put((((1u << k) | run) << 1) | s, n1);
                if (q < RLGR_ESCAPE) {
                    put(rl_ones(q) << 1, q + 1u);
                    put(u & rl_ones(kr), kr);
                } else {
                    put(rl_ones(RLGR_ESCAPE), RLGR_ESCAPE);
                    put(u >> 16, 16);
                    put(u & 0xFFFFu, 16);
                }
            } else {
                const uint32_t pre = rm ? (((1u << k) | run) << 1) | ((uint32_t)v >> 31) : 0u;
                const uint32_t code = (pre << n2) | (rl_ones(q) << (kr + 1u)) | (u & rl_ones(kr));
                put(in_run ? 0u : code, in_run ? (full ? 1u : 0u) : n);
            }
        } else {
            nbits += in_run ? (full ? 1u : 0u) : n1 + (q < RLGR_ESCAPE ? n2 : RLGR_ESCAPE + 32u);
        }
        krp = rl_adapt(krp, rl_gr_step(q));
        const int up = rm ? (full ? RLGR_RUN_UP : 0) : RLGR_GR_UP;  // after a zero
        kp = rl_adapt(kp, z ? up : (rm ? -RLGR_RUN_DOWN : -RLGR_GR_DOWN));
        run = in_run && !full ? run1 : 0u;
        open = in_run;
    }
    __device__ void finish()
    {
        const uint32_t k = kp >> RLGR_FRAC;
        if (W) {
            if (open) put((1u << k) | run, k + 1u);
            if (fill > 0) *out = cur;
        } else if (open) {
            nbits += k + 1u;
        }
    }
};

struct RlgrArgs {
    const int32_t *q;   // [nv][C]
    uint32_t nv, C, B, nb;
    uint8_t *out;       // stream: header, block table, words
    uint64_t out_cap;
    uint64_t *status;   // look-back status of the waves' block rows (zeroed)
    uint32_t *err;      // device error word (first word of the workspace)
    int32_t *info;
};

__device__ inline GAS uint32_t *rl_table(uint8_t *out) { return gp(reinterpret_cast<uint32_t *>(out + sizeof(gsc_rlgr_header))); }
__device__ inline GAS uint32_t *rl_words(uint8_t *out, uint32_t NB)
{
    return gp(reinterpret_cast<uint32_t *>(out + sizeof(gsc_rlgr_header))) + NB + 1;
}

// Codes this thread's block (count or write). The next RLGR_STEP values of every thread are
// loaded (at positions clamped to its block) while the current ones are coded.
template <bool W>
__device__ inline void rl_encode_block(const RlgrArgs &a, const RlBlock &k, RlgrEnc<W> &enc)
{
    const GAS char *src = reinterpret_cast<const GAS char *>(gp(a.q) + k.ubase);
    const uint32_t pitch = 4u * a.C, last = k.off + (k.L ? k.L - 1u : 0u) * pitch;
    int32_t v[RLGR_STEP];
    uint32_t off = k.off;
    auto load = [&](int32_t (&x)[RLGR_STEP]) {
#pragma unroll
        for (int u = 0; u < RLGR_STEP; ++u) {
            x[u] = *reinterpret_cast<const GAS int32_t *>(src + min(off, last));
            off += pitch;
        }
    };
    load(v);
    uint32_t i = 0;
    for (; i < k.lmax; i += RLGR_STEP) {
        int32_t w[RLGR_STEP];
        load(w);
        if (i + RLGR_STEP <= k.lmin) {
            if (k.L) {
#pragma unroll
                for (int u = 0; u < RLGR_STEP; ++u) enc.value(v[u]);
            }
        } else {  // (past the wave's shortest block: the last block row, which is shorter)
#pragma unroll 1
            for (int u = 0; u < RLGR_STEP; ++u) {
                int32_t x = v[0];
#pragma unroll
                for (int y = 1; y < RLGR_STEP; ++y) x = u == y ? v[y] : x;
                if (i + u < k.L) enc.value(x);
            }
        }
#pragma unroll
        for (int u = 0; u < RLGR_STEP; ++u) v[u] = w[u];
    }
    if (k.L) enc.finish();
}

// Pass 1: every block's length in words, the blocks' word offsets (an exclusive scan over the
// waves by decoupled look-back), the block table and the header.
__global__ __launch_bounds__(RLGR_THREADS) void k_rlgr_count(RlgrArgs a)
{
    const uint32_t tid = threadIdx.x, NB = a.nb * a.C;
    const RlBlock k = rl_block(a.nv, a.C, a.B, a.nb);
    RlgrEnc<false> enc;
    rl_encode_block<false>(a, k, enc);
    const uint64_t words = k.L ? ((uint64_t)enc.nbits + 31) / 32 : 0;
    const uint64_t incl = wave_incl_scan(words), row_words = read_lane(incl, (uint32_t)(WAVE - 1));
    const uint64_t base = lookback_wave<OpSum>(a.status, 1, blockIdx.x, row_words, reinterpret_cast<Ctrl *>(a.err));
    const uint64_t first = base + incl - words;
    // the stream's capacity (header, table, words) bounds the total
    const uint64_t room = (a.out_cap - sizeof(gsc_rlgr_header)) / 4 - (NB + 1);
    GAS uint32_t *tab = rl_table(a.out);
    if (k.L) {
        if (first + words > room || first + words > 0xFFFFFFFFull) atomicCAS(a.err, 0u, (uint32_t)GSC_ERR_CAPACITY);
        else tab[k.b] = (uint32_t)first;
    }
    if (blockIdx.x == gridDim.x - 1 && tid == 0) {
        const uint64_t total = base + row_words;
        if (total <= room && total <= 0xFFFFFFFFull) {
            tab[NB] = (uint32_t)total;
            gsc_rlgr_header *h = reinterpret_cast<gsc_rlgr_header *>(a.out);
            h->magic = GSC_RLGR_MAGIC;
            h->version = GSC_VERSION;
            h->nv = a.nv;
            h->C = a.C;
            h->B = a.B;
            h->nblocks = NB;
            h->total_words = (uint32_t)total;
            h->reserved = 0;
            const uint64_t bytes = sizeof(gsc_rlgr_header) + 4ull * (NB + 1 + total);
            a.info[2] = (int32_t)(uint32_t)bytes;
            a.info[3] = (int32_t)(uint32_t)(bytes >> 32);
        }
    }
}

// Pass 2: every block's code written at its offset. The device status is known by then (only the
// counting pass can fail), so the first workgroup also ends the call.
__global__ __launch_bounds__(RLGR_THREADS) void k_rlgr_write(RlgrArgs a)
{
    const uint32_t NB = a.nb * a.C;
    const uint32_t err = __builtin_amdgcn_readfirstlane(__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.info[0] = (int32_t)err;
        a.info[1] = (int32_t)a.nv;
        if (err) a.info[2] = a.info[3] = 0;
    }
    if (err) return;
    const RlBlock k = rl_block(a.nv, a.C, a.B, a.nb);
    RlgrEnc<true> enc;
    if (k.L) enc.out = rl_words(a.out, NB) + rl_table(a.out)[k.b];
    rl_encode_block<true>(a, k, enc);
}

// The workspace's error word and look-back status words start at zero.
__global__ __launch_bounds__(256) void k_rlgr_zero(uint64_t *ws, uint32_t nwords)
{
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < nwords; i += gridDim.x * 256) ws[i] = 0;
}

// A matrix without values: the header and the one-entry table of an empty stream.
__global__ __launch_bounds__(64) void k_rlgr_empty(RlgrArgs a)
{
    if (threadIdx.x == 0) {
        gsc_rlgr_header *h = reinterpret_cast<gsc_rlgr_header *>(a.out);
        h->magic = GSC_RLGR_MAGIC;
        h->version = GSC_VERSION;
        h->nv = 0;
        h->C = a.C;
        h->B = a.B;
        h->nblocks = 0;
        h->total_words = 0;
        h->reserved = 0;
        *rl_table(a.out) = 0;
        a.info[0] = GSC_OK;
        a.info[1] = 0;
        a.info[2] = (int32_t)(sizeof(gsc_rlgr_header) + 4);
        a.info[3] = 0;
    }
}

// ------------------------------------------------------------------------------ decoder
// The words of a thread's block pass through an LDS ring of RLGR_RING words (slot i % RLGR_RING of
// thread t at word t of row i % RLGR_RING: no bank conflicts), refilled after every step of RLGR_STEP
// values from RLGR_FETCH words loaded before it, so that the value that needs a new word pays an LDS
// read whose result is used one word later. A wave in which a ring runs low (blocks of more than 16
// bits a value) takes steps of a half or a quarter of the values until it is full again; a word that
// is not in the ring yet is read from the stream and waited for, and a block that has also taken all the
// words fetched meanwhile (escapes) loads the next ones at the refill. 1M x 56 uniform values, blocks of
// 512, with rings that stayed empty once they had been outrun and with these: 14 bits 492 -> 357 us,
// 20 bits 829 -> 629, 31 bits (escapes) 763 -> 579. Positions are clamped to the block's words; a block
// that reads past them is rejected by the number of bits it took.
constexpr uint32_t RLGR_RING = 16, RLGR_FETCH = 8;

struct RlgrDec {
    uint32_t kp = RLGR_START, krp = RLGR_START;
    uint32_t zeros = 0;    // zeros still to produce
    uint32_t pend = 0;     // 1: a run's terminating value follows the zeros
    bool open = false;     // the last run token was a 0 bit (the run goes on)
    bool bad = false;
    // the next bit is bit `bit` (1..32, from the top) of the 64-bit window w0:w1; w2 follows
    uint32_t w0 = 0, w1, w2, bit = 32;
    uint32_t rp = 2;       // index of the word after w2 ... (words taken from the stream, less w2)
    uint32_t hi;           // words [.., hi) have been put in the ring
    uint32_t last;         // the block's last word (clamp)
    const GAS uint32_t *w;
    uint32_t *ring;        // this thread's column

    __device__ uint32_t at(uint32_t i) const { return w[min(i, last)]; }
    __device__ void init(const GAS uint32_t *w_, uint32_t nw, uint32_t *ring_)
    {
        w = w_;
        last = nw ? nw - 1u : 0u;
        ring = ring_;
        uint32_t x[RLGR_RING];
#pragma unroll
        for (uint32_t i = 0; i < RLGR_RING; ++i) x[i] = at(i);
#pragma unroll
        for (uint32_t i = 0; i < RLGR_RING; ++i) ring[i * RLGR_THREADS] = x[i];
        hi = RLGR_RING;
        w1 = x[0];
        w2 = x[1];
    }
    __device__ void fetch(uint32_t (&x)[RLGR_FETCH]) const
    {
#pragma unroll
        for (uint32_t i = 0; i < RLGR_FETCH; ++i) x[i] = at(hi + i);
    }
    // The values until the next refill (the same for the whole wave).
    __device__ uint32_t step() const
    {
        const int32_t ahead = (int32_t)(hi - rp);
        if (!__any(ahead <= (int32_t)RLGR_FETCH)) return RLGR_STEP;
        return __any(ahead <= (int32_t)RLGR_FETCH / 2) ? RLGR_STEP / 4 : RLGR_STEP / 2;
    }
    __device__ void refill(uint32_t (&x)[RLGR_FETCH])  // (x: the words from hi on)
    {
        const int32_t ahead = (int32_t)(hi - rp);
        if (ahead > (int32_t)(RLGR_RING - RLGR_FETCH)) return;  // (no room)
        if (ahead <= -(int32_t)RLGR_FETCH) {                    // (all of them taken already)
            hi = rp;
            fetch(x);
        }
#pragma unroll
        for (uint32_t i = 0; i < RLGR_FETCH; ++i) ring[((hi + i) % RLGR_RING) * RLGR_THREADS] = x[i];
        hi += RLGR_FETCH;
    }
    __device__ __attribute__((always_inline)) void take(uint32_t n)  // n <= 32 bits
    {
        bit += n;
        if (bit > 32) {
            bit -= 32;
            w0 = w1;
            w1 = w2;
            w2 = rp < hi ? ring[(rp % RLGR_RING) * RLGR_THREADS] : at(rp);
            ++rp;
        }
    }
    __device__ uint32_t peek() const { return __builtin_amdgcn_alignbit(w0, w1, 32u - bit); }  // the next 32 bits
    __device__ uint32_t get(uint32_t n)  // 1 <= n <= 32
    {
        const uint32_t v = peek() >> (32u - n);
        take(n);
        return v;
    }
    __device__ uint32_t taken() const { return (rp - 2u) * 32u + bit - 32u; }

    // The block's next value. One run token (a 0 bit: 2^k zeros; a 1: the remaining count in k
    // bits) at most is taken per value, since a 0 bit always has zeros to produce.
    __device__ __attribute__((always_inline)) int32_t value()
    {
        const uint32_t x = peek();
        const uint32_t k = kp >> RLGR_FRAC, kr = krp >> RLGR_FRAC;
        uint32_t n = 0;
        if ((zeros | pend) == 0 && k != 0) {
            const bool one = (int32_t)x < 0;
            zeros = one ? __builtin_amdgcn_ubfe(x, 31u - k, k) : 1u << k;
            n = one ? 1u + k : 1u;
            pend = one ? 1u : 0u;
            open = !one;
            kp = min(kp + (one ? 0u : (uint32_t)RLGR_RUN_UP), RLGR_PMAX);
        }
        int32_t v = 0;
        if (zeros == 0) {
            const uint32_t y = (x << n) << pend;
            uint32_t s = pend ? (x << n) >> 31 : 0u;
            uint32_t q = __clz(~y);  // leading ones (y ends in n + pend zeros)
            uint32_t u = (q << kr) | __builtin_amdgcn_ubfe(y << ((q + 1u) & 31u), (32u - kr) & 31u, kr);
            n += pend + q + 1u + kr;
            if (q >= RLGR_ESCAPE || n > 32u) {  // an escape, or a code longer than the window
                n -= pend + q + 1u + kr;
                if (n) take(n);
                if (pend) s = get(1);
                q = min((uint32_t)__clz(~peek()), RLGR_ESCAPE);
                if (q >= RLGR_ESCAPE) {
                    take(RLGR_ESCAPE);
                    u = get(32);
                    q = u >> kr;
                    if (pend && u >= 0x7FFFFFFFu + s) bad = true;  // (|v| = u + 1 past the range of an int32)
                } else {
                    take(q + 1u);
                    u = (q << kr) | (kr ? get(kr) : 0u);
                }
                n = 0;
            }
            // after a run: the sign and |v| - 1; else 2v or -2v - 1
            const uint32_t m = pend ? u + 1u : u >> 1, neg = pend ? s : u & 1u;
            v = (int32_t)((m ^ (0u - neg)) + (pend & neg));
            kp = rl_adapt(kp, pend ? -RLGR_RUN_DOWN : (u == 0 ? RLGR_GR_UP : -RLGR_GR_DOWN));
            krp = rl_adapt(krp, rl_gr_step(q));
            pend = 0;
        } else {
            --zeros;
        }
        take(n);
        return v;
    }
    // After the last value: an open run ends in a 1 and a count of zero, no zero is left over, and
    // only the last word's low bits are.
    __device__ bool ends(uint32_t nw)
    {
        if (zeros) return false;
        if (open) {
            const uint32_t k = kp >> RLGR_FRAC;
            if (get(k + 1u) != 1u << k) return false;
        }
        const uint32_t n = taken();  // (at most 65536 values of 68 bits; nw is what the table claims)
        return !bad && (n + 31u) / 32u == nw;
    }
};

struct RlgrDecArgs {
    const uint8_t *in;
    uint64_t in_bytes;
    uint32_t nv, C, B, nb;
    int32_t *q;      // [nv][C]
    int32_t *info;
    uint32_t *err;   // [0] device error, [1] workgroups done
};

// Decodes a wave's block rows, every thread one block, whole matrix rows stored at each step. The last
// of at most RLGR_COUNTED workgroups to end writes the info words; of more, a launch of its own does
// (the additions to one word come 9 ns apart, a launch costs 4.5 us): 1M x 56 in blocks of 16 (62500
// waves) counted 729 us, not counted 127; of 64 216 and 132, of 512 (1954) 235 and 225.
constexpr uint32_t RLGR_COUNTED = 512;
__global__ __launch_bounds__(RLGR_THREADS) void k_rlgr_decode(RlgrDecArgs a)
{
    __shared__ uint32_t s_ring[RLGR_RING * RLGR_THREADS];
    const uint32_t tid = threadIdx.x, NB = a.nb * a.C;
    const GAS uint32_t *tab = gp(reinterpret_cast<const uint32_t *>(a.in + sizeof(gsc_rlgr_header)));
    const GAS uint32_t *words = tab + NB + 1;
    const CAS gsc_rlgr_header *h = cp(reinterpret_cast<const gsc_rlgr_header *>(a.in));
    // header and table bounds (the host checked that the header and table fit in in_bytes)
    const uint32_t tw = h->total_words;
    const bool hdr = h->magic == GSC_RLGR_MAGIC && h->nv == a.nv && h->C == a.C && h->B == a.B && h->nblocks == NB &&
                     tab[NB] == tw && sizeof(gsc_rlgr_header) + 4ull * (NB + 1 + (uint64_t)tw) <= a.in_bytes;
    bool ok = hdr;
    if (hdr) {
        const RlBlock k = rl_block(a.nv, a.C, a.B, a.nb);
        RlgrDec dec;
        uint32_t o0 = 0, nw = 0;
        if (k.L) {
            o0 = tab[k.b];
            const uint32_t o1 = tab[k.b + 1];
            if (o1 < o0 || o1 > tw) dec.bad = true;
            else nw = o1 - o0;
        }
        // (a block without words reads the table's first word, which every stream has)
        dec.init(nw ? words + o0 : tab, nw, s_ring + tid);
        GAS char *dst = reinterpret_cast<GAS char *>(gp(a.q) + k.ubase);
        const uint32_t pitch = 4u * a.C;
        uint32_t off = k.off;
        for (uint32_t i = 0, n; i < k.lmax; i += n) {
            n = dec.step();
            uint32_t x[RLGR_FETCH];
            dec.fetch(x);
            if (k.L && i + n <= k.lmin) {
                for (uint32_t u0 = 0; u0 < n; u0 += RLGR_STEP / 4) {
#pragma unroll
                    for (int u = 0; u < RLGR_STEP / 4; ++u) {
                        *reinterpret_cast<GAS int32_t *>(dst + off) = dec.value();
                        off += pitch;
                    }
                }
            } else {  // (past the wave's shortest block: the last block row, which is shorter)
#pragma unroll 1
                for (uint32_t u = 0; u < n; ++u) {
                    if (i + u < k.L) {
                        *reinterpret_cast<GAS int32_t *>(dst + off) = dec.value();
                        off += pitch;
                    }
                }
            }
            dec.refill(x);
        }
        ok = k.L == 0 || dec.ends(nw);
    }
    if (!ok) atomicCAS(a.err, 0u, (uint32_t)GSC_ERR_CORRUPT_STREAM);
    if (gridDim.x > RLGR_COUNTED) return;
    // the wave's error report has completed before it is counted (device-scope atomics throughout)
    __builtin_amdgcn_s_waitcnt(0);
    if (tid == 0 && __hip_atomic_fetch_add(a.err + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == gridDim.x) {
        a.info[0] = (int32_t)__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a.info[1] = (int32_t)a.nv;
    }
}

__global__ __launch_bounds__(64) void k_rlgr_dec_info(RlgrDecArgs a)
{
    if (threadIdx.x == 0) {
        a.info[0] = (int32_t)__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a.info[1] = (int32_t)a.nv;
    }
}

// An empty stream: only its header to check.
__global__ __launch_bounds__(64) void k_rlgr_dec_empty(RlgrDecArgs a)
{
    if (threadIdx.x == 0) {
        const gsc_rlgr_header *h = reinterpret_cast<const gsc_rlgr_header *>(a.in);
        const bool ok = h->magic == GSC_RLGR_MAGIC && h->nv == 0 && h->C == a.C && h->nblocks == 0 && h->total_words == 0;
        a.info[0] = ok ? GSC_OK : GSC_ERR_CORRUPT_STREAM;
        a.info[1] = 0;
    }
}

// --------------------------------------------------------------------------- launches
hipError_t launch_rlgr_encode(const int32_t *q, uint32_t nv, uint32_t C, uint32_t B, uint8_t *out,
                              uint64_t out_cap, uint64_t *ws, int32_t *info, hipStream_t s)
{
    RlgrArgs a;
    a.q = q;
    a.nv = nv;
    a.C = C;
    a.B = B;
    a.nb = (nv + B - 1) / B;
    a.out = out;
    a.out_cap = out_cap;
    a.err = reinterpret_cast<uint32_t *>(ws);
    a.status = ws + 1;
    a.info = info;
    if (a.nb == 0) {
        hipLaunchKernelGGL(k_rlgr_empty, dim3(1), dim3(64), 0, s, a);
        return hipGetLastError();
    }
    const uint32_t rpw = rl_rows(C), nwg = (a.nb + rpw - 1) / rpw, zw = nwg + 1;
    hipLaunchKernelGGL(k_rlgr_zero, dim3(min((zw + 255) / 256, 1024u)), dim3(256), 0, s, ws, zw);
    hipLaunchKernelGGL(k_rlgr_count, dim3(nwg), dim3(RLGR_THREADS), 0, s, a);
    hipLaunchKernelGGL(k_rlgr_write, dim3(nwg), dim3(RLGR_THREADS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_rlgr_decode(const uint8_t *in, uint64_t in_bytes, uint32_t nv, uint32_t C, uint32_t B,
                              int32_t *q, uint64_t *ws, int32_t *info, hipStream_t s)
{
    RlgrDecArgs a;
    a.in = in;
    a.in_bytes = in_bytes;
    a.nv = nv;
    a.C = C;
    a.B = B;
    a.nb = (nv + B - 1) / B;
    a.q = q;
    a.info = info;
    a.err = reinterpret_cast<uint32_t *>(ws);
    if (a.nb == 0) {
        hipLaunchKernelGGL(k_rlgr_dec_empty, dim3(1), dim3(64), 0, s, a);
        return hipGetLastError();
    }
    const uint32_t rpw = rl_rows(C), nwg = (a.nb + rpw - 1) / rpw;
    hipLaunchKernelGGL(k_rlgr_zero, dim3(1), dim3(256), 0, s, ws, 1u);
    hipLaunchKernelGGL(k_rlgr_decode, dim3(nwg), dim3(RLGR_THREADS), 0, s, a);
    if (nwg > RLGR_COUNTED) hipLaunchKernelGGL(k_rlgr_dec_info, dim3(1), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace gsc
