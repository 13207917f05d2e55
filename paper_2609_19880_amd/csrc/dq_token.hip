// Decode attention over per-token streams: one rANS stream of n = 128 H_kv
// values per token spanning every KV head (the paper's default grouping,
// Sec. 4.1 and Sec. 5.1), decoded once and consumed one KV head at a time as
// Sec. 4.5 ("Decoding") describes.
//
// Work split.  One workgroup per (context chunk, sequence); each wavefront
// takes 64-token tiles, one token per lane, and runs the token's key and
// value streams as two interleaved rANS chains (Alg. 2).  After every 128
// steps (one KV head) the head's G query heads get their q . k products
// (Eq. fold-key, on the 16x16x64 matrix cores, half of the head's channels at a
// time), the online softmax update and P . v (Eq. fold-value, the same product);
// the chains then continue into the next head with their state.  All query
// heads' accumulators live in the wavefront: per KV head and group of 4
// query-head slots (one group for up to 4 query heads per KV head, two for up
// to 8), lane l holds slot l / 16 of the group for 8 of the 128 channels, and
// the softmax state of head i in lane i of the row of 16 lanes.
//
// Record bytes.  Records (C bytes in S-byte slots, S a multiple of 16) are
// stored per 64-token tile with 8-byte chunks outermost: chunk c of the tile's
// token l at c * 512 + l * 8 from the tile, so the 64 lanes of a wavefront
// loading the same chunk read 512 contiguous bytes.  They are read in 8-byte
// chunks into a per-lane ring of 8 dwords in LDS, laid out
// [dword row][lane] so that every lane stays in its own bank; a ninth row
// repeats row 0 so that two consecutive dwords are always rows r, r + 1.  A
// decode step reads the two dwords holding its byte position and takes the
// next 16 bits with a funnel shift and a byte permute; with two 2^8-entry tables
// a step takes at most one byte and one read serves four steps.  Every 8 steps (16
// with such tables) a lane whose ring holds fewer than 20 bytes from its position writes its next
// chunk (held in registers since the previous refill) and loads the one
// after, and does so once more in the rare case that it is still short: those
// steps read at most 16 bytes, and their two-dword windows reach at most 19
// bytes past the position.  A chunk is written only while the ring is short,
// so the chunk four back that it replaces lies wholly behind the position
// and is never read again.  Ring rows are masked, so a corrupt stream reads
// garbage inside its ring, never outside; it is flagged at the end (state !=
// L or pointer past the record).
#include <math.h>

#include <algorithm>

#include "dq_attn.h"

namespace dq {
namespace {

constexpr int kD = 128;
constexpr int kTile = 64;
constexpr int kVSlice = 64;
constexpr int kMaxLds = 160 * 1024;
// wavefronts per workgroup at most: 12 with up to 4 query heads per KV head
// (168 VGPRs), 8 with up to 8 (the accumulators of 64 query heads take 128)
__host__ __device__ constexpr int tok_waves(int HG) { return HG == 1 ? 12 : 8; }
constexpr int kTokSplitWaves = 8;          // split tiles: 4 pairs of wavefronts (at most 256 VGPRs)
constexpr int kTokMaxHeads = 8;           // KV heads per stream (n <= 1024)
constexpr int kTokMaxChunk = 2048;        // bounds the per-window q . mu table
constexpr int kRingRow = 4 * kTile;       // bytes per ring row: one dword per lane
constexpr int kRingRows = 8;              // dwords of record bytes per lane
constexpr int kRingBytes = (kRingRows + 1) * kRingRow;   // + the copy of row 0
constexpr int kGroups = kD / 4;           // 4-step groups per head

struct TokLayout {
    int nw;
    int lut_k, lut_v;   // 8-byte tables (the same offset when K and V share one)
    int qtile;          // query digits: [H_kv][HG][2 slices][16 rows][kQRow]
    int qscale, qsum;   // float [H_q]
    int qmu;            // float [windows][H_q]
    int waves;          // first wavefront region
    int wave_stride;
    int ring_k, ring_v; // per wavefront
    int vtile;          // [64 tokens][kRowT]: levels of a 64-channel slice, keys then values, and (kRowHdr) the
                        // first words of the key and value records (fp16 scale, offset)
    int plimb;          // [HG][64 tokens][16]: weight digits, byte 4 slot + digit (digit 3 zero)
    int total;
};

struct TokArgs {
    TabArgs tk, tv;
    const uint16_t* q;
    int Hq, Hkv, G, t_cap, chunk, nchunks;
    const uint8_t* krec;
    const int8_t* kmq;
    const uint16_t* kms;
    const uint8_t* vrec;
    int k_stride, v_stride;       // bytes per token record (multiples of 16)
    Pages pg;                     // block table of a paged cache (bt null: contiguous)
    const int32_t* seq_lens;
    float q_scale;                // softmax_scale * log2(e) / d (/ 1 for prerotated keys)
    int rot_q, rot_out;           // keys / values rotated online (tables not prerotated)
    int32_t* ws_hdr;
    float* ws_m;
    float* ws_l;
    float* ws_acc;
    uint32_t* status;
    TokLayout L;
};

// Two steps of Alg. 2 on one ring read, state X = 8 x as in the per-head
// kernel; pb is the lane's bit position in its record (8 x byte position).
//   dwords j = pb >> 5 and j + 1 come from ring rows j mod 8 and the next
//   w = bytes pos .. pos + 3, little-endian = (hi:lo) >> (pb mod 32)
//   r = b_pos << 24 | b_pos+1 << 16 | b_pos+2 << 8 | b_pos+3 (byte reverse)
// r >> (29 - sh) puts the sh bits to shift in at bits 3 and up; what lands in
// the low three bits of X is never read.  Each step reads at most 2 bytes, so
// the second step's bytes are r << sh of the first.
//
// The two steps are split so that the key and value chains of a lane
// overlap: tissue_a requests the ring dwords and the first table word,
// tfinish_a completes the first step, tissue_b requests the second table
// word, tfinish_b completes the second step.  The compiler does not see the
// requested loads, so nothing may read their results until a twait<N> has run
// on them: it waits until at most N LDS or scalar-memory operations are
// outstanding (LDS returns in order; N counts the LDS reads issued after the
// awaited one, and operations the compiler adds in between only make the wait
// stricter).  The finish steps return the table words (levels in their top
// bytes).
//
// Arithmetic in inline assembly works in place (its result takes the register of
// an operand).  The compiler keeps ordinary instructions clear of matrix products
// in flight (8 wait states before a register of their result is written), but not
// instructions in assembly: a fresh result register could be one that a product
// issued just before still writes.
struct TChain {
    uint32_t X, pb, w;
    uint64_t rr, e;      // pending: ring dwords (lo, hi), table word
};

template <uint32_t LUT_OFF>
__device__ __forceinline__ void tissue_a(TChain& c, uint32_t ring_lane, uint32_t mask8) {
    uint32_t addr = __builtin_amdgcn_ubfe(c.pb, 5, 3);
    asm("v_lshl_add_u32 %0, %0, 8, %1" : "+v"(addr) : "v"(ring_lane));
    asm volatile("ds_read2st64_b32 %0, %2 offset1:1\n\t"
                 "ds_read_b64 %1, %3 offset:%4"
                 : "=&v"(c.rr), "=&v"(c.e)
                 : "v"(addr), "v"(c.X & mask8), "i"(LUT_OFF));
}

template <uint32_t LUT_OFF>
__device__ __forceinline__ void tissue_b(TChain& c, uint32_t mask8) {
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=&v"(c.e) : "v"(c.X & mask8), "i"(LUT_OFF));
}

template <int N>
__device__ __forceinline__ void twait_a(TChain& c) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(c.rr), "+v"(c.e) : "i"(N));
}

template <int N>
__device__ __forceinline__ void twait_b(TChain& c) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(c.e) : "i"(N));
}

// sh of the first step, kept for the second
__device__ __forceinline__ uint32_t tfinish_a(TChain& c, int p3, uint32_t& sh) {
    const uint32_t lo = (uint32_t)c.rr, hi = (uint32_t)(c.rr >> 32);
    const uint32_t w = __builtin_amdgcn_perm(0u, __builtin_amdgcn_alignbit(hi, lo, c.pb), 0x00010203u);
    const uint32_t ea = (uint32_t)c.e;
    uint32_t y = __umul24(ea, c.X >> p3) + (uint32_t)(c.e >> 32);
    sh = (uint32_t)__builtin_clz(y) & 24u;
    const uint32_t q = w >> (sh ^ 29u);
    asm("v_lshl_or_b32 %0, %0, %1, %2" : "+v"(y) : "v"(sh), "v"(q));
    c.X = y;
    c.w = w << sh;
    return ea;
}

__device__ __forceinline__ uint32_t tfinish_b(TChain& c, int p3, uint32_t sha) {
    const uint32_t eb = (uint32_t)c.e;
    uint32_t y = __umul24(eb, c.X >> p3) + (uint32_t)(c.e >> 32);
    const uint32_t sh = (uint32_t)__builtin_clz(y) & 24u;
    const uint32_t q = c.w >> (sh ^ 29u);
    asm("v_lshl_or_b32 %0, %0, %1, %2" : "+v"(y) : "v"(sh), "v"(q));
    c.X = y;
    asm("v_add3_u32 %0, %0, %1, %2" : "+v"(c.pb) : "v"(sha), "v"(sh));
    return eb;
}

// Four steps on one ring read, for p = 8: there a step reads at most one byte (x'
// >= f 2^13, and one byte more brings it to L), so the four bytes at the lane's
// position serve four steps, and a block between two refills is 16 steps of at
// most 16 bytes, which the same 20 bytes cover.  U: step in the group; shp: the
// shift of step U - 1.
template <int U>
__device__ __forceinline__ uint32_t tfinish4(TChain& c, int p3, uint32_t& shp) {
    if (U == 0) {
        const uint32_t lo = (uint32_t)c.rr, hi = (uint32_t)(c.rr >> 32);
        c.w = __builtin_amdgcn_perm(0u, __builtin_amdgcn_alignbit(hi, lo, c.pb), 0x00010203u);
    }
    const uint32_t e = (uint32_t)c.e;
    uint32_t y = __umul24(e, c.X >> p3) + (uint32_t)(c.e >> 32);
    const uint32_t sh = (uint32_t)__builtin_clz(y) & 24u;
    const uint32_t q = c.w >> (sh ^ 29u);
    asm("v_lshl_or_b32 %0, %0, %1, %2" : "+v"(y) : "v"(sh), "v"(q));
    c.X = y;
    if (U < 3) c.w <<= sh;
    if (U & 1) asm("v_add3_u32 %0, %0, %1, %2" : "+v"(c.pb) : "v"(shp), "v"(sh));
    shp = sh;
    return e;
}

// rec: the lane's first chunk (tile + 8 lane); chunks are 512 bytes apart.
__device__ __forceinline__ uint2 load_chunk(const uint8_t* rec, uint32_t c, uint32_t last) {
    return *reinterpret_cast<const uint2*>(rec + 512u * min(c, last));
}

// Chunk c of the record into ring rows 2 (c mod 4), + 1 (and row 8 for c
// mod 4 = 0).
__device__ __forceinline__ void put_chunk(uint32_t ring_lane, uint32_t c, const uint2& v) {
    const uint32_t a = ring_lane + (c & 3u) * 2u * kRingRow;
    *LDS_PTR(uint32_t, a) = v.x;
    *LDS_PTR(uint32_t, a + kRingRow) = v.y;
    if ((c & 3u) == 0) *LDS_PTR(uint32_t, ring_lane + kRingRows * kRingRow) = v.x;
}

// One chunk per ring toward 8 nc >= pos + 20 (the bytes the next 8 steps can
// read).  thr is 8 (8 nc - 20) - 1 in bits, so the test is one compare.  Both
// rings are written before either chunk load is issued: the loads complete in
// order, so the writes wait only for chunks loaded at earlier refills, never
// for the other ring's load of this group.
__device__ __forceinline__ void refill2(uint32_t pbk, uint32_t& nck, uint32_t& thrk, uint2& nk, uint32_t ring_k,
                                        const uint8_t* kr, uint32_t last_k, uint32_t pbv, uint32_t& ncv,
                                        uint32_t& thrv, uint2& nv, uint32_t ring_v, const uint8_t* vr,
                                        uint32_t last_v) {
    const bool rk = pbk > thrk, rv = pbv > thrv;
    if (rk) put_chunk(ring_k, nck, nk);
    if (rv) put_chunk(ring_v, ncv, nv);
    if (rk) {
        ++nck;
        thrk += 64u;
        nk = load_chunk(kr, nck, last_k);
    }
    if (rv) {
        ++ncv;
        thrv += 64u;
        nv = load_chunk(vr, ncv, last_v);
    }
}

// One chunk for one ring (keys and values decoded by separate wavefronts).
__device__ __forceinline__ void refill1(uint32_t pb, uint32_t& nc, uint32_t& thr, uint2& nxt, uint32_t ring,
                                        const uint8_t* rec, uint32_t last) {
    if (pb > thr) {
        put_chunk(ring, nc, nxt);
        ++nc;
        thr += 64u;
        nxt = load_chunk(rec, nc, last);
    }
}

// The 128 steps of one KV head on a single chain (the wavefront decodes only
// the keys or only the values of its tile): per step pair the ring dwords
// and the first table word, then the second table word, each awaited before
// it is used; the ring is refilled after every block of 8 steps (W4: 16), whose last
// reads come after the refill's writes.  level(grp, word) takes the packed
// levels of four steps; no read of the chain is in flight when it is called for
// the last group of a block.  W4: four steps per ring read and blocks of 16
// steps (p = 8).
template <uint32_t LUT, bool W4, typename Level>
__device__ __forceinline__ void chain_head(TChain& c, uint32_t ring, uint32_t mask8, int p3, uint32_t& nc,
                                           uint32_t& thr, uint2& nxt, const uint8_t* rec, uint32_t last,
                                           Level&& level) {
    constexpr int kBlock = W4 ? 3 : 1;          // groups between two refills, less one
#pragma unroll
    for (int grp = 0; grp < kGroups; ++grp) {
        const bool end = (grp & kBlock) == kBlock;
        if ((grp & kBlock) == 0) tissue_a<LUT>(c, ring, mask8);
        uint32_t w[4], sh;
        if constexpr (W4) {
            twait_a<0>(c);
            w[0] = tfinish4<0>(c, p3, sh);
            tissue_b<LUT>(c, mask8);
            twait_b<0>(c);
            w[1] = tfinish4<1>(c, p3, sh);
            tissue_b<LUT>(c, mask8);
            twait_b<0>(c);
            w[2] = tfinish4<2>(c, p3, sh);
            tissue_b<LUT>(c, mask8);
            twait_b<0>(c);
            w[3] = tfinish4<3>(c, p3, sh);
            if (!end) tissue_a<LUT>(c, ring, mask8);
        } else {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const bool more = !(end && u == 1);
                twait_a<0>(c);
                w[2 * u] = tfinish_a(c, p3, sh);
                tissue_b<LUT>(c, mask8);
                twait_b<0>(c);
                w[2 * u + 1] = tfinish_b(c, p3, sh);
                if (more) tissue_a<LUT>(c, ring, mask8);
            }
        }
        uint32_t lev = pack4(w[0], w[1], w[2], w[3]);
        asm volatile("" : "+v"(lev));
        level(grp, lev);
        if (end) {
            refill1(c.pb, nc, thr, nxt, ring, rec, last);
            // a second chunk only where a lane is still short (rare)
            if (__any(c.pb > thr)) refill1(c.pb, nc, thr, nxt, ring, rec, last);
            // the next block's ring reads come after these writes
            asm volatile("" ::: "memory");
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Key levels of group grp: every fourth group completes 16 bytes of the lane's
// row, and after 64 channels the slice meets the query digits (kq: the slice's
// operand of head h's query tiles).
template <int HG>
__device__ __forceinline__ void key_levels(int grp, uint32_t lev, uint32_t (&k4)[4], uint32_t row, uint32_t col,
                                           uint32_t kq, v4i (&d)[HG][4]) {
    k4[grp & 3] = lev;
    if ((grp & 3) == 3) {
        *LDS_PTR(v4i, row + 16 * ((grp >> 2) & 3)) = v4i{(int)k4[0], (int)k4[1], (int)k4[2], (int)k4[3]};
        if ((grp & 15) == 15) {
            wave_sync();       // rows are read by other lanes
            qk_slice<HG>(col, kq + (grp >> 4) * kQTile, d);
            wave_sync();       // and rewritten by the next slice or the values
        }
    }
}

// The softmax state of the head at hand sits in lane 0 of each row of 16 lanes;
// the rows rotate by one lane per head.
__device__ __forceinline__ float row_next(float v) { return __uint_as_float(dpp_u32<0x12F, 0xF>(__float_as_uint(v))); }
__device__ __forceinline__ float row_first(float v) { return __uint_as_float(dpp_u32<0x150, 0xF>(__float_as_uint(v))); }

// One tile's contribution to the state of the head at hand: m (the new maximum),
// corr, and the row sums of psum and osum; then on to the next head.
__device__ __forceinline__ void push_state(const SlotWeights& sw, float m, bool first, float& m_vec, float& l_vec,
                                           float& o_vec) {
    const float l = fmaf(l_vec, sw.corr, row_sum16(sw.psum)), o = fmaf(o_vec, sw.corr, row_sum16(sw.osum));
    m_vec = row_next(first ? m : m_vec);
    l_vec = row_next(first ? l : l_vec);
    o_vec = row_next(first ? o : o_vec);
}

// Accumulators of channel block cb of slice s and slot group hg: one vector
// acc[s][hg][cb] over the KV heads, for query-head slot 4 hg + l / 16 and
// channel 64 s + 16 cb + l mod 16 in lane l.  The head loop is not unrolled,
// so the vectors are rotated by one element per head and the current head is
// always element 0.
typedef float v8f __attribute__((ext_vector_type(kTokMaxHeads)));

__device__ __forceinline__ v8f rot1(const v8f& v) { return v8f{v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[0]}; }

// PAGED: records and key means through the block table; a separate
// instantiation, so that the contiguous kernel carries none of its state.
// HG: groups of 4 query-head slots per KV head (1: G <= 4, 2: G <= 8).
// SPLIT: one tile per pair of wavefronts, keys and values decoded by
// different wavefronts (chunks of at most nw / 2 tiles: small batches).
// W4: both tables have p = 8 (see tfinish4).
// What bounds it: vector issue (93 % at p = 8; LDS is active 64 % of the time).
// 16 x 32768 tokens, 8 KV heads, G = 4, p = 8: 469 us with the 4x4x4 products, 434
// with the 16x16x64 ones, 386 with W4; 1 x 4096 tokens (SPLIT): 106.5, 96 and 87.
template <uint32_t LUTV, bool PAGED, int HG, bool SPLIT, bool W4>
__global__ __launch_bounds__((SPLIT ? kTokSplitWaves : tok_waves(HG)) * kWave) void attn_token_kernel(TokArgs a) {
    constexpr int GS = 4 * HG;                 // query-head slots per KV head
    extern __shared__ __align__(16) uint8_t smem[];
    const TokLayout& L = a.L;
    const int G = a.G, Hkv = a.Hkv, Hq = a.Hq;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int nthr = L.nw * kWave;
    const int c = blockIdx.x, b = blockIdx.z;
    if ((c | b) == 0 && tid == 0) {
        a.ws_hdr[0] = a.chunk;
        a.ws_hdr[1] = a.nchunks;
        a.ws_hdr[2] = 0;          // set by the residual kernel when it runs
        a.ws_hdr[3] = a.rot_out;  // the merge rotates the output back
    }
    const int T = min(a.seq_lens[b], a.t_cap);
    const int start = c * a.chunk;
    if (start >= T) return;   // the merge ignores chunks past the length
    bool bad_page = false;    // a block-table entry outside the pool (read as page 0)

    // ---- prologue: tables, rotated queries, their digits, q . mu per window
    {
        const int Pk = 1 << a.tk.p, Pv = 1 << a.tv.p;
        uint2* lk = reinterpret_cast<uint2*>(smem + L.lut_k);
        for (int i = tid; i < Pk; i += nthr) lk[i] = a.tk.t.lut64[i];
        if (LUTV != 0) {
            uint2* lv = reinterpret_cast<uint2*>(smem + LUTV);
            for (int i = tid; i < Pv; i += nthr) lv[i] = a.tv.t.lut64[i];
        }
    }
    float* qt = reinterpret_cast<float*>(smem + L.waves);          // [H_q][d] scratch
    float* qscale = reinterpret_cast<float*>(smem + L.qscale);
    float* qsum = reinterpret_cast<float*>(smem + L.qsum);
    float* qmu = reinterpret_cast<float*>(smem + L.qmu);
    uint8_t* qtile = smem + L.qtile;
    rotate_query_heads(a.q + (int64_t)b * Hq * kD, Hq, Hq, wave, L.nw, lane, qt, qscale, qsum, a.rot_q, a.q_scale);
    __syncthreads();
    // a wavefront per query-head slot (slots past G get zero digits)
    for (int i = wave; i < Hkv * GS; i += L.nw) {
        const int h = i / GS, r = i % GS, g = h * G + r;
        const bool live = r < G;
        query_digits(qtile + h * HG * 2 * kQTile, r, lane, live ? qt[g * kD + lane] : 0.f,
                     live ? qt[g * kD + lane + 64] : 0.f, live ? qscale[g] : 0.f);
    }
    const int nwin_total = a.t_cap / DQ_MEAN_WINDOW;
    const int w0 = start / DQ_MEAN_WINDOW;
    const int nwin = (a.chunk + DQ_MEAN_WINDOW - 1) / DQ_MEAN_WINDOW + 1;
    // half a wavefront per (window, KV head), two per pass: lane l takes
    // channels 4 (l % 32) .. 4 (l % 32) + 3 and the KV head's G query heads
    {
        const int r = lane >> 5, c4 = 4 * (lane & 31);
        for (int it = 2 * wave + r; it - r < nwin * Hkv; it += 2 * L.nw) {
            const int wi = it / Hkv, hk = it % Hkv;
            float f[4] = {0.f, 0.f, 0.f, 0.f};
            // windows from the sequence's length on are never used: their
            // block-table entries may be unmapped
            if (it < nwin * Hkv && w0 + wi < nwin_total && (w0 + wi) * DQ_MEAN_WINDOW < T) {
                const int64_t widx = PAGED ? window_index(a.pg, Hkv, a.t_cap, b, hk, w0 + wi, bad_page)
                                           : ((int64_t)b * Hkv + hk) * nwin_total + w0 + wi;
                const float sc = half_bits_to_f32(a.kms[widx]);
                const uint32_t mv = *reinterpret_cast<const uint32_t*>(a.kmq + widx * kD + c4);
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k] = sc * (float)(int8_t)((mv >> (8 * k)) & 0xFF);
            }
            for (int q = 0; q < G; ++q) {
                const int g = hk * G + q;
                float s = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) s = s + qt[g * kD + c4 + k] * f[k];
                s = half_sum_f32(s);
                if ((lane & 31) == 31 && it < nwin * Hkv) qmu[wi * Hq + g] = s;
            }
        }
    }
    __syncthreads();

    // ---- per-wavefront state
    const uint32_t ring_k = (uint32_t)(L.waves + wave * L.wave_stride + L.ring_k) + 4u * lane;
    const uint32_t ring_v = (uint32_t)(L.waves + wave * L.wave_stride + L.ring_v) + 4u * lane;
    // P . v: lane l serves slot l / 16 of each group and channel l % 16 of each
    // 16-channel block; its tr8 reads start at token row 8 (l / 16) +
    // (l % 16) / 2 of a 32-token block, byte 8 (l % 2) of the row's block
    const int pslot = lane >> 4, l16 = lane & 15;
    const uint32_t wbase = (uint32_t)(L.waves + wave * L.wave_stride);
    const uint32_t trow = (uint32_t)(8 * (lane >> 4) + ((lane & 15) >> 1));
    const uint32_t a_off = trow * 16 + 8 * (lane & 1);
    const uint32_t b_lane = wbase + L.vtile + trow * kRowT + 8 * (lane & 1);
    const uint32_t row_lane = wbase + L.vtile + lane * kRowT, col_lane = wbase + L.vtile + level_operand(lane);
    const uint32_t kq_lane = (uint32_t)L.qtile + query_operand(lane);
    const uint32_t w_off = 16 * l16 + 4 * pslot;
    const int pk3 = a.tk.p + 3, pv3 = a.tv.p + 3;
    const uint32_t mask8k = ((1u << a.tk.p) - 1u) << 3, mask8v = ((1u << a.tv.p) - 1u) << 3;
    const uint32_t last_k = (uint32_t)(a.k_stride / 8 - 1), last_v = (uint32_t)(a.v_stride / 8 - 1);
    const uint32_t endk = 8u * (uint32_t)a.tk.C, endv = 8u * (uint32_t)a.tv.C;

    // running softmax state of slot l / 16 of KV head l % 16 (rotating)
    float m_vec[HG], l_vec[HG], o_vec[HG];
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) {
        m_vec[hg] = -INFINITY;
        l_vec[hg] = o_vec[hg] = 0.f;
    }
    v8f acc[2][HG][4];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int hg = 0; hg < HG; ++hg)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) acc[s][hg][cb] = v8f{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    bool corrupt = false;
    const int ntiles = (min(a.chunk, T - start) + kTile - 1) / kTile;

    // the weights of head h's groups from its digit sums (headers in the rows of
    // this wavefront), their digits to wt
    auto score_head = [&](const v4i (&d)[HG][4], int h, int t_base, uint32_t wt, SlotWeights (&sw)[HG],
                          float (&m)[HG]) {
        uint2 hd[4];
#pragma unroll
        for (int tg = 0; tg < 4; ++tg) {
            const v2u v = *LDS_PTR(v2u, wbase + L.vtile + kRowHdr + l16 * kRowT + tg * kColGroup);
            hd[tg] = uint2{v.x, v.y};
        }
        const int left = T - t_base - l16;
        const bool whole = t_base + kTile <= T;
        const float* qm = qmu + (t_base / DQ_MEAN_WINDOW - w0) * Hq;
#pragma unroll
        for (int hg = 0; hg < HG; ++hg) {
            const int r = 4 * hg + pslot, g = r < G ? h * G + r : 0;    // slots past G take no query head
            m[hg] = row_first(m_vec[hg]);
            sw[hg] = slot_softmax(d[hg], hd, qscale[g], qsum[g], qm[g], left, whole, m[hg]);
            store_weights(wt + w_off + hg * (kTile * 16), sw[hg].w);
        }
    };
    // ---- P . v over two slices of 64 channels with the weights at wt
    auto value_head = [&](const uint32_t (&vlev)[kGroups], uint32_t wt, auto&& add) {
        v4i pa[HG];
#pragma unroll
        for (int hg = 0; hg < HG; ++hg) pa[hg] = load_weights(wt + a_off + hg * (kTile * 16));
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
            if (sl) wave_sync();   // the first slice's value rows are no longer read
            store_levels(row_lane, vlev + 16 * sl);
            wave_sync();
            // all operands first, then the products
            v4i vb[4];
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) vb[cb] = load_values(b_lane + 16 * cb);
#pragma unroll
            for (int hg = 0; hg < HG; ++hg) {
                v4i dv[4];
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) dv[cb] = mfma64(pa[hg], vb[cb], v4i{0, 0, 0, 0});
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) add(sl, hg, cb, digit_sum(dv[cb]));
            }
        }
    };

    if constexpr (SPLIT) {
        // One tile per pair of wavefronts.  Per KV head the even wavefront
        // decodes the keys alone and forms the scores and the softmax weights
        // (their digits in one of two weight tiles of its region, the slots'
        // corrections and weight scales beside them), while the odd one
        // decodes the values alone; after the head's barrier the odd one forms
        // P . v with its partner's weights, while the even one goes on to the
        // next head (whose weights go to the other tile).  At the end the even
        // wavefront hands its softmax statistics to the odd one, which alone
        // then holds the pair's partial.
        static_assert(HG == 1, "split tiles: up to 4 query heads");
        const int tile = wave >> 1, role = wave & 1;
        const bool has = tile < ntiles;
        const uint32_t kreg = (uint32_t)(L.waves + (wave & ~1) * L.wave_stride);
        // the key wavefront's value ring is free: weight tile 1, then [2][GS]
        // corrections, [2][GS] weight units, and the statistics
        float* kx = reinterpret_cast<float*>(smem + kreg + L.ring_v + kTile * 16);
        const int t_base = start + tile * kTile;
        const int t = t_base + lane;
        const bool valid = t < T;
        // a tile never straddles a page
        const int64_t row0 = !has ? 0 : PAGED ? token_row(a.pg, a.t_cap, b, t_base, bad_page)
                                              : (int64_t)b * a.t_cap + t_base;
        const uint8_t* rec = role ? a.vrec + row0 * a.v_stride + 8 * lane : a.krec + row0 * a.k_stride + 8 * lane;
        const uint32_t last = role ? last_v : last_k;
        const uint32_t ring = role ? ring_v : ring_k;
        const uint32_t mask8 = role ? mask8v : mask8k;
        const int p3 = role ? pv3 : pk3;
        TChain ch;
        uint32_t nc = 4, thr = 8u * (8u * 4u - 20u) - 1u;
        uint2 nxt{0u, 0u};
        if (has) {
            const uint2 c0 = load_chunk(rec, 0, last), c1 = load_chunk(rec, 1, last), c2 = load_chunk(rec, 2, last),
                        c3 = load_chunk(rec, 3, last);
            nxt = load_chunk(rec, 4, last);
            // the key wavefront also needs the value record's scale and offset
            const uint32_t vh = role ? c0.x : load_chunk(a.vrec + row0 * a.v_stride + 8 * lane, 0, last_v).x;
            put_chunk(ring, 0, c0);
            put_chunk(ring, 1, c1);
            put_chunk(ring, 2, c2);
            put_chunk(ring, 3, c3);
            ch.X = c0.y << 3;
            if (W4) corrupt |= valid && (ch.X >> 3) < kRansL;   // (one byte a step needs a state from L on)
            ch.pb = 64;                             // payload starts at byte 8
            if (!role) *LDS_PTR(v2u, row_lane + kRowHdr) = v2u{valid ? c0.x : 0u, valid ? vh : 0u};
            asm volatile("" ::: "memory");
        }
        for (int h = 0; h < Hkv; ++h) {
            uint32_t vlev[kGroups];
            const int buf = h & 1;
            const uint32_t wt = kreg + (uint32_t)(buf ? L.ring_v : L.plimb);
            if (has && role == 0) {
                v4i d[HG][4];
#pragma unroll
                for (int tg = 0; tg < 4; ++tg) d[0][tg] = v4i{0, 0, 0, 0};
                uint32_t k4[4];
                const uint32_t kq = kq_lane + (uint32_t)(h * HG * 2 * kQTile);
                chain_head<0, W4>(ch, ring, mask8, p3, nc, thr, nxt, rec, last, [&](int grp, uint32_t lev) {
                    key_levels<HG>(grp, lev, k4, row_lane, col_lane, kq, d);
                });
                SlotWeights sw[HG];
                float m[HG];
                score_head(d, h, t_base, wt, sw, m);
                if (l16 == 0) {
                    kx[buf * GS + pslot] = sw[0].corr;
                    kx[2 * GS + buf * GS + pslot] = sw[0].wscale;
                }
                push_state(sw[0], m[0], l16 == 0, m_vec[0], l_vec[0], o_vec[0]);
            } else if (has) {
                chain_head<LUTV, W4>(ch, ring, mask8, p3, nc, thr, nxt, rec, last,
                                 [&](int grp, uint32_t lev) { vlev[grp] = lev; });
            }
            __syncthreads();   // the weights of the head are in LDS
            if (has && role == 1) {
                // ---- P . v with the partner's weights
                const float corr_l = kx[buf * GS + pslot], scale_l = kx[2 * GS + buf * GS + pslot];
                value_head(vlev, wt, [&](int sl, int hg, int cb, float f) {
                    v8f tv = acc[sl][hg][cb];
                    tv[0] = fmaf(f, scale_l, tv[0] * corr_l);
                    acc[sl][hg][cb] = rot1(tv);
                });
                wave_sync();   // the next head rewrites the value rows
            }
        }
        for (int h = Hkv; h < kTokMaxHeads; ++h)
#pragma unroll
            for (int sl = 0; sl < 2; ++sl)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) acc[sl][0][cb] = rot1(acc[sl][0][cb]);
        // every stream ends at x = L having read no byte past its record
        if (has) corrupt |= valid && ((ch.X >> 3) != kRansL || ch.pb > (role ? endv : endk));
        // the softmax statistics go to the value wavefront
        float* kst = kx + 4 * GS;
        if (has && role == 0) {
            for (int h = Hkv; h < 16; ++h) {
                m_vec[0] = row_next(m_vec[0]);
                l_vec[0] = row_next(l_vec[0]);
                o_vec[0] = row_next(o_vec[0]);
            }
            kst[lane] = m_vec[0];
            kst[kWave + lane] = l_vec[0];
            kst[2 * kWave + lane] = o_vec[0];
        }
        __syncthreads();
        if (has && role == 1) {
            m_vec[0] = kst[lane];
            l_vec[0] = kst[kWave + lane];
            o_vec[0] = kst[2 * kWave + lane];
        } else {
            m_vec[0] = -INFINITY;
        }
    }

    for (int tile = SPLIT ? ntiles : wave; tile < ntiles; tile += L.nw) {
        const int t_base = start + tile * kTile;
        const int t = t_base + lane;               // < t_cap: tiles lie inside the capacity
        const bool valid = t < T;
        // a tile never straddles a page
        const int64_t row0 = PAGED ? token_row(a.pg, a.t_cap, b, t_base, bad_page) : (int64_t)b * a.t_cap + t_base;
        const uint8_t* kr = a.krec + row0 * a.k_stride + 8 * lane;
        const uint8_t* vr = a.vrec + row0 * a.v_stride + 8 * lane;
        // chunks 0..3 (bytes 0..31) cover the first 8 steps from byte 8
        const uint2 k0 = load_chunk(kr, 0, last_k), k1 = load_chunk(kr, 1, last_k), k2 = load_chunk(kr, 2, last_k),
                    k3 = load_chunk(kr, 3, last_k);
        const uint2 v0 = load_chunk(vr, 0, last_v), v1 = load_chunk(vr, 1, last_v), v2 = load_chunk(vr, 2, last_v),
                    v3 = load_chunk(vr, 3, last_v);
        uint2 nk = load_chunk(kr, 4, last_k), nv = load_chunk(vr, 4, last_v);
        wave_sync();   // the previous tile is done with the rings
        put_chunk(ring_k, 0, k0);
        put_chunk(ring_k, 1, k1);
        put_chunk(ring_k, 2, k2);
        put_chunk(ring_k, 3, k3);
        put_chunk(ring_v, 0, v0);
        put_chunk(ring_v, 1, v1);
        put_chunk(ring_v, 2, v2);
        put_chunk(ring_v, 3, v3);
        uint32_t nck = 4, ncv = 4;
        uint32_t thrk = 8u * (8u * 4u - 20u) - 1u, thrv = thrk;
        TChain ck, cv;
        ck.X = k0.y << 3;
        cv.X = v0.y << 3;
        if (W4) corrupt |= valid && min(ck.X, cv.X) < kRansL << 3;   // (one byte a step needs a state from L on)
        ck.pb = cv.pb = 64;                         // payload starts at byte 8
        // (rows past the length may hold anything, and a weight of 0 does not clear an
        // infinity or NaN: their scale and offset are taken as zeros)
        *LDS_PTR(v2u, row_lane + kRowHdr) = v2u{valid ? k0.x : 0u, valid ? v0.x : 0u};
        // the rings are read back by this lane only: order the reads after
        // the writes (LDS keeps a wavefront's accesses in order)
        asm volatile("" ::: "memory");

        for (int h = 0; h < Hkv; ++h) {
            v4i d[HG][4];
#pragma unroll
            for (int hg = 0; hg < HG; ++hg)
#pragma unroll
                for (int tg = 0; tg < 4; ++tg) d[hg][tg] = v4i{0, 0, 0, 0};
            uint32_t vlev[kGroups], k4[4];
            const uint32_t kq = kq_lane + (uint32_t)(h * HG * 2 * kQTile);
            // steps in blocks of 8 (two groups; W4: 16): the rings are refilled after
            // each block, so the block's last reads are awaited (and the next
            // block's requested) after the refill; inside a block, step pair u
            // of both chains: wait for the key chain's first reads (the value
            // chain's follow: 2), finish, request its second table word; the
            // same for the value chain (the key chain's word follows: 1); then
            // the second steps (1, and 2 or 0 at the block's end)
            constexpr int kBlock = W4 ? 3 : 1;
#pragma unroll
            for (int grp = 0; grp < kGroups; ++grp) {
                const bool end = (grp & kBlock) == kBlock;
                if ((grp & kBlock) == 0) {
                    tissue_a<0>(ck, ring_k, mask8k);
                    tissue_a<LUTV>(cv, ring_v, mask8v);
                }
                uint32_t kw[4], vw[4], shk, shv;
                if constexpr (W4) {
                    twait_a<2>(ck);
                    kw[0] = tfinish4<0>(ck, pk3, shk);
                    tissue_b<0>(ck, mask8k);
                    twait_a<1>(cv);
                    vw[0] = tfinish4<0>(cv, pv3, shv);
                    tissue_b<LUTV>(cv, mask8v);
                    twait_b<1>(ck);
                    kw[1] = tfinish4<1>(ck, pk3, shk);
                    tissue_b<0>(ck, mask8k);
                    twait_b<1>(cv);
                    vw[1] = tfinish4<1>(cv, pv3, shv);
                    tissue_b<LUTV>(cv, mask8v);
                    twait_b<1>(ck);
                    kw[2] = tfinish4<2>(ck, pk3, shk);
                    tissue_b<0>(ck, mask8k);
                    twait_b<1>(cv);
                    vw[2] = tfinish4<2>(cv, pv3, shv);
                    tissue_b<LUTV>(cv, mask8v);
                    twait_b<1>(ck);
                    kw[3] = tfinish4<3>(ck, pk3, shk);
                    if (!end) tissue_a<0>(ck, ring_k, mask8k);
                    if (!end) twait_b<2>(cv);
                    else twait_b<0>(cv);
                    vw[3] = tfinish4<3>(cv, pv3, shv);
                    if (!end) tissue_a<LUTV>(cv, ring_v, mask8v);
                } else {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const bool more = !(end && u == 1);
                        twait_a<2>(ck);
                        kw[2 * u] = tfinish_a(ck, pk3, shk);
                        tissue_b<0>(ck, mask8k);
                        twait_a<1>(cv);
                        vw[2 * u] = tfinish_a(cv, pv3, shv);
                        tissue_b<LUTV>(cv, mask8v);
                        twait_b<1>(ck);
                        kw[2 * u + 1] = tfinish_b(ck, pk3, shk);
                        if (more) tissue_a<0>(ck, ring_k, mask8k);
                        if (more) twait_b<2>(cv);
                        else twait_b<0>(cv);
                        vw[2 * u + 1] = tfinish_b(cv, pv3, shv);
                        if (more) tissue_a<LUTV>(cv, ring_v, mask8v);
                    }
                }
                uint32_t lk = pack4(kw[0], kw[1], kw[2], kw[3]);
                vlev[grp] = pack4(vw[0], vw[1], vw[2], vw[3]);
                asm volatile("" : "+v"(lk), "+v"(vlev[grp]));
                key_levels<HG>(grp, lk, k4, row_lane, col_lane, kq, d);
                if (end) {
                    refill2(ck.pb, nck, thrk, nk, ring_k, kr, last_k, cv.pb, ncv, thrv, nv, ring_v, vr, last_v);
                    // a second chunk only where a lane is still short (rare): the
                    // test is one wavefront vote, so blocks where none is skip it
                    if (__any(ck.pb > thrk || cv.pb > thrv))
                        refill2(ck.pb, nck, thrk, nk, ring_k, kr, last_k, cv.pb, ncv, thrv, nv, ring_v, vr, last_v);
                    // the next block's ring reads come after these writes
                    asm volatile("" ::: "memory");
                }
                __builtin_amdgcn_sched_barrier(0);
            }

            // ---- scores of the head's query heads and the online softmax,
            //      at a raised issue priority: its chains of wavefront
            //      reductions then wait less behind the other wavefronts'
            //      decode steps (1.5 % less time at G = 4, 2.3 % at G = 8;
            //      raising the decode instead, as the per-head kernel does,
            //      was 1 % slower here)
            __builtin_amdgcn_s_setprio(1);
            SlotWeights sw[HG];
            float m[HG];
            score_head(d, h, t_base, wbase + L.plimb, sw, m);
#pragma unroll
            for (int hg = 0; hg < HG; ++hg) push_state(sw[hg], m[hg], l16 == 0, m_vec[hg], l_vec[hg], o_vec[hg]);
            __builtin_amdgcn_s_setprio(0);
            wave_sync();   // the weight rows are read by other lanes
            value_head(vlev, wbase + L.plimb, [&](int sl, int hg, int cb, float f) {
                v8f t = acc[sl][hg][cb];
                t[0] = fmaf(f, sw[hg].wscale, t[0] * sw[hg].corr);
                acc[sl][hg][cb] = rot1(t);
            });
            wave_sync();   // the next head rewrites the weight and value rows
        }
        for (int h = Hkv; h < 16; ++h) {
#pragma unroll
            for (int hg = 0; hg < HG; ++hg) {
                m_vec[hg] = row_next(m_vec[hg]);
                l_vec[hg] = row_next(l_vec[hg]);
                o_vec[hg] = row_next(o_vec[hg]);
            }
        }
        for (int h = Hkv; h < kTokMaxHeads; ++h)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int hg = 0; hg < HG; ++hg)
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb) acc[s][hg][cb] = rot1(acc[s][hg][cb]);
        // every stream ends at x = L having read no byte past its record
        corrupt |= valid && ((ck.X >> 3) != kRansL || ck.pb > endk);
        corrupt |= valid && ((cv.X >> 3) != kRansL || cv.pb > endv);
    }
    if (__any(corrupt) && lane == 0 && a.status) atomicOr(a.status, DQ_STATUS_CORRUPT);
    if (PAGED && __any(bad_page) && lane == 0 && a.status) atomicOr(a.status, DQ_STATUS_PAGE);

    // ---- merge the wavefronts of the workgroup, one KV head at a time
    const int NC = a.nchunks;
    float* mw = reinterpret_cast<float*>(smem);        // [nw][GS]
    float* lw = mw + L.nw * GS;                        // [nw][GS]
    float* aw = lw + L.nw * GS;                        // [nw][GS][d]
    for (int h = 0; h < Hkv; ++h) {
        float av[2][HG][4];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int hg = 0; hg < HG; ++hg)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) {
                    av[s][hg][cb] = acc[s][hg][cb][0];
                    acc[s][hg][cb] = rot1(acc[s][hg][cb]);
                }
        __syncthreads();   // LDS free (first head) / previous head merged
#pragma unroll
        for (int hg = 0; hg < HG; ++hg) {
            if (l16 == 0) {
                mw[wave * GS + 4 * hg + pslot] = m_vec[hg];
                lw[wave * GS + 4 * hg + pslot] = l_vec[hg];
            }
            const float ovt = row_first(o_vec[hg]);
            m_vec[hg] = row_next(m_vec[hg]);
            l_vec[hg] = row_next(l_vec[hg]);
            o_vec[hg] = row_next(o_vec[hg]);
            float* row = aw + (wave * GS + 4 * hg + pslot) * kD + (lane & 15);
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) row[s * kVSlice + cb * 16] = av[s][hg][cb] + ovt;
        }
        __syncthreads();
        for (int i = tid; i < G * kD; i += nthr) {
            const int r = i / kD, j = i % kD;
            float M = -INFINITY;
            for (int w = 0; w < L.nw; ++w) M = fmaxf(M, mw[w * GS + r]);
            float acc_o = 0.f, l = 0.f;
            for (int w = 0; w < L.nw; ++w) {
                const float mv = mw[w * GS + r];
                if (mv == -INFINITY) continue;
                const float e = exp2f(mv - M);
                acc_o += aw[(w * GS + r) * kD + j] * e;
                l += lw[w * GS + r] * e;
            }
            const int64_t slot = ((int64_t)b * Hq + h * G + r) * (NC + kResSlots) + c;
            a.ws_acc[slot * kD + j] = acc_o;
            if (j == 0) {
                a.ws_m[slot] = M;
                a.ws_l[slot] = l;
            }
        }
    }
}

constexpr TokLayout tok_layout(int pk, int pv, bool shared_lut, int Hq, int Hkv, int chunk, int nw, int HG) {
    TokLayout L{};
    int off = 0;
    L.lut_k = off;
    off += 8 << pk;
    L.lut_v = shared_lut ? L.lut_k : off;
    if (!shared_lut) off += 8 << pv;
    L.qtile = off;
    off += Hkv * HG * 2 * kQTile;
    L.qscale = off;
    off += 4 * Hq;
    L.qsum = off;
    off += 4 * Hq;
    L.qmu = off;
    off += 4 * Hq * ((chunk + DQ_MEAN_WINDOW - 1) / DQ_MEAN_WINDOW + 1);
    off = (off + 15) & ~15;
    L.waves = off;
    L.ring_k = 0;
    L.ring_v = kRingBytes;
    L.vtile = 2 * kRingBytes;
    L.plimb = L.vtile + kTile * kRowT;
    L.wave_stride = L.plimb + HG * kTile * 16;
    L.nw = nw;
    // the prologue's query scratch and the epilogue's merge buffers use the
    // wavefront regions
    const int scratch = std::max(Hq * kD * 4, nw * 4 * HG * (kD + 2) * 4);
    L.total = L.waves + std::max(nw * L.wave_stride, scratch);
    return L;
}

}  // namespace

// At least one workgroup per CU where the batch allows it, chunks of at most
// kTokMaxChunk tokens and at least kMinChunk (two tiles: at batch 1 a
// token's 1024-step chains bound the time, so more, smaller workgroups
// shorten it, one decoding wavefront per SIMD).
int32_t token_chunk(int32_t B, int32_t t_cap) {
    const int64_t nc = std::max<int64_t>((t_cap + kTokMaxChunk - 1) / kTokMaxChunk, (cu_count() + B - 1) / B);
    int chunk = (int)((t_cap + nc - 1) / nc);
    chunk = ((chunk + kTile - 1) / kTile) * kTile;
    chunk = std::max(chunk, kMinChunk);
    return std::min(chunk, kTokMaxChunk);
}

namespace {

template <uint32_t LUTV, int HG, bool W4>
int launch_token_kernel(const TokArgs& a, dim3 grid, int nw, hipStream_t stream) {
    const bool paged = a.pg.bt != nullptr;
    // chunks of at most 4 tiles (small batches, short contexts): keys and
    // values in different wavefronts (up to 4 query heads, when LDS holds 8
    // wavefronts)
    if constexpr (HG == 1) {
        TokArgs s = a;
        s.L = tok_layout(a.tk.p, a.tv.p, a.L.lut_v == a.L.lut_k, a.Hq, a.Hkv, a.chunk, kTokSplitWaves, 1);
        // (two 4096-entry tables leave no room for 8 wavefronts: both chains in one)
        if (2 * ((a.chunk + kTile - 1) / kTile) <= kTokSplitWaves && s.L.total <= kMaxLds) {
            const void* fn = paged ? reinterpret_cast<const void*>(&attn_token_kernel<LUTV, true, 1, true, W4>)
                                   : reinterpret_cast<const void*>(&attn_token_kernel<LUTV, false, 1, true, W4>);
            if (int rc = hip_check("hipFuncSetAttribute",
                                   hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, s.L.total)))
                return rc;
            if (paged)
                attn_token_kernel<LUTV, true, 1, true, W4><<<grid, kTokSplitWaves * kWave, (size_t)s.L.total, stream>>>(s);
            else
                attn_token_kernel<LUTV, false, 1, true, W4><<<grid, kTokSplitWaves * kWave, (size_t)s.L.total, stream>>>(s);
            return hip_check("attn_token launch", hipGetLastError());
        }
    }
    const void* fn = paged ? reinterpret_cast<const void*>(&attn_token_kernel<LUTV, true, HG, false, W4>)
                           : reinterpret_cast<const void*>(&attn_token_kernel<LUTV, false, HG, false, W4>);
    if (int rc = hip_check("hipFuncSetAttribute",
                           hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, a.L.total)))
        return rc;
    const size_t smem = (size_t)a.L.total;
    if (paged)
        attn_token_kernel<LUTV, true, HG, false, W4><<<grid, nw * kWave, smem, stream>>>(a);
    else
        attn_token_kernel<LUTV, false, HG, false, W4><<<grid, nw * kWave, smem, stream>>>(a);
    return hip_check("attn_token launch", hipGetLastError());
}

template <int HG>
int launch_token_hg(const TokArgs& a, dim3 grid, int nw, bool shared, hipStream_t stream) {
    // four steps per ring read where both tables have p = 8, whose steps take at
    // most one byte, else two (16 x 32768 tokens at p = 8: 386 and 434 us)
    const bool w4 = a.tk.p == 8 && a.tv.p == 8;
    switch (shared ? 0u : (uint32_t)a.L.lut_v) {
        case 0:
            return w4 ? launch_token_kernel<0, HG, true>(a, grid, nw, stream)
                      : launch_token_kernel<0, HG, false>(a, grid, nw, stream);
        case 8u << 8:
            return w4 ? launch_token_kernel<8u << 8, HG, true>(a, grid, nw, stream)
                      : launch_token_kernel<8u << 8, HG, false>(a, grid, nw, stream);
        case 8u << 9: return launch_token_kernel<8u << 9, HG, false>(a, grid, nw, stream);
        case 8u << 10: return launch_token_kernel<8u << 10, HG, false>(a, grid, nw, stream);
        case 8u << 11: return launch_token_kernel<8u << 11, HG, false>(a, grid, nw, stream);
        case 8u << 12: return launch_token_kernel<8u << 12, HG, false>(a, grid, nw, stream);
        default: return DQ_ERR_INVALID_ARG;
    }
}

}  // namespace

int launch_attention_token_partial(const dq_tables* tk, const dq_tables* tv, const Pages& pg, const uint16_t* q,
                                   int32_t B,
                                   int32_t Hq, int32_t Hkv, const uint8_t* krec, int32_t k_stride,
                                   const int8_t* kmq, const uint16_t* kms, const uint8_t* vrec,
                                   int32_t v_stride, const int32_t* seq_lens, int32_t t_cap, float scale,
                                   void* ws, uint32_t* status, hipStream_t stream) {
    TokArgs a;
    a.tk = tab_args(tk);
    a.tv = tab_args(tv);
    const bool shared = tk == tv;
    a.q = q;
    a.Hq = Hq;
    a.Hkv = Hkv;
    a.G = Hq / Hkv;
    a.t_cap = t_cap;
    a.chunk = token_chunk(B, t_cap);
    a.nchunks = (t_cap + a.chunk - 1) / a.chunk;
    a.krec = krec;
    a.kmq = kmq;
    a.kms = kms;
    a.vrec = vrec;
    a.k_stride = k_stride;
    a.v_stride = v_stride;
    a.pg = pg;
    a.seq_lens = seq_lens;
    a.rot_q = tk->cfg.prerotated ? 0 : 1;
    a.rot_out = tv->cfg.prerotated ? 0 : 1;
    a.q_scale = scale * 1.4426950408889634f / (a.rot_q ? (float)kD : 1.0f);
    const int64_t slots = ws_slots(B, Hq, t_cap);
    a.ws_hdr = static_cast<int32_t*>(ws);
    a.ws_acc = reinterpret_cast<float*>(static_cast<uint8_t*>(ws) + kWsHeader);
    a.ws_m = a.ws_acc + slots * kD;
    a.ws_l = a.ws_m + slots;
    a.status = status;
    if (a.G < 1 || a.G > 8) return DQ_ERR_INVALID_ARG;
    const int HG = a.G > 4 ? 2 : 1;
    int nw = tok_waves(HG);
    for (; nw > 0; --nw) {
        a.L = tok_layout(a.tk.p, a.tv.p, shared, Hq, Hkv, a.chunk, nw, HG);
        if (a.L.total <= kMaxLds) break;
    }
    if (nw == 0) return DQ_ERR_INVALID_ARG;
    const dim3 grid(a.nchunks, 1, B);
    return HG == 1 ? launch_token_hg<1>(a, grid, nw, shared, stream) : launch_token_hg<2>(a, grid, nw, shared, stream);
}

}  // namespace dq
