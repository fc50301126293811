// Baseline JPEG encoder for CDNA4 (gfx950): the per-frame payload of the
// paper's backend (Section 5.1, Rendering Engine: frames leave as 8-bit JPEG;
// Sections 4.2 and 5.2: one stateless JPEG per request; Table 1 pairs each
// resolution of the bitrate ladder with a quality factor).
//
//   k_jpeg_seg    one workgroup per restart interval (40 MCUs in raster
//                 order, eight lanes per 8x8 block): colour transform, forward
//                 DCT and quantisation into LDS, the entropy-coded length of
//                 every eighth of a block (DC prediction inside the interval),
//                 a workgroup scan of those lengths, then the Huffman codes
//                 ORed into an LDS window of the interval's bit stream, which
//                 leaves for global memory padded with 1-bits; the interval's
//                 output length (one 0x00 for every 0xFF byte, the marker)
//   k_jpeg_pack   per interval: output offset = header + the intervals before
//                 it; the bytes with stuffing, the RSTn marker (EOI after the
//                 last); the first interval's workgroup writes the header
//
// One pair of launches encodes up to JPEG_MAX_JOBS frames, whose parameters
// travel as kernel arguments.
//
// Format choices (the standard leaves them open; the JPEG oracle makes the
// same ones): JFIF full-range YCbCr, 4:4:4, orthonormal DCT-II as two FP32
// FMA chains (columns of each row first, then rows), quantisation
// x = F (1/Q), q = trunc(x + copysign(1/2, x)), AC clamped to +-1023, the
// Annex K tables scaled by quality, restart intervals of 40 MCUs.
#include "tigas_internal.h"

namespace tigas {

namespace {

// Zig-zag scan position (Figure A.6) of column l, row k at byte l * 8 + k:
// a lane that holds a column of coefficients reads its eight positions as two
// words.  Built by walking the anti-diagonals: upwards on even ones, downwards
// on odd ones.
struct ZigZagColumns {
    uint32_t w[16];
    constexpr ZigZagColumns() : w{} {
        uint32_t i = 0;
        for (int d = 0; d < 15; ++d) {
            const int hi = d < 8 ? d : 7, lo = d < 8 ? 0 : d - 7;
            for (int j = hi; j >= lo; --j) {
                const int row = (d & 1) ? d - j : j, col = d - row;
                w[col * 2 + row / 4] |= i++ << (8 * (row & 3));
            }
        }
    }
};
__constant__ ZigZagColumns kZigZag = ZigZagColumns();

__device__ __forceinline__ int magnitude_bits(int v) { return 32 - __clz(v < 0 ? -v : v); }
// A value's nb magnitude bits: negative values as v - 1.
__device__ __forceinline__ uint32_t value_bits(int v, int nb) {
    return (uint32_t)(v < 0 ? v - 1 : v) & ((1u << nb) - 1u);
}

// Bit writer: put(value, nbits), value holding exactly nbits bits, most
// significant first, into a window of nwords words of the interval's stream
// (stream bit i at bit 31 - i % 32 of word i / 32) that starts at word w0;
// bits outside it are dropped.
struct BitWrite {
    uint32_t* win;
    uint32_t w0, nwords;
    uint64_t acc;  // pending bits, left-aligned
    int n;         // pending bit count
    uint32_t w;    // word the pending bits start in
    __device__ BitWrite(uint32_t* b, uint32_t first, uint32_t words, uint32_t start)
        : win(b), w0(first), nwords(words), acc(0), n((int)(start & 31u)), w(start >> 5) {}
    __device__ void emit() {  // a word may be shared with the neighbouring lane's codes
        if (w - w0 < nwords) atomicOr(&win[w - w0], (uint32_t)(acc >> 32));
    }
    __device__ void put(uint32_t v, int nb) {  // nb <= 27, so one word at most becomes full
        acc |= (uint64_t)v << (64 - n - nb);
        n += nb;
        if (n >= 32) {
            emit();
            acc <<= 32;
            n -= 32;
            ++w;
        }
    }
    __device__ void flush() {
        if (n > 0) emit();
    }
};

// A symbol's Huffman code (e: length << 16 | code) followed by its value's nb
// bits (at most 16 + 10), as total length << 27 | bits.
__device__ __forceinline__ uint32_t packed_code(uint32_t e, int v, int nb) {
    return (((e >> 16) + (uint32_t)nb) << 27) | ((e & 0xffffu) << nb) | value_bits(v, nb);
}

// Inclusive prefix sum over a wave's 64 lanes (DPP row shifts and broadcasts).
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

// 0xFF bytes among the first n (<= 4) bytes of a word, most significant first.
__device__ __forceinline__ uint32_t count_ff(uint32_t w, uint32_t n) {
    uint32_t c = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) c += (k < n && ((w >> (24 - 8 * k)) & 0xffu) == 0xffu) ? 1u : 0u;
    return c;
}

// The job of workgroup `wg` (the intervals of all jobs are numbered through).
__device__ __forceinline__ int job_of(const JpegBatch& a, uint32_t wg) {
    int j = 0;
    while (j + 1 < a.njobs && wg >= a.job[j + 1].seg_base) ++j;
    return j;
}

// Annex K base tables (Tables K.1 and K.2), row-major.
__constant__ uint8_t kQBase[2][64] = {JPEG_QLUMA, JPEG_QCHROMA};

__device__ __forceinline__ uint32_t quant_step(int table, int i, int quality) {
    return (uint32_t)jpeg_quant_step(kQBase[table][i], quality);
}

}  // namespace

// What bounds it: in small frames one workgroup's chain of load, transform,
// code, scan and write, in large ones VALU issue (about 1000 instructions a
// wave, a quarter of them the transform's FMAs), never the 3 bytes per pixel.
// So a block is spread over eight lanes, the whole stream of an interval is
// formed in LDS, and every code is looked up once and kept packed in a
// register from the length count to the write.  A wave codes one eighth of
// the scan of 64 blocks, not eight blocks whole: the high eighths are nearly
// empty at any usual quality and cost little (1006 against 1800 VALU
// instructions a wave).  512 threads and 80 VGPRs hold three workgroups per
// CU; 1024 threads gained 1 us below 200 intervals and lost 46 us at 3240, and
// 64 VGPRs spill.  Against one thread per block (128-thread workgroups, codes
// ORed into global memory): 1280x720 27 -> 11 us, 3840x2160 73 -> 44 us.
__global__ __launch_bounds__(JPEG_SEG_THREADS, 6) void k_jpeg_seg(JpegBatch a) {
    constexpr int NT = JPEG_SEG_THREADS;
    constexpr int NB = 3 * JPEG_SEG_MCUS;
    constexpr int NW = NT / 64, TASKS = 16, TPW = TASKS / NW;
    static_assert(NB <= 128 && TASKS % NW == 0, "the eighths of 128 blocks are 16 tasks of one wave");
    // quantised coefficients in zig-zag order, rows of 72 halves (16-byte
    // aligned eighths, 36 words apart: 16 lanes read theirs in one step), later
    // the window of the bit stream; transposed rows of 72 floats per block
    // (the eight columns of eight blocks meet in 64 different banks), later
    // the eighths' lengths and offsets
    constexpr int ZS = 72, TS = 72;
    constexpr uint32_t WIN = 2048;
    __shared__ __align__(16) int16_t s_coef[NB * ZS];
    __shared__ __align__(16) float s_tr[NT / 8 * TS];
    static_assert(WIN * 2 <= NB * ZS && NT / 8 * TS >= 1024, "room for the window and the eighths' lengths");
    uint32_t* const s_win = reinterpret_cast<uint32_t*>(s_coef);
    uint32_t* const s_len = reinterpret_cast<uint32_t*>(s_tr);
    __shared__ __align__(8) uint8_t s_nz[128 * 8];     // per block and eighth: its non-zero positions
    __shared__ uint32_t s_ac[2 * 256], s_dct[2 * 16];  // Huffman codes: AC and DC, luma and chroma
    __shared__ float s_rq[2 * 64];
    __shared__ uint32_t s_ws[NW], s_ff[NW];
    const int t = threadIdx.x, lane = t & 63, l = t & 7;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int ji = job_of(a, blockIdx.x);
    const JpegJobArgs& job = a.job[ji];
    const uint32_t seg = blockIdx.x - job.seg_base;
    const uint32_t m0 = seg * JPEG_SEG_MCUS;
    const int nb = 3 * (int)min((uint32_t)JPEG_SEG_MCUS, job.n_mcu - m0);
    const int W = job.width, H = job.height;

    for (int i = t; i < 512; i += NT) s_ac[i] = a.huff[(i >> 8) * 512 + 256 + (i & 255)];
    if (t < 32) s_dct[t] = a.huff[(t >> 4) * 512 + (t & 15)];
    if (t < 128) s_rq[t] = 1.0f / (float)quant_step(t >> 6, t & 63, job.quality);
    const uint2 zz = make_uint2(kZigZag.w[2 * l], kZigZag.w[2 * l + 1]);
    __syncthreads();

    // transform and quantise: eight lanes per block (Y, Cb, Cr of each MCU);
    // lanes past the interval's last block take its first one's pixels and are
    // dropped by the coder
#pragma unroll 1
    for (int b = t >> 3; b < NB; b += NT / 8) {  // whole waves
        const int comp = b % 3;
        const uint32_t mcu = m0 + (b < nb ? (uint32_t)b / 3u : 0u);
        const int my = (int)(mcu / (uint32_t)job.w8), mx = (int)(mcu - (uint32_t)my * (uint32_t)job.w8);
        const int x0 = mx * 8, y = min(my * 8 + l, H - 1);
        const uint8_t* row = job.rgb + (size_t)y * W * 3;
        uint32_t pw[6];  // the row's 24 bytes
        if (x0 + 8 <= W) {
            __builtin_memcpy(pw, row + (size_t)x0 * 3, 24);
        } else {  // edge pixels repeated
#pragma unroll
            for (int i = 0; i < 6; ++i) pw[i] = 0u;
#pragma unroll
            for (int i = 0; i < 24; ++i) {
                const uint32_t v = row[(size_t)min(x0 + i / 3, W - 1) * 3 + i % 3];
                pw[i >> 2] |= v << (8 * (i & 3));
            }
        }
        // one form for the three components: fma(kb, B, fma(kg, G, kr R)) - k0
        const float kr = comp == 0 ? 0.299f : comp == 1 ? -0.168736f : 0.5f;
        const float kg = comp == 0 ? 0.587f : comp == 1 ? -0.331264f : -0.418688f;
        const float kb = comp == 0 ? 0.114f : comp == 1 ? 0.5f : -0.081312f;
        const float k0 = comp == 0 ? 128.0f : 0.0f;
        float f[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            auto byte = [&](int i) { return (float)((pw[i >> 2] >> (8 * (i & 3))) & 0xffu); };
            f[c] = __builtin_fmaf(kb, byte(3 * c + 2), __builtin_fmaf(kg, byte(3 * c + 1), kr * byte(3 * c))) - k0;
        }
        // this lane's row along x, then (through LDS) its column along y
        float* tr = s_tr + (t >> 3) * TS;
        float o[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float acc = 0.0f;
#pragma unroll
            for (int c = 0; c < 8; ++c) acc = __builtin_fmaf(f[c], a.dct[k * 8 + c], acc);
            o[k] = acc;
        }
        float4* trow = reinterpret_cast<float4*>(tr + l * 8);
        trow[0] = make_float4(o[0], o[1], o[2], o[3]);
        trow[1] = make_float4(o[4], o[5], o[6], o[7]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        float col[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) col[r] = tr[r * 8 + l];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const float* rq = s_rq + (comp ? 64 : 0);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float acc = 0.0f;
#pragma unroll
            for (int r = 0; r < 8; ++r) acc = __builtin_fmaf(a.dct[k * 8 + r], col[r], acc);
            const float x = acc * rq[k * 8 + l];
            int v = (int)(x + __builtin_copysignf(0.5f, x));  // towards zero
            if (k > 0) v = max(-1023, min(1023, v));
            else v = l ? max(-1023, min(1023, v)) : v;
            const uint32_t p = ((k < 4 ? zz.x : zz.y) >> (8 * (k & 3))) & 0xffu;
            s_coef[b * ZS + (int)p] = (int16_t)v;
        }
    }
    __syncthreads();

    // Entropy coding (Annex F), one task per eighth (scan positions 8j .. 8j +
    // 7) of 64 blocks: a lane's block is the same in all of them, and the
    // waves of the high eighths, where few blocks hold a value, skip most
    // positions.  First which positions are non-zero ...
    auto coefs = [&](int j, int b) {  // the eight values as half words
        return b < nb ? *reinterpret_cast<const uint4*>(s_coef + b * ZS + 8 * j) : make_uint4(0u, 0u, 0u, 0u);
    };
    auto task = [&](int q) { return q * NW + ((q & 1) ? NW - 1 - wv : wv); };
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        const int j = task(q) >> 1, b = (task(q) & 1) * 64 + lane;
        const uint4 c = coefs(j, b);
        const uint32_t w[4] = {c.x, c.y, c.z, c.w};
        uint32_t m = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) m |= ((w[k / 2] >> (16 * (k & 1))) & 0xffffu) ? 1u << k : 0u;
        s_nz[b * 8 + j] = (uint8_t)m;
    }
    __syncthreads();
    // ... then each position's code and value bits (DC: the difference to the
    // previous block of the component, starting at zero in each interval)
    uint32_t sym[TPW][8], nzrl[TPW], eob[TPW];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        const int j = task(q) >> 1, b = (task(q) & 1) * 64 + lane;
        const uint32_t* hac = s_ac + (b % 3 ? 256 : 0);
        uint64_t ac = *reinterpret_cast<const uint64_t*>(s_nz + b * 8) & ~1ull;
        if (b >= nb) ac = 0;
        const uint4 c = coefs(j, b);
        const uint32_t w[4] = {c.x, c.y, c.z, c.w};
        const uint32_t mine = (uint32_t)(ac >> (8 * j)) & 0xffu;
        // scan position of the last value before this eighth (the DC's at least)
        const uint64_t earlier = (ac & ((1ull << (8 * j)) - 1ull)) | 1ull;
        int prev = 63 - __clzll((long long)earlier);
        uint32_t total = 0;
        nzrl[q] = 0;
        eob[q] = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            sym[q][k] = 0u;
            if (k == 0 && j == 0) {
                if (b < nb) {
                    const int dc = (int)(int16_t)w[0];
                    const int diff = dc - (b >= 3 ? (int)s_coef[(b - 3) * ZS] : 0);
                    const int nd = magnitude_bits(diff);
                    sym[q][0] = packed_code(s_dct[(b % 3 ? 16 : 0) + nd], diff, nd);
                }
            } else if (mine & (1u << k)) {
                const int i = 8 * j + k;
                const int run = i - prev - 1;
                if (run > 15) nzrl[q] = (uint32_t)run >> 4;  // only an eighth's first value can follow 16 zeros
                const int v = (k & 1) ? (int)w[k / 2] >> 16 : (int)(int16_t)w[k / 2];
                const int nv = magnitude_bits(v);
                sym[q][k] = packed_code(hac[((run & 15) << 4) | nv], v, nv);
                prev = i;
            }
            total += sym[q][k] >> 27;
        }
        if (nzrl[q]) total += nzrl[q] * (hac[0xF0] >> 16);
        if (j == 7 && b < nb && (ac >> 63) == 0) {
            eob[q] = hac[0x00];
            total += eob[q] >> 16;
        }
        s_len[b * 8 + j] = total;
        __builtin_amdgcn_sched_barrier(0);  // one task's temporaries at a time: within the 80 VGPRs of three workgroups per CU
    }
    __syncthreads();
    // the eighths' bit offsets: a scan in stream order, in place
    constexpr int SC = 1024 / NT;
    uint32_t ln[SC], sum = 0;
#pragma unroll
    for (int i = 0; i < SC; ++i) sum += ln[i] = s_len[t * SC + i];
    const uint32_t incl = wave_scan(sum);
    if (lane == 63) s_ws[wv] = incl;
    __syncthreads();
    uint32_t bits = 0, before = incl - sum;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        const uint32_t x = s_ws[v];
        before += v < wv ? x : 0u;
        bits += x;
    }
#pragma unroll
    for (int i = 0; i < SC; ++i) {
        s_len[t * SC + i] = before;
        before += ln[i];
    }

    // the codes, window by window (one window but for the noisiest intervals);
    // the coefficients are in registers by now
    const uint32_t nbytes = (bits + 7) / 8, nwords = (bits + 31) / 32;
    uint32_t* const out = a.bits + (size_t)blockIdx.x * a.seg_words;
    uint32_t ff = 0;
    for (uint32_t w0 = 0; w0 < nwords; w0 += WIN) {
        const uint32_t nw = min(WIN, nwords - w0);
        for (uint32_t i = t; i < nw; i += NT) s_win[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int j = task(q) >> 1, b = (task(q) & 1) * 64 + lane;
            const uint32_t* hac = s_ac + (b % 3 ? 256 : 0);
            BitWrite w(s_win, w0, nw, s_len[b * 8 + j]);
            if (nzrl[q]) {
                const uint32_t e = hac[0xF0];
                for (uint32_t i = 0; i < nzrl[q]; ++i) w.put(e & 0xffffu, (int)(e >> 16));
            }
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (sym[q][k]) w.put(sym[q][k] & 0x7ffffffu, (int)(sym[q][k] >> 27));
            if (eob[q]) w.put(eob[q] & 0xffffu, (int)(eob[q] >> 16));
            w.flush();
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        for (uint32_t i = t; i < nw; i += NT) {
            uint32_t v = s_win[i];
            const uint32_t w = w0 + i;
            if (w + 1 == nwords && (bits & 31u)) v |= ~0u >> (bits & 31u);  // pad bits are ones
            out[w] = v;
            ff += count_ff(v, nbytes - 4 * w);
        }
        __syncthreads();
    }
    ff = wave_scan(ff);
    if (lane == 63) s_ff[wv] = ff;
    __syncthreads();
    if (t == 0) {
        uint32_t total = 0;
        for (int v = 0; v < NW; ++v) total += s_ff[v];
        a.seg_bytes[blockIdx.x] = nbytes;
        a.seg_len[blockIdx.x] = nbytes + total + (seg + 1 < job.nseg ? 2u : 0u);
    }
}

__global__ __launch_bounds__(JPEG_PACK_THREADS) void k_jpeg_pack(JpegBatch a) {
    constexpr int NT = JPEG_PACK_THREADS, NW = NT / 64;
    __shared__ uint32_t s_w[NW];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int ji = job_of(a, blockIdx.x);
    const JpegJobArgs& job = a.job[ji];
    const uint32_t seg = blockIdx.x - job.seg_base;
    const uint32_t nbytes = a.seg_bytes[blockIdx.x];
    const uint32_t* buf = a.bits + (size_t)blockIdx.x * a.seg_words;
    // output offset of the interval: the header and every interval before it
    uint32_t before = 0;
    for (uint32_t r = t; r < seg; r += NT) before += a.seg_len[job.seg_base + r];
    before = wave_scan(before);
    if (lane == 63) s_w[wv] = before;
    __syncthreads();
    uint64_t base = a.header_len;
#pragma unroll
    for (int v = 0; v < NW; ++v) base += s_w[v];
    if (seg == 0) {
        // the header: the constant template with the frame size and the
        // quantisation tables (zig-zag order) filled in
        for (uint32_t i = t; i < a.header_len; i += NT) {
            uint32_t v = a.header[i];
            if (i >= JPEG_HDR_SIZE && i < JPEG_HDR_SIZE + 4) {
                const uint32_t d = i < JPEG_HDR_SIZE + 2 ? (uint32_t)job.height : (uint32_t)job.width;
                v = ((i - JPEG_HDR_SIZE) & 1u) ? d & 0xffu : d >> 8;
            }
#pragma unroll
            for (int tab = 0; tab < 2; ++tab) {
                const uint32_t q0 = tab ? JPEG_HDR_QCHROMA : JPEG_HDR_QLUMA;
                if (i >= q0 && i < q0 + 64) {
                    const uint32_t zi = a.zigzag[i - q0];
                    v = quant_step(tab, (int)zi, job.quality);
                }
            }
            if (i < job.capacity) job.out[i] = (uint8_t)v;
        }
    }
    // four bytes of the stream per lane, placed by the 0xFF bytes before them
    uint32_t ff_done = 0;
    for (uint32_t w0 = 0; 4 * w0 < nbytes; w0 += NT) {
        const uint32_t j = 4 * (w0 + (uint32_t)t);
        const uint32_t n = j < nbytes ? min(4u, nbytes - j) : 0u;
        const uint32_t v = n ? buf[w0 + t] : 0u;
        const uint32_t ff = count_ff(v, n);
        const uint32_t incl = wave_scan(ff);
        __syncthreads();
        if (lane == 63) s_w[wv] = incl;
        __syncthreads();
        uint32_t ahead = ff_done + incl - ff;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const uint32_t x = s_w[k];
            ahead += k < wv ? x : 0u;
            ff_done += x;
        }
        uint64_t pos = base + j + ahead;
        for (uint32_t k = 0; k < n; ++k) {
            const uint32_t byte = (v >> (24 - 8 * k)) & 0xffu;
            if (pos < job.capacity) job.out[pos] = (uint8_t)byte;
            ++pos;
            if (byte == 0xffu) {
                if (pos < job.capacity) job.out[pos] = 0;
                ++pos;
            }
        }
    }
    if (t == 0) {
        const uint64_t end = base + nbytes + ff_done;
        const bool last = seg + 1 == job.nseg;
        const uint8_t m = last ? 0xD9 : (uint8_t)(0xD0 + (seg & 7));  // RSTn, or EOI after the last interval
        if (end < job.capacity) job.out[end] = 0xFF;
        if (end + 1 < job.capacity) job.out[end + 1] = m;
        if (last) *job.out_len = end + 2;
    }
}

#define TIGAS_JPEG_LAUNCH(kernel, grid, block, st, a)                             \
    do {                                                                          \
        KernelTimer* kt_ = g_kernel_timer;                                        \
        if (kt_) kt_->before(reinterpret_cast<const void*>(kernel), st);         \
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, st, a);            \
        if (kt_) kt_->after(st);                                                  \
    } while (0)

void launch_jpeg(const JpegBatch& a, uint32_t nseg, hipStream_t st) {
    TIGAS_JPEG_LAUNCH(k_jpeg_seg, nseg, JPEG_SEG_THREADS, st, a);
    TIGAS_JPEG_LAUNCH(k_jpeg_pack, nseg, JPEG_PACK_THREADS, st, a);
}

}  // namespace tigas
