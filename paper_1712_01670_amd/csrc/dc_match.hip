// Block matching (Section 4, Steps 1-4) for gfx950.
//
// Kernel 1 (search): one workgroup per block of the grid.  The search window of the
// previous frame and the block of the current frame are staged in LDS with coalesced
// dword loads; every lane owns a few candidate vectors and evaluates
//     SSD = sum a^2 + sum b^2 - 2 sum a*b
// four samples per instruction with packed-u8 dot products; the arg-min key
// (ssd, |dx|+|dy|, dy, dx) is packed in 64 bits and reduced with wavefront shuffles.
// Kernel 2 (motion + re-test): every workgroup recomputes the stream's mean motion
// from the per-block results (a few hundred values) and re-tests its own block.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "dc_internal.h"

namespace dc {

namespace {

constexpr int kSearchThreads = 512;

__device__ __forceinline__ uint32_t udot4(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_udot4(a, b, c, false);
}

__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        unsigned long long o = __shfl_xor(v, off, 64);
        v = o < v ? o : v;
    }
    return v;
}

// Sum over the 64 lanes, returned to every lane.  Data-parallel-primitive moves instead of LDS permutes (a
// dependent chain of six permutes costs more than a round of the diamond search should): within quads by
// quad permutation, within a row of 16 by row shifts, across rows by broadcasting lane 15 / lane 31 into
// the following rows; lanes without a source add zero.  The total ends up in lane 63.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_add(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ int wave_sum_i32(int v) {
    v = dpp_add<0xb1, 0xf>(v);    // quad_perm [1,0,3,2]
    v = dpp_add<0x4e, 0xf>(v);    // quad_perm [2,3,0,1]
    v = dpp_add<0x114, 0xf>(v);   // row_shr:4
    v = dpp_add<0x118, 0xf>(v);   // row_shr:8
    v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}

// LDS layout (bytes):
//   win : (B+2R) rows of `ws` bytes; row r holds previous-frame bytes
//         [a0, a0+ws) of frame row y0-R+r, a0 = 4-byte-aligned start at or below the
//         window's first byte; bytes outside the frame are zero
//   blk : B rows of `cs` bytes (cs = B*C rounded up to 4), zero padded
// CDW > 0: the block row is CDW dwords (compile-time, inner loop fully unrolled so that the LDS reads of a
// row are issued together); CDW == 0: any row length.
template <bool ALIGNED, int CDW>
__global__ __launch_bounds__(kSearchThreads) void match_search_kernel(
    const uint8_t* __restrict__ cur, const uint8_t* __restrict__ prev, int H, int W, int C, int B,
    int R, int gw, int gh, int ws, int cs, int k_skip, int16_t* __restrict__ mv, uint32_t* __restrict__ best_ssd) {
    extern __shared__ __align__(16) uint8_t lds[];
    const int tid = threadIdx.x;
    // k-skip: the grid covers only the blocks on every k-th grid row and column
    const int lgw = (gw + k_skip - 1) / k_skip;
    const int bx = ((int)blockIdx.x % lgw) * k_skip, by = ((int)blockIdx.x / lgw) * k_skip;
    const int blk_id = by * gw + bx, stream = blockIdx.y;
    const int x0 = bx * B, y0 = by * B;
    const int rows = B + 2 * R;
    const int row_bytes = W * C;
    const size_t frame_bytes = (size_t)H * row_bytes;
    const uint8_t* pf = prev + (size_t)stream * frame_bytes;
    const uint8_t* cf = cur + (size_t)stream * frame_bytes;
    uint8_t* win = lds;
    uint8_t* blk = lds + (size_t)rows * ws;
    __shared__ unsigned long long red[kSearchThreads / 64];

    const int gx0 = (x0 - R) * C;        // first window byte within the frame row (may be < 0)
    const int a0 = gx0 & ~3;             // aligned start (two's complement floor)
    const int skew = gx0 - a0;

    // ---- stage the search window ----
    const int wdw = ws / 4;
    for (int i = tid; i < rows * wdw; i += kSearchThreads) {
        int r = i / wdw, j = i - r * wdw;
        int y = y0 - R + r;
        int fb = a0 + 4 * j;
        uint32_t v = 0;
        if (y >= 0 && y < H) {
            const uint8_t* src = pf + (size_t)y * row_bytes;
            if (ALIGNED && fb >= 0 && fb + 3 < row_bytes) {
                v = *reinterpret_cast<const uint32_t*>(src + fb);
            } else {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    int f = fb + b;
                    if (f >= 0 && f < row_bytes) v |= (uint32_t)src[f] << (8 * b);
                }
            }
        }
        reinterpret_cast<uint32_t*>(win)[i] = v;
    }
    // ---- stage the current block, zero padded to whole dwords ----
    const int cdw = CDW > 0 ? CDW : cs / 4;
    const int blk_bytes = B * C;
    for (int i = tid; i < B * cdw; i += kSearchThreads) {
        int r = i / cdw, j = i - r * cdw;
        const uint8_t* src = cf + (size_t)(y0 + r) * row_bytes + (size_t)x0 * C;
        uint32_t v = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            int f = 4 * j + b;
            if (f < blk_bytes) v |= (uint32_t)src[f] << (8 * b);
        }
        reinterpret_cast<uint32_t*>(blk)[i] = v;
    }
    __syncthreads();

    // sum a^2 (every lane computes it: B*cdw broadcast reads)
    uint32_t saa = 0;
    for (int i = 0; i < B * cdw; ++i) {
        uint32_t a = reinterpret_cast<const uint32_t*>(blk)[i];
        saa = udot4(a, a, saa);
    }
    const int tail = blk_bytes - 4 * (cdw - 1);                 // valid bytes of a row's last dword
    const uint32_t tail_mask = tail >= 4 ? 0xffffffffu : ((1u << (8 * tail)) - 1u);

    const int side = 2 * R + 1;
    unsigned long long best = ~0ull;
    for (int c = tid; c < side * side; c += kSearchThreads) {
        int dy = c / side - R, dx = c - (c / side) * side - R;
        if (x0 + dx < 0 || y0 + dy < 0 || x0 + dx + B > W || y0 + dy + B > H) continue;
        const int boff = skew + (dx + R) * C;   // byte offset of the candidate inside a window row
        const int sh = boff & 3;
        uint32_t sab = 0, sbb = 0;
        for (int r = 0; r < B; ++r) {
            const uint32_t* wrow = reinterpret_cast<const uint32_t*>(win + (size_t)(r + dy + R) * ws) + (boff >> 2);
            const uint32_t* arow = reinterpret_cast<const uint32_t*>(blk + (size_t)r * cs);
            if (CDW > 0) {
                uint32_t wv[CDW + 1], av[CDW > 0 ? CDW : 1];
#pragma unroll
                for (int j = 0; j <= CDW; ++j) wv[j] = wrow[j];
#pragma unroll
                for (int j = 0; j < CDW; ++j) av[j] = arow[j];
#pragma unroll
                for (int j = 0; j < CDW; ++j) {
                    uint32_t b = __builtin_amdgcn_alignbyte(wv[j + 1], wv[j], sh);
                    if (j == CDW - 1) b &= tail_mask;
                    sab = udot4(av[j], b, sab);
                    sbb = udot4(b, b, sbb);
                }
            } else {
                uint32_t lo = wrow[0];
                for (int j = 0; j < cdw; ++j) {
                    uint32_t hi = wrow[j + 1];
                    uint32_t b = __builtin_amdgcn_alignbyte(hi, lo, sh);
                    if (j == cdw - 1) b &= tail_mask;
                    uint32_t a = arow[j];
                    sab = udot4(a, b, sab);
                    sbb = udot4(b, b, sbb);
                    lo = hi;
                }
            }
        }
        uint32_t ssd = saa + sbb - 2u * sab;
        int ad = (dx < 0 ? -dx : dx) + (dy < 0 ? -dy : dy);
        unsigned long long key = ((unsigned long long)ssd << 32) | ((unsigned long long)ad << 16) |
                                 ((unsigned long long)(dy + R) << 8) | (unsigned long long)(dx + R);
        best = key < best ? key : best;
    }
    best = wave_min_u64(best);
    if ((tid & 63) == 0) red[tid >> 6] = best;
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int i = 1; i < kSearchThreads / 64; ++i) best = red[i] < best ? red[i] : best;
        size_t o = (size_t)stream * gh * gw + blk_id;
        mv[2 * o + 0] = (int16_t)((int)(best & 0xff) - R);
        mv[2 * o + 1] = (int16_t)((int)((best >> 8) & 0xff) - R);
        best_ssd[o] = (uint32_t)(best >> 32);
    }
}

// ---- search on the matrix cores ----------------------------------------------------------
// SSD = sum a'^2 + sum b'^2 - 2 sum a'b' with a' = a - 128, b' = b - 128 (signed bytes; the offset
// cancels in a - b).  The cross term of all candidates of a block is one integer GEMM per window row
// wr:  X[dx][dy] += A_wr[dx][k] * B_wr[k][dy],  k = byte within the block row,
//   A_wr[dx][k] = window row wr, byte C*dx + k          (the block-wide run that candidate dx sees)
//   B_wr[k][dy] = block row wr - dy, byte k              (zero if that is not a row of the block)
// (dx, dy count from -R), so that the sum over the window rows is the cross term of candidate
// (dx, dy).  v_mfma_i32_16x16x64_i8 covers 16 dx x 16 dy x 64 bytes; NT x NT tiles cover the
// (2R+1)^2 candidates, KS K-steps the block row.  sum b'^2 per candidate is a box sum of per-pixel
// sums.  The wavefronts split the window rows and add their partial tiles pairwise through LDS.  The arg-min
// key is the same as in the scalar kernel, so both give identical results.
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
constexpr int kMfmaWaves = 4;           // wavefronts per block: they split the window rows and the summing loops
constexpr int kMfmaThreads = 64 * kMfmaWaves;

// BT, CT: block edge and channel count when known at compile time (the summing loops are then unrolled and
// their LDS reads issued together), 0: taken from the arguments.
template <bool ALIGNED, int NT, int KS, int BT, int CT>
__global__ __launch_bounds__(kMfmaThreads, 7) void match_mfma_kernel(
    const uint8_t* __restrict__ cur, const uint8_t* __restrict__ prev, int H, int W, int C_rt, int B_rt,
    int R, int gw, int gh, int ws, int k_skip, int16_t* __restrict__ mv, uint32_t* __restrict__ best_ssd) {
    const int B = BT ? BT : B_rt, C = CT ? CT : C_rt;
    extern __shared__ __align__(16) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // k-skip: the grid covers only the blocks on every k-th grid row and column
    const int lgw = (gw + k_skip - 1) / k_skip;
    const int bx = ((int)blockIdx.x % lgw) * k_skip, by = ((int)blockIdx.x / lgw) * k_skip;
    const int blk_id = by * gw + bx, stream = blockIdx.y;
    const int x0 = bx * B, y0 = by * B;
    const int rows = B + 2 * R, cols = rows, nd = 2 * R + 1;
    const int row_bytes = W * C;
    const size_t frame_bytes = (size_t)H * row_bytes;
    const uint8_t* pf = prev + (size_t)stream * frame_bytes;
    const uint8_t* cf = cur + (size_t)stream * frame_bytes;
    constexpr int BS = 64 * KS;                       // bytes of a staged block row
    // With the block shape known at compile time the row sums of squares are taken straight from the window bytes
    // and the per-pixel sums (p2) do not exist: one phase and 9 KB of LDS less (the kernel is bound by the latency of
    // its chain of phases, i.e. by how many workgroups a CU holds).
    constexpr bool kFused = BT > 0 && CT > 0 && CT <= 4 && (BT * CT) % 4 == 0;
    // LDS: [win rows*ws][blk B*BS][p2 rows*cols ints, unless kFused][h2 rows*nd ints][misc][v2 nd*nd ints]
    uint8_t* win = lds;
    uint8_t* blk = win + (size_t)rows * ws;
    int* p2 = reinterpret_cast<int*>(blk + (size_t)B * BS);
    const int n_p2 = kFused ? 0 : rows * cols;
    int* h2 = p2 + n_p2;
    int* misc = h2 + rows * nd + (4 - (n_p2 + rows * nd) % 4) % 4;   // 16-byte aligned
    // The summed tiles land at the start of LDS, over the window, the block and the sums, which are dead by then.
    int* tiles = reinterpret_cast<int*>(lds);
    unsigned long long* red = reinterpret_cast<unsigned long long*>(misc + kMfmaWaves);   // partial sums a'^2, then the arg-min keys
    int* v2 = misc + 3 * kMfmaWaves;

    const int gx0 = (x0 - R) * C;
    const int a0 = gx0 & ~3;
    const int skew = gx0 - a0;

    // ---- stage the window (signed bytes; out-of-frame bytes are never part of a valid candidate).  Only the
    // dwords that hold window bytes are fetched (the rest of a row is only read for candidates beyond the
    // search range); the loads of a thread are issued eight at a time before any of them is used ----
    // The block of the current frame is requested first and used after the window is in place, so that its load
    // travels together with the window's instead of after them (one memory latency less per block).  One dword per
    // thread; only when the block's rows are whole aligned dwords.
    const int blk_bytes = B * C;
    const bool blk_early = kFused && ALIGNED && BT * (BS / 4) <= kMfmaThreads && (reinterpret_cast<uintptr_t>(cf) & 3) == 0;
    uint32_t blk_raw = 0x80808080u;
    if (blk_early && tid < B * (BS / 4)) {
        const int r = tid / (BS / 4), j = tid - r * (BS / 4);
        if (4 * j < blk_bytes)
            blk_raw = *reinterpret_cast<const uint32_t*>(cf + (size_t)(y0 + r) * row_bytes + (size_t)x0 * C + 4 * j);
    }
    const int wdw = ws / 4;
    const int ldw = (skew + cols * C + 3) / 4;        // dwords per row that hold window bytes
    for (int base = 0; base < rows * ldw; base += 8 * kMfmaThreads) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * kMfmaThreads + tid;
            const int r = i / ldw, j = i - r * ldw;
            const int y = y0 - R + r;
            const int fb = a0 + 4 * j;
            v[u] = 0x80808080u;
            if (i < rows * ldw && y >= 0 && y < H) {
                const uint8_t* src = pf + (size_t)y * row_bytes;
                if (ALIGNED && fb >= 0 && fb + 3 < row_bytes) {
                    v[u] = *reinterpret_cast<const uint32_t*>(src + fb);
                } else {
                    uint32_t t = 0;
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const int f = fb + b;
                        t |= (uint32_t)((f >= 0 && f < row_bytes) ? src[f] : 128) << (8 * b);
                    }
                    v[u] = t;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * kMfmaThreads + tid;
            const int r = i / ldw, j = i - r * ldw;
            if (i < rows * ldw) reinterpret_cast<uint32_t*>(win)[r * wdw + j] = v[u] ^ 0x80808080u;
        }
    }
    for (int i = tid; i < rows * (wdw - ldw); i += kMfmaThreads) {   // the tail of every row: any defined value
        const int r = i / (wdw - ldw), j = ldw + (i - r * (wdw - ldw));
        reinterpret_cast<uint32_t*>(win)[r * wdw + j] = 0;
    }
    // ---- stage the block: signed bytes, true zeros behind the row so that the padding adds nothing ----
    int saa = 0;
    if (blk_early) {
        if (tid < B * (BS / 4)) {       // a dword outside the row arrives as 0x80808080: zeros once the offset is taken off
            const uint32_t v = blk_raw ^ 0x80808080u;
            saa = __builtin_amdgcn_sdot4((int)v, (int)v, 0, false);
            reinterpret_cast<uint32_t*>(blk)[tid] = v;
        }
    } else {
        for (int i = tid; i < B * (BS / 4); i += kMfmaThreads) {
            const int r = i / (BS / 4), j = i - r * (BS / 4);
            const uint8_t* src = cf + (size_t)(y0 + r) * row_bytes + (size_t)x0 * C;
            uint32_t v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int f = 4 * j + b;
                if (f < blk_bytes) {
                    const int a = (int)src[f] - 128;
                    saa += a * a;
                    v |= (uint32_t)(a & 0xff) << (8 * b);
                }
            }
            reinterpret_cast<uint32_t*>(blk)[i] = v;
        }
    }
    saa = wave_sum_i32(saa);
    __syncthreads();
    if (lane == 0) misc[wave] = saa;

    // ---- box sums of squares over the block: B columns (h2), then B rows (v2) ----
    if constexpr (kFused) {
        // h2[r][d] = sum of squares of the BT * CT window bytes of row r that candidate d sees.  A thread takes four
        // neighbouring d: it aligns the bytes it needs once, sums the first run with byte dot products and slides it
        // three times by one pixel (CT bytes enter, CT leave).
        constexpr int NB = BT * CT;                                 // bytes of a block row
        constexpr int NA = (NB + 3 * CT + 3) / 4;                   // aligned dwords that hold NB + 3 CT bytes
        constexpr uint32_t kPix = CT == 4 ? 0xffffffffu : (1u << (8 * CT)) - 1u;
        const int ng = (nd + 3) / 4;
        for (int i = tid; i < rows * ng; i += kMfmaThreads) {
            const int r = i / ng, d0 = 4 * (i - r * ng);
            const int o0 = skew + CT * d0;
            const uint32_t* w32 = reinterpret_cast<const uint32_t*>(win + (size_t)r * ws) + (o0 >> 2);
            const int sh = o0 & 3;
            uint32_t raw[NA + 1], al[NA + 1];
#pragma unroll
            for (int k = 0; k <= NA; ++k) raw[k] = w32[k];
#pragma unroll
            for (int k = 0; k < NA; ++k) al[k] = __builtin_amdgcn_alignbyte(raw[k + 1], raw[k], sh);
            al[NA] = 0;
            int sq = 0;
#pragma unroll
            for (int k = 0; k < NB / 4; ++k) sq = __builtin_amdgcn_sdot4((int)al[k], (int)al[k], sq, false);
            h2[r * nd + d0] = sq;
#pragma unroll
            for (int q = 1; q < 4; ++q) {
                const int tin = NB + CT * (q - 1), tout = CT * (q - 1);       // first byte entering / leaving
                const uint32_t vin = __builtin_amdgcn_alignbyte(al[tin / 4 + 1], al[tin / 4], tin % 4) & kPix;
                const uint32_t vout = __builtin_amdgcn_alignbyte(al[tout / 4 + 1], al[tout / 4], tout % 4) & kPix;
                sq += __builtin_amdgcn_sdot4((int)vin, (int)vin, 0, false) - __builtin_amdgcn_sdot4((int)vout, (int)vout, 0, false);
                if (d0 + q < nd) h2[r * nd + d0 + q] = sq;
            }
        }
    } else {
        const int8_t* swin = reinterpret_cast<const int8_t*>(win);
        for (int i = tid; i < rows * cols; i += kMfmaThreads) {
            const int r = i / cols, x = i - r * cols;
            const int8_t* px = swin + (size_t)r * ws + skew + x * C;
            int s = 0;
#pragma unroll
            for (int c = 0; c < C; ++c) s += (int)px[c] * (int)px[c];
            p2[i] = s;
        }
        __syncthreads();
        for (int i = tid; i < rows * nd; i += kMfmaThreads) {
            const int r = i / nd, d = i - r * nd;
            int s = 0;
#pragma unroll
            for (int x = 0; x < B; ++x) s += p2[r * cols + d + x];
            h2[i] = s;
        }
    }
    __syncthreads();
    if constexpr (BT > 0) {
        // a thread takes eight candidates dy of one dx: the first sum over its B rows, then seven steps down the column
        // (one row enters, one leaves): 2 B - 2 + 16 reads for eight sums instead of 8 B
        const int nch = (nd + 7) / 8;
        for (int i = tid; i < nd * nch; i += kMfmaThreads) {
            const int ch = i / nd, dxi = i - ch * nd, dy0 = 8 * ch;
            int s = 0;
#pragma unroll
            for (int r = 0; r < BT; ++r) s += h2[(dy0 + r) * nd + dxi];
            v2[dy0 * nd + dxi] = s;
#pragma unroll
            for (int q = 1; q < 8; ++q) {
                if (dy0 + q >= nd) break;
                s += h2[(dy0 + q + BT - 1) * nd + dxi] - h2[(dy0 + q - 1) * nd + dxi];
                v2[(dy0 + q) * nd + dxi] = s;
            }
        }
    } else {
        for (int i = tid; i < nd * nd; i += kMfmaThreads) {
            const int dyi = i / nd, dxi = i - dyi * nd;
            int s = 0;
            for (int r = 0; r < B; ++r) s += h2[(dyi + r) * nd + dxi];
            v2[i] = s;
        }
    }

    // ---- cross terms: this wavefront's share of the window rows ----
    const int n = lane & 15, kq = lane >> 4;
    intx4 acc[NT][NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = intx4{0, 0, 0, 0};
    // Window row wr meets block rows only for the candidates dy with 0 <= wr - dy < B: a tile of 16 dy whose
    // block rows all fall outside is a product with zeros and is skipped (about half of the tiles).  The rows are
    // dealt round-robin so that every wavefront gets its share of the rows with one and with two live tiles.
    for (int wr = wave; wr < rows; wr += kMfmaWaves) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            intx4 af[NT], bf[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) {      // lane: candidate dx = 16 i + n, bytes [16 kq, 16 kq + 16) of its run
                const int o = skew + C * (16 * i + n) + 16 * kq + 64 * ks;
                const uint32_t* w32 = reinterpret_cast<const uint32_t*>(win + (size_t)wr * ws) + (o >> 2);
                const int sh = o & 3;
                uint32_t wv[5];
#pragma unroll
                for (int e = 0; e < 5; ++e) wv[e] = w32[e];
#pragma unroll
                for (int e = 0; e < 4; ++e) af[i][e] = (int)__builtin_amdgcn_alignbyte(wv[e + 1], wv[e], sh);
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) {      // lane: candidate dy = 16 j + n, block row wr - dy
                const bool live = wr >= 16 * j && wr - 16 * j < B + 15;   // wavefront-uniform: some dy of the tile has a block row
                if (!live) continue;
                const int r = wr - (16 * j + n);
                const bool ok = r >= 0 && r < B;
                const intx4 v = *reinterpret_cast<const intx4*>(blk + (size_t)(ok ? r : 0) * BS + 64 * ks + 16 * kq);
                bf[j] = ok ? v : intx4{0, 0, 0, 0};
#pragma unroll
                for (int i = 0; i < NT; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[i], bf[j], acc[i][j], 0, 0, 0);
            }
        }
    }
    // The four partial copies are added through one LDS buffer with plain 16-byte accesses (integer atomics, 36 per
    // lane, cost more): wavefront 3 stores its tiles, 2 adds them to its own and stores the sum, then 1, then 0, whose
    // sum the evaluation below reads.  A lane only ever touches its own slots, so a wavefront's reads and writes need
    // no barrier between them.  The buffer lies over the window, which is dead after the barrier (the launcher checks
    // that NT^2 KiB fit into what is dead by then).
    {
        intx4* buf = reinterpret_cast<intx4*>(tiles);
        __syncthreads();                       // every wavefront is done with the window, the block and the sums
#pragma unroll
        for (int w = kMfmaWaves - 1; w >= 0; --w) {
            if (wave == w) {
#pragma unroll
                for (int i = 0; i < NT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) {
                        if (w < kMfmaWaves - 1) acc[i][j] += buf[(i * NT + j) * 64 + lane];
                        buf[(i * NT + j) * 64 + lane] = acc[i][j];
                    }
            }
            __syncthreads();
        }
    }

    // ---- SSD and arg-min: tile t is evaluated by wavefront t % kMfmaWaves; lane (n, kq) holds rows
    // dx = 16 i + 4 kq + e of column dy = 16 j + n ----
    int saa_all = 0;
#pragma unroll
    for (int w = 0; w < kMfmaWaves; ++w) saa_all += misc[w];
    unsigned long long best = ~0ull;
    for (int t = wave; t < NT * NT; t += kMfmaWaves) {
        const int i = t / NT, j = t - i * NT;
        const intx4 c = *reinterpret_cast<const intx4*>(tiles + (t * 64 + lane) * 4);
        const int dyi = 16 * j + n;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int dxi = 16 * i + 4 * kq + e;
            const int dx = dxi - R, dy = dyi - R;
            if (dxi >= nd || dyi >= nd || x0 + dx < 0 || y0 + dy < 0 || x0 + dx + B > W || y0 + dy + B > H) continue;
            const uint32_t ssd = (uint32_t)(saa_all + v2[dyi * nd + dxi] - 2 * c[e]);
            const int ad = (dx < 0 ? -dx : dx) + (dy < 0 ? -dy : dy);
            const unsigned long long key = ((unsigned long long)ssd << 32) | ((unsigned long long)ad << 16) |
                                           ((unsigned long long)dyi << 8) | (unsigned long long)dxi;
            best = key < best ? key : best;
        }
    }
    best = wave_min_u64(best);
    if (lane == 0) red[wave] = best;
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < kMfmaWaves; ++w) best = red[w] < best ? red[w] : best;
        const size_t o = (size_t)stream * gh * gw + blk_id;
        mv[2 * o + 0] = (int16_t)((int)(best & 0xff) - R);
        mv[2 * o + 1] = (int16_t)((int)((best >> 8) & 0xff) - R);
        best_ssd[o] = (uint32_t)(best >> 32);
    }
}

// ---- the usual search (3 channels, range = block edge) on the matrix cores -------------------------------
// The same sums as match_mfma_kernel with the operands the other way round, for blocks of BT = 8 or 16 pixels, C = 3
// and R = BT.  What bounded that kernel was the vector ALU (1600 instructions per wavefront and block: every operand
// fragment assembled from unaligned dwords, divisions and byte loads in the staging, five of nine 16 x 16 tiles for the
// one candidate that 2 BT + 1 has more than 2 BT).  Here:
//   * the cross terms of the 2 BT x 2 BT candidates below the last row and column are, per block row r,
//       X[dy][dx] += W[dy + r][k] * T_r[k][dx],   T_r[k][dx] = block row r, byte k - 3 dx (zero outside the row),
//     so the window operand is read as it lies (16-byte reads, no arithmetic) and the shifted one is a fragment of the
//     block: it depends on dx mod 16 only, so two fragments per block row serve all tiles.  A wavefront takes BT / 4
//     block rows of every tile; the partial tiles are added through LDS.
//   * the last row of candidates (dy = R): with dx = 4 m + b, S[m][b] += V_r[m][k] * T_r[k][b], V_r[m][k] = window row
//     2 BT + r, byte 12 m + k: one product per block row with the fragment that is there already.
//   * the last column (dx = R): Z[wr][r] = sum_k W[wr][6 BT + k] * block[r][k] for all window and block rows (three
//     products), then sums along the diagonals wr - r = dy.
//   * every 16 bytes of the window are one load, unaligned where the frame's rows are (only 16 bytes that straddle
//     an end of the frame are fetched byte by byte; bytes outside the frame's rows are part of no valid candidate).
// Window rows are 160 (96) bytes apart: an odd multiple of 32, for which the 16-byte reads of 16 rows have no bank conflicts
// (176: a third of all LDS cycles).  16x16 blocks, 416x416, 16 streams: 115 us with match_mfma_kernel (whose vector ALU was
// busy throughout), 43 with this: about 2500 cycles of a CU per block, 2000 of them with LDS active, half of those for the
// window operand, and 1850 of vector instructions on each SIMD.
template <int BT>
struct WindowShape {
    static constexpr int C = 3, R = BT, ROWS = 3 * BT, ND = 2 * BT + 1, NB = C * BT;      // NB: bytes of a block row
    static constexpr int NT = 2 * BT / 16;                   // tiles of 16 candidates per direction
    static constexpr int WS = BT == 16 ? 160 : 96;           // window row in LDS (a read that runs into the next row meets zeros of T)
    static constexpr int BS = 192, BO = 48;                  // block row in LDS: zeros, the row from byte BO, zeros (T_r reaches 45 bytes to the left)
    static constexpr int CW = (C * ROWS + 15) / 16;          // 16-byte pieces of a window row
    static constexpr int CB = BT == 16 ? 16 : 8;             // bytes per load of the block (a row is a whole number of them)
    static constexpr int ZS = 18;
    static constexpr int kWin = 0, kBlk = kWin + ROWS * WS, kH2 = kBlk + BT * BS, kH2End = (kH2 + ROWS * ND * 4 + 15) / 16 * 16,
                         kSums = (kMfmaWaves - 1) * (NT * NT + 1) * 1024,             // partial tiles, over what is dead by then
                         kV2 = kH2End > kSums ? kH2End : kSums, kZ = kV2 + (ND * ND * 4 + 15) / 16 * 16, kMisc = kZ + (ROWS + 15) / 16 * 16 * ZS * 4,
                         kBytes = kMisc + 64;
    static_assert(WS >= 16 * CW, "window row");
};

// 16 bytes of a frame from byte `at` on; bytes in front of the frame or behind it read as zero (a frame has 16 bytes at least)
__device__ __forceinline__ uintx4 load16_within(const uint8_t* frame, int at, int bytes) {
    const int in = at < 0 ? 0 : (at > bytes - 16 ? bytes - 16 : at);
    uintx4 v;
    __builtin_memcpy(&v, frame + (uint32_t)in, 16);
    if (in != at) {
        unsigned __int128 w;
        __builtin_memcpy(&w, &v, 16);
        const int d = at - in;
        w = d <= -16 || d >= 16 ? 0 : (d < 0 ? w << (-8 * d) : w >> (8 * d));
        __builtin_memcpy(&v, &w, 16);
    }
    return v;
}

// Smallest value over the 64 lanes (moves as in wave_sum_i32; a lane without a source keeps its own).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_min(uint32_t v) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, CTRL, ROW_MASK, 0xf, false);
    return o < v ? o : v;
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
    v = dpp_min<0xb1, 0xf>(v);
    v = dpp_min<0x4e, 0xf>(v);
    v = dpp_min<0x114, 0xf>(v);
    v = dpp_min<0x118, 0xf>(v);
    v = dpp_min<0x142, 0xa>(v);
    v = dpp_min<0x143, 0xc>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

template <int BT>
__global__ __launch_bounds__(kMfmaThreads, 6) void match_window_kernel(
    const uint8_t* __restrict__ cur, const uint8_t* __restrict__ prev, int H, int W, int gw, int gh, int k_skip,
    int16_t* __restrict__ mv, uint32_t* __restrict__ best_ssd) {
    typedef WindowShape<BT> S;
    constexpr int R = S::R, ROWS = S::ROWS, ND = S::ND, NB = S::NB, NT = S::NT, WS = S::WS, BS = S::BS, BO = S::BO;
    __shared__ __align__(16) uint8_t lds[S::kBytes];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bx = (int)blockIdx.x * k_skip, by = (int)blockIdx.y * k_skip;      // the searched blocks
    const int blk_id = by * gw + bx, stream = blockIdx.z;
    const int x0 = bx * BT, y0 = by * BT;
    const int row_bytes = W * 3, frame_bytes = H * row_bytes;
    const uint8_t* const pf = prev + (size_t)stream * (uint32_t)frame_bytes;
    const uint8_t* const cf = cur + (size_t)stream * (uint32_t)frame_bytes;
    int* const h2 = reinterpret_cast<int*>(lds + S::kH2);
    int* const v2 = reinterpret_cast<int*>(lds + S::kV2);
    int* const z = reinterpret_cast<int*>(lds + S::kZ);
    int* const misc = reinterpret_cast<int*>(lds + S::kMisc);        // per wavefront: sum a'^2, then {key, vector} of its best
    uint8_t* const win = lds + S::kWin;
    uint8_t* const blk = lds + S::kBlk;

    // ---- stage window and block as signed bytes; all loads of a thread are on their way before the first is used ----
    constexpr int CW = S::CW, NWIN = ROWS * CW, WI = (NWIN + kMfmaThreads - 1) / kMfmaThreads;
    constexpr int CB = S::CB, PB = BS / CB;
    static_assert(BT * PB <= kMfmaThreads, "one piece of the block per thread");
    uintx4 wv[WI], bv = {0, 0, 0, 0};
    const int br = tid / PB, bc = tid - br * PB - BO / CB;           // block row and piece; outside [0, NB / CB): zeros
    const bool in_blk = br < BT, has_blk = in_blk && bc >= 0 && bc < NB / CB;
    if (has_blk) __builtin_memcpy(&bv, cf + (uint32_t)((y0 + br) * row_bytes + x0 * 3 + bc * CB), CB);
#pragma unroll
    for (int u = 0; u < WI; ++u) {                                   // (rows above and below the frame: any row's bytes)
        const int i = u * kMfmaThreads + tid, r = i / CW, j = i - r * CW;
        int y = y0 - R + (r < ROWS ? r : ROWS - 1);
        y = y < 0 ? 0 : (y < H ? y : H - 1);
        wv[u] = load16_within(pf, y * row_bytes + (x0 - R) * 3 + 16 * j, frame_bytes);
    }
#pragma unroll
    for (int e = 0; e < CB / 4; ++e) bv[e] = has_blk ? bv[e] ^ 0x80808080u : 0;
    int saa = 0;
#pragma unroll
    for (int e = 0; e < CB / 4; ++e) saa = __builtin_amdgcn_sdot4((int)bv[e], (int)bv[e], saa, false);
    if (in_blk) {
        if constexpr (CB == 16) *reinterpret_cast<uintx4*>(blk + tid * CB) = bv;
        else *reinterpret_cast<uint2*>(blk + tid * CB) = uint2{bv[0], bv[1]};
    }
#pragma unroll
    for (int u = 0; u < WI; ++u) {
        const int i = u * kMfmaThreads + tid, r = i / CW, j = i - r * CW;
        if (i < NWIN) *reinterpret_cast<uintx4*>(win + r * WS + 16 * j) = wv[u] ^ 0x80808080u;
    }
    saa = wave_sum_i32(saa);
    if (lane == 0) misc[wave] = saa;
    __syncthreads();

    // ---- h2[r][d]: sum of squares of the NB bytes of window row r that candidate dx = d sees; D neighbouring d per
    // thread (the run of the first summed, then moved on by a pixel at a time) ----
    {
        constexpr int D = 8, NG = (ND + D - 1) / D, NA = (NB + 3 * (D - 1) + 3) / 4;
        static_assert(ROWS * NG <= kMfmaThreads, "one run per thread");
        if (tid < ROWS * NG) {
            const int r = tid / NG, g = tid - r * NG;
            const uint2* const w64 = reinterpret_cast<const uint2*>(win + r * WS) + 3 * D / 8 * g;
            uint32_t al[NA + 2];
#pragma unroll
            for (int k = 0; k < NA; k += 2) { const uint2 v = w64[k / 2]; al[k] = v.x; al[k + 1] = v.y; }
            if (NA % 2 == 0) al[NA] = 0;
            int sq = 0;
#pragma unroll
            for (int k = 0; k < NB / 4; ++k) sq = __builtin_amdgcn_sdot4((int)al[k], (int)al[k], sq, false);
            int* const h = h2 + r * ND + D * g;
            h[0] = sq;
#pragma unroll
            for (int q = 1; q < D; ++q) {
                const int tin = NB + 3 * (q - 1), tout = 3 * (q - 1);       // first byte entering / leaving
                const uint32_t vin = __builtin_amdgcn_alignbyte(al[tin / 4 + 1], al[tin / 4], tin % 4) & 0xffffffu;
                const uint32_t vout = __builtin_amdgcn_alignbyte(al[tout / 4 + 1], al[tout / 4], tout % 4) & 0xffffffu;
                sq = __builtin_amdgcn_sdot4((int)vin, (int)vin, sq, false) - __builtin_amdgcn_sdot4((int)vout, (int)vout, 0, false);
                if (D * g + q < ND) h[q] = sq;
            }
        }
    }
    __syncthreads();
    // ---- v2[dy][dx] = sum of h2 over BT rows: five candidates dy of one dx per thread, one row entering and one leaving ----
    {
        constexpr int U = 5, NCH = (ND + U - 1) / U;
        static_assert(ND * NCH <= kMfmaThreads, "one run per thread");
        if (tid < ND * NCH) {
            const int ch = tid / ND, dxi = tid - ch * ND, dy0 = U * ch;
            const int* const h = h2 + dy0 * ND + dxi;
            int s = 0;
#pragma unroll
            for (int r = 0; r < BT; ++r) s += h[r * ND];
            v2[dy0 * ND + dxi] = s;
#pragma unroll
            for (int q = 1; q < U; ++q) {
                if (dy0 + q >= ND) break;
                s += h[(q + BT - 1) * ND] - h[(q - 1) * ND];
                v2[(dy0 + q) * ND + dxi] = s;
            }
        }
    }

    // ---- cross terms ----
    const int n = lane & 15, kq = lane >> 4;
    intx4 acc[NT][NT], last_row = {0, 0, 0, 0};            // acc[j][i]: lane holds dy = 16 j + 4 kq + e, dx = 16 i + n
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[j][i] = intx4{0, 0, 0, 0};
    // K steps: bytes 0 .. 63 of a block row's band, and bytes 64 .. 95 (the band has 3 * 15 + NB <= 93) of two block rows
    // together, the second row in the K groups 2 and 3.
    const int to = BO + 16 * kq - 3 * n, tsh = to & 3, odd = kq >> 1;
    const uint32_t* const tsrc = reinterpret_cast<const uint32_t*>(blk) + (to >> 2);
    const uint32_t* const tsrc2 = tsrc + odd * (BS / 4) + 16 - 8 * odd;
    const uint8_t* const wsrc = win + n * WS + 16 * kq;
    const uint8_t* const wsrc2 = wsrc + odd * WS + 64 - 32 * odd;
    const uint32_t* const lsrc = reinterpret_cast<const uint32_t*>(win + 2 * BT * WS + 12 * (n < BT / 2 ? n : BT / 2) + 16 * kq);
    auto shifted = [&](const uint32_t* src) {          // 16 bytes from byte tsh on
        uint32_t raw[5];
        intx4 t;
#pragma unroll
        for (int e = 0; e < 5; ++e) raw[e] = src[e];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = (int)__builtin_amdgcn_alignbyte(raw[e + 1], raw[e], tsh);
        return t;
    };
    static_assert(BT / kMfmaWaves % 2 == 0 && 3 * 15 + NB <= 96, "block rows in pairs");
#pragma unroll
    for (int rr = 0; rr < BT / kMfmaWaves; rr += 2) {
        const int r = wave * (BT / kMfmaWaves) + rr;
        const intx4 t[3] = {shifted(tsrc + r * (BS / 4)), shifted(tsrc + (r + 1) * (BS / 4)), shifted(tsrc2 + r * (BS / 4))};
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    const uint8_t* const src = k < 2 ? wsrc + (16 * j + r + k) * WS : wsrc2 + (16 * j + r) * WS;
                    const intx4 a = *reinterpret_cast<const intx4*>(src + 48 * i);
                    acc[j][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, t[k], acc[j][i], 0, 0, 0);
                }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            intx4 a;
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = (int)lsrc[(r + k) * (WS / 4) + e];
            last_row = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, t[k], last_row, 0, 0, 0);
        }
    }
    if (wave < (ROWS + 15) / 16) {
        const intx4 a = *reinterpret_cast<const intx4*>(wsrc + 16 * wave * WS + 2 * NB);
        const intx4 b = *reinterpret_cast<const intx4*>(blk + (n & (BT - 1)) * BS + BO + 16 * kq);
        const intx4 c = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, intx4{0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) z[(16 * wave + 4 * kq + e) * S::ZS + n] = c[e];
    }
    // Partial tiles, over the window, the block and h2: tile t is summed by wavefront t, the last row by the last one.
    intx4* const buf = reinterpret_cast<intx4*>(lds) + lane;
    constexpr int NTT = NT * NT, LAST = kMfmaWaves - 1;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NTT; ++t)
        if (wave != t) buf[(t * LAST + (wave < t ? wave : wave - 1)) * 64] = acc[t / NT][t % NT];
    if (wave != LAST) buf[(NTT * LAST + wave) * 64] = last_row;
    __syncthreads();

    int saa_all = 0;
#pragma unroll
    for (int w = 0; w < kMfmaWaves; ++w) saa_all += misc[w];
    // The best candidate by (ssd, |dx| + |dy|, dy, dx): the first two in one word (ssd <= 768 * 255^2 < 2^26), the vector
    // in another.
    uint32_t best = ~0u, vec = ~0u;
    const int dx_lo = R - x0, dx_n = W - BT, dy_lo = R - y0, dy_n = H - BT;        // candidates inside the frame: d_lo .. d_lo + d_n
    auto distance = [](uint32_t d) { return d < (uint32_t)R ? (uint32_t)R - d : d - (uint32_t)R; };
    // up to four candidates of a lane: (dy, dx) and step_dy, step_dx further each, in the order of their vectors
    auto consider = [&](bool on, uint32_t dyi, uint32_t dxi, uint32_t step_dy, uint32_t step_dx, int count, const intx4& cross) {
        uint32_t b = ~0u, c = 0;
        const int* const sq = v2 + dyi * ND + dxi;
#pragma unroll
        for (int e = 0; e < count; ++e) {
            const uint32_t y = dyi + e * step_dy, x = dxi + e * step_dx;
            const bool ok = on && (step_dx == 0 || x < ND) && y - (uint32_t)dy_lo <= (uint32_t)dy_n && x - (uint32_t)dx_lo <= (uint32_t)dx_n;
            uint32_t key = ((uint32_t)(saa_all + (ok ? sq[e * (step_dy * ND + step_dx)] : 0)) << 6) + distance(y) + distance(x) - ((uint32_t)cross[e] << 7);
            key = ok ? key : ~0u;
            if (key < b) { b = key; c = y << 8 | x; }
        }
        if (b < best || (b == best && c < vec)) { best = b; vec = c; }
    };
#pragma unroll
    for (int t = 0; t < NTT; ++t)
        if (wave == t) {
            intx4 c = acc[t / NT][t % NT];
#pragma unroll
            for (int w = 0; w < LAST; ++w) c += buf[(t * LAST + w) * 64];
            consider(true, 16 * (t / NT) + 4 * kq, 16 * (t % NT) + n, 1, 0, 4, c);
        }
    if (wave == LAST) {
        intx4 c = last_row;
#pragma unroll
        for (int w = 0; w < LAST; ++w) c += buf[(NTT * LAST + w) * 64];
        consider(n < 4, 2 * BT, 16 * kq + n, 0, 4, 4, c);
    }
    if (wave == LAST - 1) {
        const int d = lane < ND ? lane : 0;
        int c = 0;
#pragma unroll
        for (int r = 0; r < BT; ++r) c += z[(d + r) * S::ZS + r];
        consider(lane < ND, d, 2 * BT, 0, 0, 1, intx4{c, 0, 0, 0});
    }
    const uint32_t wbest = wave_min_u32(best);
    const uint32_t wvec = wave_min_u32(best == wbest ? vec : ~0u);
    if (lane == 0) { misc[4 + 2 * wave] = (int)wbest; misc[5 + 2 * wave] = (int)wvec; }
    __syncthreads();
    if (tid == 0) {
        uint32_t key = (uint32_t)misc[4], code = (uint32_t)misc[5];
#pragma unroll
        for (int w = 1; w < kMfmaWaves; ++w) {
            const uint32_t k2 = (uint32_t)misc[4 + 2 * w], c2 = (uint32_t)misc[5 + 2 * w];
            if (k2 < key || (k2 == key && c2 < code)) { key = k2; code = c2; }
        }
        const size_t o = (size_t)stream * gh * gw + blk_id;
        mv[2 * o + 0] = (int16_t)((int)(code & 0xff) - R);
        mv[2 * o + 1] = (int16_t)((int)(code >> 8) - R);
        best_ssd[o] = key >> 6;
    }
}

__device__ __forceinline__ int round_half_away(int num, int den) {
    int mag = num < 0 ? -num : num;
    int q = (2 * mag + den) / (2 * den);
    return num < 0 ? -q : q;
}

// Step 3 (redundantly per workgroup), then Step 4: one wavefront per block, four blocks per workgroup.  What bounded it was
// instructions: a mean over all vectors of the stream per block, and a byte of the block at a time with a division each.  Now four
// blocks share a mean, its reads are dealt to 256 threads, and the samples are compared E = 4 bytes at a time where a block row is a
// whole number of them (unaligned loads: the moved block starts at any byte; a sample never leaves its block row); the
// current block's samples are on their way before the mean is known.  416x416 in 16x16 blocks, 16 streams: 22.0 -> 8.9 us.
constexpr int kRetestWaves = 4;
template <int E>
__global__ __launch_bounds__(kRetestWaves * 64) void motion_retest_kernel(
    const uint8_t* __restrict__ cur, const uint8_t* __restrict__ prev, int H, int W, int C, int B,
    int gw, int gh, uint32_t max_ssd, int16_t* mv, uint32_t* best_ssd, int32_t* __restrict__ gmv,
    int32_t* __restrict__ n_pass, uint8_t* __restrict__ mask, int k_skip, uint32_t row_magic) {
    constexpr int U = 4;                                 // independent loads per lane at a time
    __shared__ int part[kRetestWaves][3];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int stream = blockIdx.y;
    const int nb = gh * gw;
    const int blk_id = (int)blockIdx.x * kRetestWaves + wave;
    const bool real = blk_id < nb;                       // (uniform over the wavefront)
    const int by = real ? blk_id / gw : 0, bx = real ? blk_id - by * gw : 0;
    const int x0 = bx * B, y0 = by * B;
    const size_t frame_bytes = (size_t)H * W * C, pitch = (size_t)W * C;
    const uint8_t* const cb = cur + stream * frame_bytes + y0 * pitch + (size_t)x0 * C;
    const int per_row = B * C / E, n_elem = B * per_row; // samples of E bytes
    // place of sample i from the block's first byte; past the end: the first sample
    auto place = [&](int i) {
        if (i >= n_elem) i = 0;
        uint32_t r = row_magic ? __umulhi((uint32_t)i, row_magic) : (uint32_t)i;      // (0: one sample a row)
        if (r * (uint32_t)per_row > (uint32_t)i) --r;    // the product is one too large at most
        return r * pitch + (size_t)((uint32_t)i - r * (uint32_t)per_row) * E;
    };
    auto load = [](const uint8_t* p) {
        if constexpr (E == 4) {
            uint32_t v;
            __builtin_memcpy(&v, p, 4);
            return v;
        } else {
            return (uint32_t)*p;
        }
    };
    uint32_t first[U];
#pragma unroll
    for (int u = 0; u < U; ++u) first[u] = load(cb + place(u * 64 + lane));

    int16_t* smv = mv + (size_t)stream * nb * 2;
    uint32_t* sbest = best_ssd + (size_t)stream * nb;
    int sx = 0, sy = 0, K = 0;
    for (int base = 0; base < nb; base += U * kRetestWaves * 64) {
        uint32_t bs[U];
        int vx[U], vy[U];
        bool has[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * (kRetestWaves * 64) + tid;
            // with k-skip only the blocks on every k-th grid row and column carry a vector; the entries of the others
            // are written further down by their own workgroups and are not read here
            const bool in = i < nb && (k_skip == 1 || ((i / gw) % k_skip == 0 && (i % gw) % k_skip == 0));
            has[u] = in;
            bs[u] = in ? sbest[i] : 0xffffffffu;
            vx[u] = in ? smv[2 * i] : 0;
            vy[u] = in ? smv[2 * i + 1] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool pass = has[u] && bs[u] <= max_ssd;
            sx += pass ? vx[u] : 0;
            sy += pass ? vy[u] : 0;
            K += pass ? 1 : 0;
        }
    }
    sx = wave_sum_i32(sx);
    sy = wave_sum_i32(sy);
    K = wave_sum_i32(K);
    if (lane == 0) { part[wave][0] = sx; part[wave][1] = sy; part[wave][2] = K; }
    __syncthreads();
    if (!real) return;
    sx = sy = K = 0;
#pragma unroll
    for (int w = 0; w < kRetestWaves; ++w) { sx += part[w][0]; sy += part[w][1]; K += part[w][2]; }
    sx = __builtin_amdgcn_readfirstlane(sx);
    sy = __builtin_amdgcn_readfirstlane(sy);
    K = __builtin_amdgcn_readfirstlane(K);
    int mx = 0, my = 0;
    if (K > 0) {
        mx = round_half_away(sx, K);
        my = round_half_away(sy, K);
    }
    if (blk_id == 0 && lane == 0) {
        gmv[2 * stream] = mx;
        gmv[2 * stream + 1] = my;
        n_pass[stream] = K;
    }
    if (k_skip > 1 && (bx % k_skip != 0 || by % k_skip != 0) && lane == 0) {
        // not searched: no vector (no workgroup reads these entries: the mean above leaves them out)
        smv[2 * blk_id] = 0; smv[2 * blk_id + 1] = 0;
        sbest[blk_id] = 0xffffffffu;
    }
    bool inside = K > 0 && x0 + mx >= 0 && y0 + my >= 0 && x0 + mx + B <= W && y0 + my + B <= H;
    uint32_t ssd = 0;
    if (inside) {
        const uint8_t* const pb = prev + stream * frame_bytes + (size_t)(y0 + my) * pitch + (size_t)(x0 + mx) * C;
        for (int base = 0; base < n_elem; base += U * 64) {
            uint32_t a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t at = place(base + u * 64 + lane);
                b[u] = load(pb + at);
                a[u] = base == 0 ? first[u] : load(cb + at);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (base + u * 64 + lane >= n_elem) a[u] = b[u] = 0;
                if constexpr (E == 4) {      // sum (a - b)^2, modulo 2^32
                    ssd = udot4(a[u], a[u], udot4(b[u], b[u], ssd)) - 2u * udot4(a[u], b[u], 0u);
                } else {
                    const int d = (int)a[u] - (int)b[u];
                    ssd += (uint32_t)(d * d);
                }
            }
        }
        ssd = (uint32_t)wave_sum_i32((int)ssd);
    }
    if (lane == 0) mask[(size_t)stream * nb + blk_id] = (inside && ssd <= max_ssd) ? 1 : 0;
}
// Both searches end here.
hipError_t launch_motion_retest(const uint8_t* cur, const uint8_t* prev, int n_streams, int H, int W, int C, int B, int gw, int gh,
                                uint32_t max_ssd, int16_t* mv, uint32_t* best_ssd, int32_t* gmv, int32_t* n_pass, uint8_t* mask,
                                int k_skip, hipStream_t st) {
    const bool words = (B * C) % 4 == 0;
    const uint64_t per_row = (uint64_t)(words ? B * C / 4 : B * C);
    const uint32_t magic = (uint32_t)((0x100000000ull + per_row - 1) / per_row);      // 2^32 (one sample a row) becomes 0
    const dim3 grid((unsigned)((gh * gw + kRetestWaves - 1) / kRetestWaves), (unsigned)n_streams);
    if (words)
        hipLaunchKernelGGL(motion_retest_kernel<4>, grid, dim3(kRetestWaves * 64), 0, st, cur, prev, H, W, C, B, gw, gh, max_ssd, mv,
                           best_ssd, gmv, n_pass, mask, k_skip, magic);
    else
        hipLaunchKernelGGL(motion_retest_kernel<1>, grid, dim3(kRetestWaves * 64), 0, st, cur, prev, H, W, C, B, gw, gh, max_ssd, mv,
                           best_ssd, gmv, n_pass, mask, k_skip, magic);
    return hipGetLastError();
}

// ---- diamond search (Section 4, Step 2 as the paper runs it) with k-skip ----------------------
// One wavefront per block of the grid.  The walk is sequential, so what counts is the latency of a round:
// the wavefront first copies its search window of the previous frame ((B+2R)^2 pixels) and its block into
// LDS (one pass of independent loads), then every round reads LDS only.  The lanes share the block's
// samples (sample i goes to lane i % 64), the eight new points of the large pattern are evaluated
// together, and every decision is taken on wavefront-uniform values.  Windows too large for LDS are read
// from memory instead (WIN = false).
//   large pattern: centre, (0,-2), (-1,-1), (1,-1), (-2,0), (2,0), (-1,1), (1,1), (0,2)
//   small pattern: centre, (0,-1), (-1,0), (1,0), (0,1)
// The best point of a pattern is the valid one with the smallest (cost, position in the list above); the
// centre is position 0, so it moves only to a strictly smaller cost and the walk ends; max_rounds (the
// number of vectors in the search range) bounds it independently of the data.
// Blocks off the k-skip lattice get mv = (0,0) and best_ssd = 2^32 - 1.
__constant__ const signed char kLargeDx[8] = {0, -1, 1, -2, 2, -1, 1, 0};
__constant__ const signed char kLargeDy[8] = {-2, -1, -1, 0, 0, 1, 1, 2};
__constant__ const signed char kSmallDx[4] = {0, -1, 1, 0};
__constant__ const signed char kSmallDy[4] = {-1, 0, 0, 1};

struct DiamondBlock {
    const uint8_t* cblk;   // the block: memory (pitch W*C) or LDS (pitch B*C)
    const uint8_t* pwin;   // WIN: LDS window whose origin is the frame position (x0-R, y0-R); else the previous frame
    int H, W, C, B, R, x0, y0;
    uint32_t rb_magic;     // ceil(2^32 / (B*C)): sample index -> block row by one multiplication (exact for B^3 C^2 < 2^32)
};

// Costs of NP points around (cx, cy): cost[p] = SSD of the block against the previous frame at
// (cx + pdx[p], cy + pdy[p]), or 2^32 - 1 for a point outside the range or the frame.
template <int NP, bool WIN>
__device__ __forceinline__ void diamond_costs(const DiamondBlock& k, int cx, int cy, const signed char* pdx,
                                              const signed char* pdy, int lane, uint32_t (&cost)[NP]) {
    const int rb = k.B * k.C, n_elem = k.B * rb;
    const int cpitch = WIN ? rb : k.W * k.C;                    // block rows
    const int ppitch = WIN ? (k.B + 2 * k.R) * k.C : k.W * k.C; // previous-frame rows
    const uint8_t* src[NP];
    bool ok[NP];
    uint32_t s[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int dx = cx + pdx[p], dy = cy + pdy[p];
        ok[p] = dx >= -k.R && dx <= k.R && dy >= -k.R && dy <= k.R && k.x0 + dx >= 0 && k.y0 + dy >= 0 &&
                k.x0 + dx + k.B <= k.W && k.y0 + dy + k.B <= k.H;
        const int ex = ok[p] ? dx : 0, ey = ok[p] ? dy : 0;       // a point that is not usable is never read
        src[p] = WIN ? k.pwin + (size_t)(k.R + ey) * ppitch + (k.R + ex) * k.C
                     : k.pwin + ((size_t)(k.y0 + ey) * k.W + k.x0 + ex) * k.C;
        s[p] = 0;
    }
    // Straight-line code: every read is unconditional, so that the reads of a batch are issued together instead
    // of one latency after the other.  A sample beyond the block reads the block's first byte on both sides
    // (difference zero); a point that is not usable reads the centre's samples and is discarded below.
    for (int base = 0; base < n_elem; base += 4 * 64) {       // four samples per lane at a time
        int a[4], off[4];
        bool in[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = base + u * 64 + lane;
            in[u] = i < n_elem;
            const int r = rb == 1 ? i : (int)__umulhi((uint32_t)i, k.rb_magic), j = i - r * rb;
            off[u] = r * ppitch + j;
            const uint8_t* pa = in[u] ? k.cblk + (r * cpitch + j) : k.cblk;
            a[u] = *pa;
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint8_t* pb = in[u] ? src[p] + off[u] : k.cblk;
                const int d = a[u] - (int)*pb;
                s[p] += (uint32_t)(d * d);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) cost[p] = ok[p] ? (uint32_t)wave_sum_i32((int)s[p]) : 0xffffffffu;
}

template <bool WIN>
__global__ __launch_bounds__(256) void match_diamond_kernel(
    const uint8_t* __restrict__ cur, const uint8_t* __restrict__ prev, int H, int W, int C, int B, int R, int gw,
    int gh, int k_skip, int max_rounds, int region_bytes, uint32_t rb_magic, int16_t* __restrict__ mv,
    uint32_t* __restrict__ best_ssd) {
    extern __shared__ __align__(16) unsigned char dsm[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int nb = gh * gw;
    const int blk_id = blockIdx.x * waves + wave, stream = blockIdx.y;
    const int bx = blk_id % gw, by = blk_id / gw;
    const bool searched = blk_id < nb && bx % k_skip == 0 && by % k_skip == 0;
    const size_t frame_bytes = (size_t)H * W * C;
    const uint8_t* pf = prev + stream * frame_bytes;
    const int x0 = bx * B, y0 = by * B;
    const int rb = B * C, side = B + 2 * R;
    DiamondBlock k{cur + stream * frame_bytes + ((size_t)y0 * W + x0) * C, pf, H, W, C, B, R, x0, y0, rb_magic};
    if (WIN) {
        unsigned char* win = dsm + (size_t)wave * region_bytes;   // side rows of side*C bytes, then the block
        unsigned char* lblk = win + (size_t)side * side * C;
        if (searched) {
            // Row by row, the lanes across a row's bytes; four rows at a time, so that a pass issues 4 * ceil(wb/64)
            // independent loads per lane and the copy costs a few memory latencies, not one per byte.
            const int wb = side * C, per_row = (wb + 63) / 64;
            const int fb0 = (x0 - R) * C;
            for (int r0 = 0; r0 < side; r0 += 4) {
                for (int q = 0; q < per_row; ++q) {
                    const int j = q * 64 + lane, fb = fb0 + j;
                    unsigned char v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {             // bytes outside the frame are never used: zero
                        const int r = r0 + u, fy = y0 - R + r;
                        const bool in = r < side && j < wb && fy >= 0 && fy < H && fb >= 0 && fb < W * C;
                        const unsigned char g = pf[in ? (size_t)fy * W * C + fb : 0];   // unconditional: the loads overlap
                        v[u] = in ? g : 0;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (r0 + u < side && j < wb) win[(r0 + u) * wb + j] = v[u];
                }
            }
            for (int r0 = 0; r0 < B; r0 += 8) {
                for (int q = 0; q < (rb + 63) / 64; ++q) {
                    const int j = q * 64 + lane;
                    unsigned char v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = k.cblk[(r0 + u < B && j < rb) ? (size_t)(r0 + u) * W * C + j : 0];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (r0 + u < B && j < rb) lblk[(r0 + u) * rb + j] = v[u];
                }
            }
        }
        __syncthreads();     // every wavefront of the workgroup arrives here, searched block or not
        k.cblk = lblk;
        k.pwin = win;
    }
    if (blk_id >= nb) return;
    int16_t* out_mv = mv + ((size_t)stream * nb + blk_id) * 2;
    uint32_t* out_ssd = best_ssd + (size_t)stream * nb + blk_id;
    if (!searched) {
        if (lane == 0) { out_mv[0] = 0; out_mv[1] = 0; *out_ssd = 0xffffffffu; }
        return;
    }
    const signed char zero = 0;
    uint32_t c0[1];
    diamond_costs<1, WIN>(k, 0, 0, &zero, &zero, lane, c0);
    int cx = 0, cy = 0;
    uint32_t ccost = c0[0];
    for (int round = 0; round < max_rounds; ++round) {
        uint32_t c[8];
        diamond_costs<8, WIN>(k, cx, cy, kLargeDx, kLargeDy, lane, c);
        int best = -1;
        uint32_t bcost = ccost;
#pragma unroll
        for (int p = 0; p < 8; ++p)
            if (c[p] < bcost) { bcost = c[p]; best = p; }
        if (best < 0) break;
        cx += kLargeDx[best]; cy += kLargeDy[best]; ccost = bcost;
    }
    uint32_t c[4];
    diamond_costs<4, WIN>(k, cx, cy, kSmallDx, kSmallDy, lane, c);
    int best = -1;
    uint32_t bcost = ccost;
#pragma unroll
    for (int p = 0; p < 4; ++p)
        if (c[p] < bcost) { bcost = c[p]; best = p; }
    if (best >= 0) { cx += kSmallDx[best]; cy += kSmallDy[best]; }
    if (lane == 0) { out_mv[0] = (int16_t)cx; out_mv[1] = (int16_t)cy; *out_ssd = bcost; }
}

// The same walk for blocks whose rows are whole dwords, 256 of them at most (16x16 blocks of up to four channels).  What
// bounded a round was instructions: a byte at a time it takes a read, a subtraction and a multiply-add per sample and point,
// 1.7 us, and the longest walk of a launch makes up to 19 rounds.  Here a lane keeps U dwords of the block in registers, a
// point is SSD = sum a^2 + sum b^2 - 2 sum a b in byte dot products on two LDS dwords and one alignment (the shift is the
// same for all lanes: the window's rows are whole dwords apart), and the window arrives in 16-byte pieces.  Only the searched
// blocks are launched; motion_retest_kernel writes the entries of the others.
// 416x416, 16 streams, every second block row and column: 112 -> 33 us.
template <int U>
__global__ __launch_bounds__(256) void match_diamond_words_kernel(
    const uint8_t* __restrict__ cur, const uint8_t* __restrict__ prev, int H, int W, int C, int B, int R, int gw, int gh,
    int k_skip, int max_rounds, int pitch, uint32_t row_magic, uint32_t piece_magic, int16_t* __restrict__ mv,
    uint32_t* __restrict__ best_ssd) {
    extern __shared__ __align__(16) unsigned char dsm[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int lgw = (gw + k_skip - 1) / k_skip, lgh = (gh + k_skip - 1) / k_skip;
    const int at = (int)blockIdx.x * waves + wave;
    if (at >= lgw * lgh) return;                                     // (no barrier below: a wavefront has its own window)
    const int stream = blockIdx.y, by = at / lgw * k_skip, bx = (at - at / lgw * lgw) * k_skip;
    const int x0 = bx * B, y0 = by * B;
    const int row_bytes = W * C, frame_bytes = H * row_bytes, side = B + 2 * R;
    const uint8_t* const pf = prev + (size_t)stream * (uint32_t)frame_bytes;
    const uint8_t* const cf = cur + (size_t)stream * (uint32_t)frame_bytes;
    unsigned char* const win = dsm + (size_t)wave * side * pitch;

    // the block: dword lane + 64 u, its place below the point's first byte, zeros past the end
    const int per_row = B * C / 4, n_dw = B * per_row;
    uint32_t a[U], keep[U];
    int off[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = lane + 64 * u < n_dw ? lane + 64 * u : 0;
        const int r = row_magic ? (int)__umulhi((uint32_t)i, row_magic) : i, j = i - r * per_row;
        keep[u] = lane + 64 * u < n_dw ? ~0u : 0u;
        off[u] = r * pitch + 4 * j;
        __builtin_memcpy(&a[u], cf + (uint32_t)((y0 + r) * row_bytes + x0 * C + 4 * j), 4);
    }
    // the window, eight pieces of a lane in flight (rows above and below the frame: any row's bytes)
    const int pieces = pitch / 16, n_pieces = side * pieces;
    for (int base = 0; base < n_pieces; base += 8 * 64) {
        uintx4 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = base + 64 * q + lane, r = piece_magic ? (int)__umulhi((uint32_t)i, piece_magic) : i, j = i - r * pieces;
            int y = y0 - R + (r < side ? r : side - 1);
            y = y < 0 ? 0 : (y < H ? y : H - 1);
            if (base + 64 * q < n_pieces) v[q] = load16_within(pf, y * row_bytes + (x0 - R) * C + 16 * j, frame_bytes);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = base + 64 * q + lane;
            if (i < n_pieces) *reinterpret_cast<uintx4*>(win + 16 * i) = v[q];
        }
    }
    uint32_t saa = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) { a[u] &= keep[u]; saa = udot4(a[u], a[u], saa); }
    saa = (uint32_t)wave_sum_i32((int)saa);
    __builtin_amdgcn_wave_barrier();                                 // (LDS operations of a wavefront stay in order)

    // costs of NP points around (cx, cy); 2^32 - 1 for a point outside the range or the frame
    auto costs = [&](auto np_tag, int cx, int cy, const signed char* pdx, const signed char* pdy, uint32_t* cost) {
        constexpr int NP = decltype(np_tag)::value;
        uint32_t s[NP];
        bool ok[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int dx = cx + pdx[p], dy = cy + pdy[p];
            ok[p] = dx >= -R && dx <= R && dy >= -R && dy <= R && x0 + dx >= 0 && y0 + dy >= 0 && x0 + dx + B <= W && y0 + dy + B <= H;
            const int first = (R + (ok[p] ? dy : 0)) * pitch + (R + (ok[p] ? dx : 0)) * C, sh = first & 3;
            uint32_t sbb = 0, sab = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t* const w = reinterpret_cast<const uint32_t*>(win + (first - sh) + off[u]);
                const uint32_t b = __builtin_amdgcn_alignbyte(w[1], w[0], sh) & keep[u];
                sbb = udot4(b, b, sbb);
                sab = udot4(a[u], b, sab);
            }
            s[p] = sbb - 2u * sab;
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uint32_t sum = (uint32_t)wave_sum_i32((int)s[p]);
            cost[p] = ok[p] ? saa + sum : 0xffffffffu;
        }
    };
    const signed char zero = 0;
    uint32_t c0[1], c[8];
    costs(std::integral_constant<int, 1>(), 0, 0, &zero, &zero, c0);
    int cx = 0, cy = 0, best = 0;
    uint32_t ccost = c0[0];
    for (int round = 0; round < max_rounds; ++round) {
        costs(std::integral_constant<int, 8>(), cx, cy, kLargeDx, kLargeDy, c);
        best = -1;
        uint32_t bcost = ccost;
#pragma unroll
        for (int p = 0; p < 8; ++p)
            if (c[p] < bcost) { bcost = c[p]; best = p; }
        if (best < 0) break;
        cx += kLargeDx[best]; cy += kLargeDy[best]; ccost = bcost;
    }
    costs(std::integral_constant<int, 4>(), cx, cy, kSmallDx, kSmallDy, c);
    best = -1;
#pragma unroll
    for (int p = 0; p < 4; ++p)
        if (c[p] < ccost) { ccost = c[p]; best = p; }
    if (best >= 0) { cx += kSmallDx[best]; cy += kSmallDy[best]; }
    if (lane == 0) {
        const size_t o = (size_t)stream * gh * gw + by * gw + bx;
        mv[2 * o] = (int16_t)cx; mv[2 * o + 1] = (int16_t)cy; best_ssd[o] = ccost;
    }
}

}  // namespace

hipError_t launch_match(const uint8_t* cur, const uint8_t* prev, int n_streams, int H, int W, int C,
                        int B, int R, int k_skip, uint32_t max_ssd, int16_t* mv, uint32_t* best_ssd,
                        int32_t* gmv, int32_t* n_pass, uint8_t* mask, hipStream_t st) {
    const int gh = H / B, gw = W / B;
    k_skip = std::min(k_skip, std::max(gw, gh));           // beyond, the first block alone is searched either way (and sums overflow)
    const int rows = B + 2 * R;
    const bool aligned = ((reinterpret_cast<uintptr_t>(prev) & 3) == 0) && ((W * C) % 4 == 0);
    dim3 grid(((gw + k_skip - 1) / k_skip) * ((gh + k_skip - 1) / k_skip), n_streams);   // the searched blocks
    constexpr bool use_mfma = true;
    const int nt = (2 * R + 1 + 15) / 16, ksteps = (B * C + 63) / 64;
    bool done = false;
    // a kernel of its own for the usual shape (43 against 115 us, see there); it addresses a frame with 32 bits
    const int lgw = (gw + k_skip - 1) / k_skip, lgh = (gh + k_skip - 1) / k_skip;
    if (C == 3 && R == B && (B == 8 || B == 16) && lgh <= 65535 && (double)H * W * C < 2147400000.0) {
        const dim3 blocks((unsigned)lgw, (unsigned)lgh, (unsigned)n_streams);
        if (B == 16) hipLaunchKernelGGL(match_window_kernel<16>, blocks, dim3(kMfmaThreads), 0, st, cur, prev, H, W, gw, gh, k_skip, mv, best_ssd);
        else hipLaunchKernelGGL(match_window_kernel<8>, blocks, dim3(kMfmaThreads), 0, st, cur, prev, H, W, gw, gh, k_skip, mv, best_ssd);
        done = true;
    }
    if (!done && use_mfma && nt <= 3 && ksteps <= 2 && B + 2 * R <= 255) {
        const int nd = 2 * R + 1;
        const int need = 3 + C * (16 * nt - 1) + 64 * ksteps + 4, real = 3 + rows * C + 4;
        const int wsm = (int)align_up((size_t)(need > real ? need : real), 16);
        // the instantiations below that know the block shape take their row sums from the window bytes: no per-pixel sums (they
        // serve the ranges from 17 to 23 and 9 to 15; those of the block edge have gone above)
        const bool fused = (nt == 3 && B == 16 && C == 3) || (nt == 2 && B == 8 && C == 3);
        const size_t dead = (size_t)rows * wsm + (size_t)B * 64 * ksteps + (size_t)((fused ? 0 : rows * rows) + rows * nd) * 4;
        const size_t ldsm = dead + 16 + (size_t)(3 * kMfmaWaves + nd * nd) * 4;
        if (ldsm <= 64 * 1024 && (size_t)nt * nt * 1024 <= dead) {   // the tile buffer of the final sum fits over the dead part
#define DC_MFMA_LAUNCH(AL, NTT, KSS, BT, CT)                                                                          \
    hipLaunchKernelGGL((match_mfma_kernel<AL, NTT, KSS, BT, CT>), grid, dim3(kMfmaThreads), ldsm, st, cur, prev, H, W, C, \
                       B, R, gw, gh, wsm, k_skip, mv, best_ssd)
#define DC_MFMA_KS(AL, NTT)                            \
    do {                                               \
        if (ksteps == 1) DC_MFMA_LAUNCH(AL, NTT, 1, 0, 0); \
        else DC_MFMA_LAUNCH(AL, NTT, 2, 0, 0);             \
    } while (0)
#define DC_MFMA_NT(AL)                                                     \
    do {                                                                   \
        if (nt == 3 && B == 16 && C == 3) DC_MFMA_LAUNCH(AL, 3, 1, 16, 3); \
        else if (nt == 2 && B == 8 && C == 3) DC_MFMA_LAUNCH(AL, 2, 1, 8, 3); \
        else if (nt == 1) DC_MFMA_KS(AL, 1);                               \
        else if (nt == 2) DC_MFMA_KS(AL, 2);                               \
        else DC_MFMA_KS(AL, 3);                                            \
    } while (0)
            if (aligned) DC_MFMA_NT(true);
            else DC_MFMA_NT(false);
#undef DC_MFMA_NT
#undef DC_MFMA_KS
#undef DC_MFMA_LAUNCH
            done = true;
        }
    }
    const int ws = (int)align_up((size_t)rows * C + 3, 4) + 8;  // skew (<=3) + window + over-read of the last dword pair
    const int cs = (int)align_up((size_t)B * C, 4);
    const size_t lds = (size_t)rows * ws + (size_t)B * cs;
#define DC_MATCH_LAUNCH(AL, CD)                                                                                      \
    hipLaunchKernelGGL((match_search_kernel<AL, CD>), grid, dim3(kSearchThreads), lds, st, cur, prev, H, W, C, B, R, \
                       gw, gh, ws, cs, k_skip, mv, best_ssd)
#define DC_MATCH_ALIGN(CD)             \
    do {                               \
        if (aligned) DC_MATCH_LAUNCH(true, CD); \
        else DC_MATCH_LAUNCH(false, CD);        \
    } while (0)
    if (!done) switch (cs / 4) {
        case 6: DC_MATCH_ALIGN(6); break;     // 8x8x3
        case 8: DC_MATCH_ALIGN(8); break;     // 10x10x3, 8x8x4
        case 12: DC_MATCH_ALIGN(12); break;   // 16x16x3
        case 16: DC_MATCH_ALIGN(16); break;   // 16x16x4
        default: DC_MATCH_ALIGN(0); break;
    }
#undef DC_MATCH_ALIGN
#undef DC_MATCH_LAUNCH
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_motion_retest(cur, prev, n_streams, H, W, C, B, gw, gh, max_ssd, mv, best_ssd, gmv, n_pass, mask, k_skip, st);
}

hipError_t launch_match_diamond(const uint8_t* cur, const uint8_t* prev, int n_streams, int H, int W, int C, int B,
                                int R, int k_skip, uint32_t max_ssd, int16_t* mv, uint32_t* best_ssd, int32_t* gmv,
                                int32_t* n_pass, uint8_t* mask, hipStream_t st) {
    const int gh = H / B, gw = W / B;
    k_skip = std::min(k_skip, std::max(gw, gh));           // as above
    const unsigned long long nvec = (2ull * R + 1) * (2ull * R + 1);
    const int cap = (int)(nvec < 0x7fffffffull ? nvec : 0x7fffffffull);
    auto magic = [](int d) { return (uint32_t)((0x100000000ull + (uint64_t)d - 1) / (uint64_t)d); };
    // whole dwords in a block row, four of them per lane at most, windows that leave two wavefronts in 64 KiB
    const int pitch = (int)align_up(((size_t)B + 2 * (size_t)R) * C + 4, 16);          // a point's second dword may lie behind its row
    const size_t window = ((size_t)B + 2 * (size_t)R) * pitch;
    const int n_dw = B * B * C / 4;
    if (B * C % 4 == 0 && n_dw <= 256 && window <= 32 * 1024 && (double)H * W * C < 2147400000.0 &&
        H * W * C >= 16) {                                 // (a 16-byte piece of a frame)
        const int searched = ((gw + k_skip - 1) / k_skip) * ((gh + k_skip - 1) / k_skip), waves = window <= 16 * 1024 ? 4 : 2;
        const dim3 grid((unsigned)((searched + waves - 1) / waves), (unsigned)n_streams);
#define DC_DIAMOND(U)                                                                                                        \
    hipLaunchKernelGGL(match_diamond_words_kernel<U>, grid, dim3(waves * 64), window * waves, st, cur, prev, H, W, C, B, R,   \
                       gw, gh, k_skip, cap, pitch, magic(B * C / 4), magic(pitch / 16), mv, best_ssd)
        switch ((n_dw + 63) / 64) {
            case 1: DC_DIAMOND(1); break;
            case 2: DC_DIAMOND(2); break;
            case 3: DC_DIAMOND(3); break;
            default: DC_DIAMOND(4); break;
        }
#undef DC_DIAMOND
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_motion_retest(cur, prev, n_streams, H, W, C, B, gw, gh, max_ssd, mv, best_ssd, gmv, n_pass, mask, k_skip, st);
    }
    const uint32_t rb_magic = magic(B * C);
    // LDS per wavefront: the search window and the block; as many wavefronts per workgroup as fit into 64 KiB
    const size_t side = (size_t)B + 2 * (size_t)R;
    const size_t region = align_up(side * side * C + (size_t)B * B * C, 16);
    const int waves = region <= 16 * 1024 ? 4 : (region <= 32 * 1024 ? 2 : 1);
    if (region <= 64 * 1024)
        hipLaunchKernelGGL(match_diamond_kernel<true>, dim3((gh * gw + waves - 1) / waves, n_streams), dim3(waves * 64),
                           region * waves, st, cur, prev, H, W, C, B, R, gw, gh, k_skip, cap, (int)region, rb_magic, mv, best_ssd);
    else
        hipLaunchKernelGGL(match_diamond_kernel<false>, dim3((gh * gw + 3) / 4, n_streams), dim3(256), 0, st, cur, prev,
                           H, W, C, B, R, gw, gh, k_skip, cap, 0, rb_magic, mv, best_ssd);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_motion_retest(cur, prev, n_streams, H, W, C, B, gw, gh, max_ssd, mv, best_ssd, gmv, n_pass, mask, k_skip, st);
}

}  // namespace dc
