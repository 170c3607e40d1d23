// Cache-aware convolution (Section 5 "Reuse", steps 2-3), the kernels for the common layer shape: 3x3 taps,
// stride 1, and their neighbours.  The kernels of this file:
//   conv_fast_kernel   channel counts that are whole 64-byte rows, 64 or 128 output channels per workgroup (5x5 taps
//                      as well, in bf16);
//   conv_map_kernel    bf16, 3x3, maps of up to 14x14 of which nearly every unit has work (see there);
//   conv_deep_kernel   bf16, 3x3, many units: weights from L2 into registers (see there);
//   conv_pw_kernel     1x1 layers, with a residual sum behind or several of one tensor in a launch (see there);
//   conv_stem4_kernel  7x7 and 11x11 stems in bf16 (see there);
//   conv_regw_kernel   64 input channels in bf16 and many units: persistent, weights in registers (see there);
//   conv_first_kernel  input pixels of one 16-byte vector (the padded first layer), nothing staged (see there).
//
// conv_fast_kernel is the same implicit GEMM over 4x4-pixel units as the general kernels, with everything that
// shapes the inner loop fixed at compile time, so that the loop is straight-line code: LDS reads at register +
// immediate addresses, no address arithmetic between MFMAs, and exact wait counts between the reads of one
// K step and the MFMAs of the previous one.
//
//   workgroup  = g units (g <= WM*UPW, a launch parameter) x NT channels x a range of channel chunks
//   wavefront  = UPW units (slots wave_m, wave_m + WM, ...) x NBW 16-channel blocks
//   stage      = one kernel row (3 or 5 taps) x one channel chunk (KC channels)
//
// LDS: the patch of a unit is 6 lines of 8 row slots (6 used; 5x5 taps: 8 lines, all used), one row = KC channels = RB bytes.  Chunk c
// (16 bytes) of the row at (line py, slot px) sits at chunk position c ^ sw(py, px), of weight row r at
// c ^ (r / 2) % NVEC.  sw = (2 py + px / 4) % 4 for 64-byte rows, (py % 4) * 2 + (px % 4) / 2 for 128-byte rows:
// these are the swizzles for which SQ_LDS_BANK_CONFLICT stays at zero for every tap (a 16-byte read of a
// wavefront is not served 16 consecutive lanes at a time, so "16 different bank groups per quarter wavefront"
// is not the rule; the candidates were measured).  Both buffers are filled by buffer_load ... lds,
// double-buffered; the patch of the next chunk arrives in three parts, one per stage.  The weights come from
// the plain [cout][3][3][cin] layout or, when the caller has one, from the packed copy whose 1 KiB load units
// are contiguous (launch_pack_weights).
//
// Few units and a deep K (the small maps at the end of a stack): the launch splits the channel
// chunks among ks workgroups per tile, which store fp32 partial sums to scratch memory; a second
// kernel adds them in a fixed order and applies the epilogue.  Every workgroup then loads only its
// share of the weights, which is what bounds these layers.
#include <algorithm>
#include <cstdio>
#include <atomic>
#include <cstdlib>
#include <mutex>
#include <type_traits>

#include "dc_conv_common.h"

namespace dc {

namespace {

// LDS header of this kernel.  uq[g] = {byte offset in the input of the patch origin of unit g (the
// pixel at (-p, -p) of the unit; may lie outside the tensor), row and column of that origin, element
// offset in the output of the unit's first pixel}; skip[16 g + i] = 1: pixel i of unit g is not stored
// (missing unit, outside the map, or inside a reusable rectangle).
template <int G>
struct FastHeader {
    int4* uq;
    int* ustream;
    int* ukind;             // -1: no unit, otherwise the 16-bit mask of the unit's reusable pixels
    unsigned char* skip;
    int4* uorg;             // tensors on a torus: {input ox, oy, output ox, oy} of the unit's stream
    __device__ __forceinline__ explicit FastHeader(unsigned char* smem)
        : uq(reinterpret_cast<int4*>(smem)), ustream(reinterpret_cast<int*>(smem + 16 * G)),
          ukind(reinterpret_cast<int*>(smem + 20 * G)), skip(smem + 24 * G),
          uorg(reinterpret_cast<int4*>(smem + 40 * G)) {}   // 56 G <= 1008 bytes (G <= 18)
};

template <int G, int NTHREADS, int ES>
__device__ __forceinline__ void decode_units_fast(const ConvParams& P, const FastHeader<G>& H, int ug, int tid, int n_units) {
    static_assert(G * 16 <= NTHREADS, "one thread per pixel of the unit table");
    if (tid < G) {
        const int u = ug * P.g_rt + tid;
        const bool valid = tid < P.g_rt && u < n_units;
        int stream = 0, uy = 0, ux = 0, mixed = 0;
        if (valid) {
            if (P.units) {
                const TileDev t = P.units[u];
                stream = t.stream; uy = t.ty; ux = t.tx; mixed = t.reuse_mask;
            } else {   // raster order
                stream = fast_div_any(u, P.npix_magic, P.units_x * P.units_y);
                const int r = u - stream * (P.units_x * P.units_y);
                uy = fast_div(r, P.pw_magic); ux = r - uy * P.units_x;
            }
        }
        const int oy = uy * 4 - P.p, ox = ux * 4 - P.p;
        int4 v;
        v.x = ((stream * P.Hin + oy) * P.Win + ox) * P.Cin * ES;
        v.y = valid ? oy : -(1 << 24);      // every pixel of a missing unit fails the range test
        v.z = ox;
        v.w = ((stream * P.Hout + uy * 4) * P.Wout + ux * 4) * P.Cout;
        H.uq[tid] = v;
        H.ustream[tid] = stream;
        H.ukind[tid] = valid ? mixed : -1;
        if (P.in_origin || P.out_origin) {
            int4 og{0, 0, 0, 0};
            const size_t at = (size_t)stream * P.origin_stride;
            if (P.in_origin) { og.x = P.in_origin[at]; og.y = P.in_origin[at + 1]; }
            if (P.out_origin) { og.z = P.out_origin[at]; og.w = P.out_origin[at + 1]; }
            H.uorg[tid] = og;
        }
    }
    __syncthreads();
    if (tid < G * 16) {
        const int g = tid >> 4, kind = H.ukind[g];
        const int y = H.uq[g].y + P.p + ((tid >> 2) & 3), x = H.uq[g].z + P.p + (tid & 3);
        const unsigned char hit = (kind < 0 || y >= P.Hout || x >= P.Wout || ((kind >> (tid & 15)) & 1)) ? 1 : 0;
        H.skip[tid] = hit;
    }
    __syncthreads();
}

// Chunk swizzle of the patch row at (line py, slot px) for rows of RB bytes.
template <int RB>
__device__ __forceinline__ int patch_swizzle(int py, int px) {
    return RB == 64 ? (2 * py + px / 4) % 4 : (py % 4) * 2 + (px % 4) / 2;
}

template <typename T, int KSZ, int KC, int UPW, int WM, int WN, int NBW>
__global__ __launch_bounds__(WM* WN * 64) void conv_fast_kernel(ConvParams P) {
    typedef Frag<T> F;
    typedef typename F::vec vec;
    constexpr int VE = F::VE;
    constexpr int ES = (int)sizeof(T);
    constexpr int KG = 4 * VE;                  // K elements per MFMA group
    constexpr int NW = WM * WN;
    constexpr int NTHREADS = NW * 64;
    constexpr int G = WM * UPW;
    constexpr int NT = WN * NBW * 16;
    constexpr int GPC = KC / KG;                // K groups per chunk
    constexpr int NVEC = KC / VE;               // 16-byte chunks per row
    constexpr int RB = KC * ES;                 // row bytes
    constexpr int RPI = 64 / NVEC;              // rows per load instruction (1 KiB)
    constexpr int PWP = 8;                      // row slots per patch line
    constexpr int PH = 3 + KSZ;                 // patch lines and used slots per line
    constexpr int PR = PH * PWP;                // LDS rows per unit
    constexpr int P_INSTR = G * PR / RPI;       // patch load instructions per chunk
    constexpr int W_INSTR = KSZ * NT / RPI;     // weight load instructions per stage
    constexpr int NPI = (P_INSTR + NW - 1) / NW;
    constexpr int NWI = (W_INSTR + NW - 1) / NW;
    constexpr int PBYTES = P_INSTR * 1024;
    constexpr int WBYTES = W_INSTR * 1024;
    constexpr int NS = KSZ * GPC;               // K steps per stage
    static_assert((KSZ == 3 || KSZ == 5) && RB >= 64 && RB <= 128 && (G * PR) % RPI == 0 && (KSZ * NT) % RPI == 0, "shape");

    extern __shared__ __align__(16) unsigned char smem[];
    const FastHeader<G> H(smem);
    unsigned char* const patch0 = smem + kHeaderBytes;
    unsigned char* const wts0 = patch0 + 2 * PBYTES;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_n = wave % WN, wave_m = wave / WN;
    const int l16 = lane & 15, q = lane >> 4;

    int ug, ntile;
    decode_workgroup(P.R, ug, ntile);
    const int n_units = unit_count(P);
    if (ug * P.g_rt >= n_units) return;     // the launch is sized for the longest possible list (whole workgroup, before any barrier)
    const int n0 = ntile * NT;
    const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(keep_scalar(reinterpret_cast<uintptr_t>(P.in))), 0, keep_scalar(P.in_bytes), kBufferFlags);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(keep_scalar(reinterpret_cast<uintptr_t>(P.w))), 0, keep_scalar(P.w_bytes), kBufferFlags);
    const int Cin = keep_scalar(P.Cin);
    const bool packed = keep_scalar(P.w_packed) != 0;

    // ---- load side: instruction j of a buffer fills LDS bytes [1024 j, 1024 j + 1024); this wavefront
    // issues instructions wave, wave + NW, ...; the lane fills chunk position lane % NVEC of row
    // j * RPI + lane / NVEC and fetches the logical chunk that belongs there.
    const int lrow = lane / NVEC, lpos = lane % NVEC;
    uint32_t wgo[NWI];
#pragma unroll
    for (int i = 0; i < NWI; ++i) {
        const int row = (wave + i * NW) * RPI + lrow;   // tl * NT + n
        const int tl = row / NT, n = row - tl * NT;
        const int c = lpos ^ ((row / 2) % NVEC);
        uint32_t off;
        if (packed)   // [channel / 16][64-byte chunk of the row][tap][channel % 16][64 bytes]
            off = (uint32_t)((((n0 + n) / 16 * (Cin * ES / 64) * (KSZ * KSZ) + tl) * 16 + n % 16) * 64 + (c / 4) * (KSZ * KSZ * 1024) + ((c % 4) << 4));
        else
            off = (uint32_t)(((n0 + n) * (KSZ * KSZ) + tl) * Cin) * ES + (uint32_t)(c << 4);
        wgo[i] = tl < KSZ ? off : kOob;
    }

    auto issue_w = [&](int chunk, int ky, int wbuf) {
        unsigned char* dst = wts0 + wbuf * WBYTES + wave * 1024;
        const uint32_t so = packed ? (uint32_t)((chunk * (RB / 64) * KSZ + ky) * (KSZ * 1024)) : (uint32_t)(ky * KSZ * Cin + chunk * KC) * ES;
#pragma unroll
        for (int i = 0; i < NWI; ++i) {
            const uint32_t off = wgo[i] + so;   // (a named value: an expression in the builtin's argument list loses the host stub)
            if ((i + 1) * NW <= W_INSTR || wave + i * NW < W_INSTR)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (__attribute__((address_space(3))) void*)(dst + i * (NW * 1024)),
                                                         16, off, 0, 0, 0);
        }
    };
    const int cb = keep_scalar((int)blockIdx.y * P.chunks_per_split);
    const int ce0 = cb + P.chunks_per_split;
    const int ce = keep_scalar(ce0 < P.n_chunks ? ce0 : P.n_chunks);

    issue_w(cb, 0, 0);   // the first weights do not depend on the units: they travel while the unit table is decoded

    decode_units_fast<G, NTHREADS, ES>(P, H, ug, tid, n_units);

    // patch: IPU instructions per unit; instruction j covers lines [(j % IPU) * RPI / 8, ...) of unit j / IPU,
    // so the slot column and the line within the instruction are fixed per lane
    constexpr int IPU = PR / RPI;
    uint32_t pgo[NPI];
    {
        const int px = lrow % PWP, pyl = lrow / PWP;
        const int CinES = Cin * ES;
        const int pxoff = px * CinES;
#pragma unroll
        for (int i = 0; i < NPI; ++i) {
            const int j = wave + i * NW;
            int unit = j / IPU;
            const int part = j - unit * IPU;
            unit = unit < G ? unit : G - 1;
            const int4 uq = H.uq[unit];
            const int py = part * (RPI / PWP) + pyl;
            const int sw = patch_swizzle<RB>(py, px);
            const bool ok = px < PH && (unsigned)(uq.y + py) < (unsigned)P.Hin && (unsigned)(uq.z + px) < (unsigned)P.Win;
            uint32_t off = (uint32_t)(uq.x + py * (P.Win * CinES) + pxoff + ((lpos ^ sw) << 4));
            if (P.in_origin && ok) {      // the input lies on a torus: the patch may cross its seams
                const int4 og = H.uorg[unit];
                const int iy = torus_wrap(uq.y + py, og.y, P.Hin), ix = torus_wrap(uq.z + px, og.x, P.Win);
                off = (uint32_t)(((H.ustream[unit] * P.Hin + iy) * P.Win + ix) * CinES + ((lpos ^ sw) << 4));
            }
            pgo[i] = ok ? off : kOob;
        }
    }
    // part < 0: the whole patch; otherwise the instructions with index % KSZ == part
    auto issue_p = [&](int chunk, int part, int pbuf) {
        unsigned char* dst = patch0 + pbuf * PBYTES + wave * 1024;
        const uint32_t so = (uint32_t)(chunk * KC) * ES;
#pragma unroll
        for (int i = 0; i < NPI; ++i) {
            if (part >= 0 && i % KSZ != part) continue;
            const uint32_t off = pgo[i] + so;
            if ((i + 1) * NW <= P_INSTR || wave + i * NW < P_INSTR)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(in_rsrc, (__attribute__((address_space(3))) void*)(dst + i * (NW * 1024)),
                                                         16, off, 0, 0, 0);
        }
    };

    // ---- read side: byte address of this lane's row and chunk for every tap and K group
    // (the swizzle of 64-byte rows repeats every two lines: kernel row ky is row ky % 2 plus an immediate offset)
    constexpr int PK = RB == 64 ? 2 : KSZ;      // kernel rows with addresses of their own
    int paddr[PK * KSZ][GPC];
    {
        const int oy = l16 >> 2, ox = l16 & 3;
#pragma unroll
        for (int t = 0; t < PK * KSZ; ++t) {
            const int py = oy + t / KSZ, px = ox + t % KSZ;
            const int sw = patch_swizzle<RB>(py, px);
#pragma unroll
            for (int g = 0; g < GPC; ++g)
                paddr[t][g] = (wave_m * PR + py * PWP + px) * RB + (((g * 4 + q) ^ sw) << 4);
        }
    }
    int waddr[GPC];
#pragma unroll
    for (int g = 0; g < GPC; ++g)
        waddr[g] = (wave_n * NBW * 16 + l16) * RB + (((g * 4 + q) ^ ((l16 / 2) % NVEC)) << 4);

    floatx4 acc[UPW][NBW];
#pragma unroll
    for (int u = 0; u < UPW; ++u)
#pragma unroll
        for (int j = 0; j < NBW; ++j) acc[u][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // 5x5: the sums of a stage alone, then added to the total, so that no chain of roundings is longer than a stage's few
    // taps and the stages (the general kernel, which these layers came from, splits their K into up to eight sums)
    constexpr bool SHORT = KSZ == 5;
    // epilogue operands that do not depend on the accumulators
    const int chan = n0 + wave_n * NBW * 16 + 4 * q;
    floatx4 bias[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j)
        bias[j] = P.bias ? *reinterpret_cast<const floatx4*>(P.bias + chan + j * 16) : floatx4{0.f, 0.f, 0.f, 0.f};

    // Loads of stage s = KSZ c + ky (c counts this workgroup's chunks): the weights of kernel row ky and one of KSZ
    // parts of a patch: 3x3 stages 3c+1, 3c+2 and 3c+3 bring parts 0, 1 and 2 of chunk c+1.  They are issued
    // two stages ahead, right after the barrier that ends the reads of the buffers they overwrite.
    const int n_ch = ce - cb;
    auto issue_stage = [&](int c, int ky, int s) {     // ky is a compile-time constant at every call
        if (c >= n_ch) return;
        issue_w(cb + c, ky, s & 1);
        if (ky == 0) { if (c > 0) issue_p(cb + c, KSZ - 1, c & 1); }
        else if (c + 1 < n_ch) issue_p(cb + c + 1, ky - 1, (c + 1) & 1);
    };
    // The main loop for a wavefront with NU units.  The units of a workgroup are dealt to the wave_m groups
    // round-robin, so a group holds UPW or UPW - 1 of them; both variants run the same stages and barriers.
    auto main_loop = [&](auto nu_tag) {
        constexpr int NU = decltype(nu_tag)::value;
        vec x[2][NU > 0 ? NU : 1], w[2][NBW];
        auto frag = [&](int pbuf, int wbuf, int ky, int st, int b) {
            const int kx = st / GPC, g = st % GPC;
            const unsigned char* xp = patch0 + pbuf * PBYTES + paddr[ky % PK * KSZ + kx][g] + (ky - ky % PK) * (PWP * RB);
#pragma unroll
            for (int u = 0; u < NU; ++u) x[b][u] = *reinterpret_cast<const vec*>(xp + u * (WM * PR * RB));
            const unsigned char* wp = wts0 + wbuf * WBYTES + waddr[g] + kx * (NT * RB);
#pragma unroll
            for (int j = 0; j < NBW; ++j) w[b][j] = *reinterpret_cast<const vec*>(wp + j * (16 * RB));
        };
        typedef floatx4 Sums[UPW][NBW];
        auto mma = [&](int b, Sums& sum) {
#pragma unroll
            for (int e = 0; e < F::NE; ++e)
#pragma unroll
                for (int u = 0; u < NU; ++u)
#pragma unroll
                    for (int j = 0; j < NBW; ++j) F::mma1(w[b][j], x[b][u], sum[u][j], e);
        };

        issue_p(cb, -1, 0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        issue_stage(0, 1, 1);
        frag(0, 0, 0, 0, 0);
        int sidx = 0;
        for (int c = 0; c < n_ch; ++c) {
            const int pbuf = c & 1;
#pragma unroll
            for (int ky = 0; ky < KSZ; ++ky, ++sidx) {
                // fragments of step 0 of this stage are on their way (buffer (ky * NS) & 1)
                Sums part = {};                                   // (SHORT) of this stage
                Sums& sum = SHORT ? part : acc;
#pragma unroll
                for (int st = 0; st + 1 < NS; ++st) {
                    frag(pbuf, sidx & 1, ky, st + 1, (ky * NS + st + 1) & 1);
                    __builtin_amdgcn_sched_barrier(0);
                    mma((ky * NS + st) & 1, sum);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // Last step: first end the stage for the memory system.  After the barrier every wavefront has
                // its last fragments of this stage in registers and the loads of the next stage are in LDS.
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                if (ky + 2 < KSZ) issue_stage(c, ky + 2, sidx + 2);
                else issue_stage(c + 1, ky + 2 - KSZ, sidx + 2);
                if (ky + 1 < KSZ) frag(pbuf, (sidx + 1) & 1, ky + 1, 0, ((ky + 1) * NS) & 1);
                else if (c + 1 < n_ch) frag(pbuf ^ 1, (sidx + 1) & 1, 0, 0, (KSZ * NS) & 1);
                __builtin_amdgcn_sched_barrier(0);
                mma((ky * NS + NS - 1) & 1, sum);
                if constexpr (SHORT) {
#pragma unroll
                    for (int u = 0; u < NU; ++u)
#pragma unroll
                        for (int j = 0; j < NBW; ++j) {
                            acc[u][j] += part[u][j];
                            asm volatile("" : "+v"(acc[u][j]));      // now: put off, the sums of five stages need registers at once
                        }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if ((KSZ * NS) & 1) {   // the next chunk expects its first fragments in buffer 0
#pragma unroll
                for (int u = 0; u < NU; ++u) x[0][u] = x[1][u];
#pragma unroll
                for (int j = 0; j < NBW; ++j) w[0][j] = w[1][j];
            }
        }
    };
    const int n_u = keep_scalar((P.g_rt - wave_m + WM - 1) / WM);
    if (n_u == UPW) main_loop(std::integral_constant<int, UPW>());
    else main_loop(std::integral_constant<int, UPW - 1>());

    if (P.ks == 1) {
        T* const out = reinterpret_cast<T*>(P.out) + ((l16 >> 2) * P.Wout + (l16 & 3)) * P.Cout + chan;
        const bool relu = P.relu != 0;
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const int g = wave_m + u * WM;
            if (H.skip[g * 16 + l16]) continue;
            T* px = out + H.uq[g].w;
            if (P.out_origin) {           // the output lies on a torus: the unit may cross its seams
                const int4 og = H.uorg[g];
                const int y = torus_wrap(H.uq[g].y + P.p + (l16 >> 2), og.w, P.Hout), x = torus_wrap(H.uq[g].z + P.p + (l16 & 3), og.z, P.Wout);
                px = reinterpret_cast<T*>(P.out) + ((H.ustream[g] * P.Hout + y) * P.Wout + x) * P.Cout + chan;
            }
#pragma unroll
            for (int j = 0; j < NBW; ++j) {
                floatx4 v = acc[u][j] + bias[j];
                if (relu) activate4(v, P.relu);
                F::store4(px + j * 16, v);
            }
        }
        return;
    }
    // partial sums: [split][unit][pixel][channel]
    float* part = P.partial + (size_t)blockIdx.y * n_units * 16 * P.Cout + (size_t)l16 * P.Cout + chan;
#pragma unroll
    for (int u = 0; u < UPW; ++u) {
        const int g = wave_m + u * WM;
        if (H.ukind[g] < 0) continue;
        float* px = part + (size_t)(ug * P.g_rt + g) * 16 * P.Cout;
#pragma unroll
        for (int j = 0; j < NBW; ++j) *reinterpret_cast<floatx4*>(px + j * 16) = acc[u][j];
    }
}

// ---- 3x3, bf16, tiles of 128 or 256 output channels: a wavefront's weights come straight from L2 ----------------
// conv_fast_kernel stages the weights of a kernel row in LDS, where four wavefronts read each fragment: 7 or 8 LDS reads
// for 12 or 16 MFMAs, a barrier per kernel row, and one workgroup per CU, whose wavefronts reach every barrier together
// (matrix pipes busy in 0.54 of a CU's cycles).  Here a wavefront holds all units of its workgroup against 64 channels of
// its own, so that a weight fragment has one reader and needs no LDS: it is loaded into registers two taps ahead.  Only
// the patches go through LDS (double-buffered, one barrier per 32 channels = nine taps), a fragment of them feeds four
// MFMAs, and two workgroups of four wavefronts (four of two) share a CU out of step: pipes busy in 0.72 of the cycles.
//   workgroup = UPW units x 64 NW channels; wavefront = UPW units x 64 channels (128 accumulator registers for 8 units)
// 56x56 256->256 on 64 streams: 214 -> 175 us (1.35 PFLOP/s issued), 28x28 512->512 199 -> 186, 112x112 128->128 254 -> 222.
// What bounds it now: power (the clock falls to 1.85 GHz) and the look-ups of the weight fragments in the CU's cache, two
// per four lanes in the packed layout (rows of 64 bytes); without any weight loads the first of these takes 153 us, and
// without the LDS reads or the patch loads as long as with them.  Through an LDS ring of each wavefront's own the weights
// took longer (183, 189, 265 us).  The sums are taken in the order of conv_fast_kernel with chunks of 32 channels and no
// split of K: the same bits.
//
// The MFMA as one instruction on a tied accumulator: left to the compiler, a third of them write to other registers than
// they read, and 8 units do not fit.  The compiler does not see an MFMA then, so the wait states before other
// instructions touch the registers are written out where that happens.
__device__ __forceinline__ void mfma_in_place(const bf16x8& a, const bf16x8& b, floatx4& c) {
    asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
template <int NW, int UPW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv_deep_kernel(ConvParams P) {
    typedef __hip_bfloat16 T;
    typedef Frag<T> F;
    typedef F::vec vec;
    constexpr int NBW = 4, NT = NW * NBW * 16, RB = 64, PW = 6, PR = PW * PW;     // channels of a workgroup; a patch row: 32 channels
    constexpr int P_INSTR = (UPW * PR + 15) / 16, NPI = (P_INSTR + NW - 1) / NW, PBYTES = P_INSTR * 1024;
    constexpr int NQ = (UPW + 1) / 2;               // steps of a tap: two units each, whose fragments are read together
    static_assert(UPW >= 2 && UPW <= 8 && NPI <= 10, "fits the registers; patch loads end four taps before the barrier");

    extern __shared__ __align__(16) unsigned char smem[];
    const FastHeader<8> H(smem);                    // (its tables are aligned for even numbers)
    unsigned char* const patch0 = smem + kHeaderBytes;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4;

    int ug, ntile;
    decode_workgroup(P.R, ug, ntile);
    const int n_units = unit_count(P);
    if (ug * P.g_rt >= n_units) return;             // the whole workgroup, before any barrier
    const int n0 = ntile * NT + wave * 64;          // first channel of this wavefront
    const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(keep_scalar(reinterpret_cast<uintptr_t>(P.in))), 0, keep_scalar(P.in_bytes), kBufferFlags);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(keep_scalar(reinterpret_cast<uintptr_t>(P.w))), 0, keep_scalar(P.w_bytes), kBufferFlags);
    const int CinES = P.Cin * 2;
    const int n_ch = keep_scalar(P.n_chunks);

    // Weights: row l16 of MFMA block j carries channel (l16 / 4) * 16 + 4 j + l16 % 4 of the wavefront's 64, so that a
    // lane ends with 16 consecutive channels of a pixel and stores them in 16-byte pieces.
    const bool packed = P.w_packed != 0;
    const int ts = keep_scalar(packed ? 1024 : CinES);               // byte distance of two taps, chunks, blocks
    const int cs = keep_scalar(packed ? 9 * 1024 : RB);
    const int js = keep_scalar(packed ? 4 * 64 : 4 * 9 * CinES);
    const int wch = n0 + (l16 >> 2) * 16 + (l16 & 3);
    const uint32_t wlane = packed ? (uint32_t)(wch / 16 * (n_ch * 9) * 1024 + wch % 16 * 64 + q * 16)
                                  : (uint32_t)(wch * 9 * CinES + q * 16);
    vec w[3][NBW];
    auto load_w = [&](int slot, int soff) {
#pragma unroll
        for (int j = 0; j < NBW; ++j) {
            const int so = soff + j * js;
            w[slot][j] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, wlane, so, 0));
        }
    };
    int wo = 0;                                     // of the current chunk's first tap
    load_w(0, wo);                                  // they travel while the unit table is decoded
    load_w(1, wo + ts);

    decode_units_fast<8, NW * 64, 2>(P, H, ug, tid, n_units);

    // patch loads: 16 rows of 64 bytes each, dealt to the wavefronts in turn.  A patch is 36 rows without gaps; chunk c
    // (16 bytes) of the row at (py, px) sits at position c ^ 2 (py % 2): no bank conflicts for any tap.
    uint32_t pgo[NPI];
    const int lrow = lane >> 2, lpos = lane & 3;
#pragma unroll
    for (int i = 0; i < NPI; ++i) {
        const int row = (wave + i * NW) * 16 + lrow, unit0 = row / PR, r = row - unit0 * PR;
        const int py = r / PW, px = r - py * PW;
        const int unit = unit0 < UPW ? unit0 : UPW - 1;
        const int4 uq = H.uq[unit];
        const int c16 = (lpos ^ (py % 2 * 2)) << 4;
        const bool ok = unit0 < UPW && (unsigned)(uq.y + py) < (unsigned)P.Hin && (unsigned)(uq.z + px) < (unsigned)P.Win;
        uint32_t off = (uint32_t)(uq.x + (py * P.Win + px) * CinES + c16);
        if (P.in_origin && ok) {                    // the input lies on a torus: the patch may cross its seams
            const int4 og = H.uorg[unit];
            const int iy = torus_wrap(uq.y + py, og.y, P.Hin), ix = torus_wrap(uq.z + px, og.x, P.Win);
            off = (uint32_t)(((H.ustream[unit] * P.Hin + iy) * P.Win + ix) * CinES + c16);
        }
        pgo[i] = ok ? off : kOob;
    }
    auto issue_p1 = [&](int i, int so, int pbuf) {
        unsigned char* dst = patch0 + pbuf * PBYTES + (wave + i * NW) * 1024;
        const uint32_t off = pgo[i];
        if ((i + 1) * NW <= P_INSTR || wave + i * NW < P_INSTR)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(in_rsrc, (__attribute__((address_space(3))) void*)dst, 16, off, so, 0, 0);
    };

    int paddr[6];                                   // kernel rows 0 and 1; row 2 is row 0 two lines further down
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        const int py = (l16 >> 2) + t / 3, px = (l16 & 3) + t % 3;
        paddr[t] = (py * PW + px) * RB + ((q ^ (py % 2 * 2)) << 4);
    }
    vec x[2][2];
    auto read_x = [&](int pbuf, int t, int h, int b) {     // step h of tap t
        const int ky = t / 3, kx = t % 3;
        const unsigned char* xp = patch0 + pbuf * PBYTES + paddr[ky % 2 * 3 + kx] + (ky / 2) * (2 * PW * RB);
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (h * 2 + u < UPW) x[b][u] = *reinterpret_cast<const vec*>(xp + (h * 2 + u) * (PR * RB));
    };
    floatx4 acc[UPW][NBW];
#pragma unroll
    for (int u = 0; u < UPW; ++u)
#pragma unroll
        for (int j = 0; j < NBW; ++j) acc[u][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](int h, int b, int slot) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (h * 2 + u < UPW)
#pragma unroll
                for (int j = 0; j < NBW; ++j) mfma_in_place(w[slot][j], x[b][u], acc[h * 2 + u][j]);
    };

#pragma unroll
    for (int i = 0; i < NPI; ++i) issue_p1(i, 0, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    read_x(0, 0, 0, 0);
    asm volatile("s_nop 4");                        // (the accumulators were cleared)
    for (int c = 0; c < n_ch; ++c) {
        const int pbuf = c & 1;
        const bool more = c + 1 < n_ch;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            // (the last chunk's loads beyond its taps fetch weights that nothing uses, or zeros from outside the tensor)
            load_w((t + 2) % 3, t + 2 < 9 ? wo + (t + 2) * ts : wo + cs + (t - 7) * ts);
#pragma unroll
            for (int i = 2 * t; i < 2 * t + 2 && i < NPI; ++i)
                if (more) issue_p1(i, (c + 1) * RB, pbuf ^ 1);
#pragma unroll
            for (int h = 0; h < NQ; ++h) {
                const int b = (t * NQ + h) & 1;
                if (h + 1 < NQ) read_x(pbuf, t, h + 1, b ^ 1);
                else if (t < 8) read_x(pbuf, t + 1, 0, b ^ 1);
                else if (more) {
                    // This wavefront's share of the next patches has landed: at least sixteen weight loads were issued
                    // after them.  Behind the barrier all shares have, and nobody reads the current buffer any more.
                    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
                    lds_barrier();
                    read_x(pbuf ^ 1, 0, 0, b ^ 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                mma(h, b, t % 3);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if ((9 * NQ) & 1) { x[0][0] = x[1][0]; x[0][1] = x[1][1]; asm volatile("s_nop 4"); }   // the next chunk expects its first fragments in buffer 0
        wo += cs;
    }

#pragma unroll
    for (int u = 0; u < UPW; ++u)       // the sums are read by other than MFMAs from here on
        asm volatile("s_nop 15\n\ts_nop 4" : "+v"(acc[u][0]), "+v"(acc[u][1]), "+v"(acc[u][2]), "+v"(acc[u][3]));
    const int chan = n0 + 16 * q;
    floatx4 bias[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j)
        bias[j] = P.bias ? *reinterpret_cast<const floatx4*>(P.bias + chan + j * 4) : floatx4{0.f, 0.f, 0.f, 0.f};
    T* const out = reinterpret_cast<T*>(P.out) + ((l16 >> 2) * P.Wout + (l16 & 3)) * P.Cout + chan;
    const bool relu = P.relu != 0;
#pragma unroll
    for (int u = 0; u < UPW; ++u) {
        if (H.skip[u * 16 + l16]) continue;
        T* px = out + H.uq[u].w;
        if (P.out_origin) {                         // the output lies on a torus: the unit may cross its seams
            const int4 og = H.uorg[u];
            const int y = torus_wrap(H.uq[u].y + P.p + (l16 >> 2), og.w, P.Hout), xo = torus_wrap(H.uq[u].z + P.p + (l16 & 3), og.z, P.Wout);
            px = reinterpret_cast<T*>(P.out) + ((H.ustream[u] * P.Hout + y) * P.Wout + xo) * P.Cout + chan;
        }
        uint32_t v[2 * NBW];
#pragma unroll
        for (int j = 0; j < NBW; ++j) {
            floatx4 sum = acc[u][j] + bias[j];
            if (relu) activate4(sum, P.relu);
            v[2 * j] = (uint32_t)F::bits(sum[0]) | ((uint32_t)F::bits(sum[1]) << 16);
            v[2 * j + 1] = (uint32_t)F::bits(sum[2]) | ((uint32_t)F::bits(sum[3]) << 16);
        }
        *reinterpret_cast<uintx4*>(px) = uintx4{v[0], v[1], v[2], v[3]};
        *reinterpret_cast<uintx4*>(px + 8) = uintx4{v[4], v[5], v[6], v[7]};
    }
}

// ---- 3x3, bf16, small maps of which (nearly) every pixel is computed ----------------------------------------------
// On a 13x13 map the 4x4 units cover 256 pixels for 169, on 14x14 256 for 196: MFMAs, LDS reads and patch loads for
// nothing.  Where nearly every unit has work, a workgroup takes a whole map instead: the rows of the GEMM are the map's
// pixels one after another, 16 to a tile, and the map with its border lies in LDS once (16 slots a line, so maps of up to
// 14x14) where units have a patch each: 15 KB per 32 channels for 11 tiles.
// Everything else is conv_fast_kernel: stages of one kernel row, double buffers, eight wavefronts (four rows of tiles, dealt
// round-robin, x two halves of the channels), and the order of the sums with chunks of 32 channels: the same bits.
// The reusable pixels of a cached frame come from the units' masks, so a list that is shorter than expected costs time only.
// 13x13 384->384 on 64 streams 44 -> 36 us, 512->1024 on 16 streams 36 -> 30, 14x14 512->512 on 64 streams 61 -> 52.  What bounds it:
// a barrier per kernel row at two wavefronts per SIMD (registers allow no more), and few workgroups (192 to 512 for 256 CUs).
// LDS: the row of slot (line, column) at (16 line + column) * 64 bytes, its 16-byte chunk c at c ^ 2 (column / 4 % 2): a read
// of 16 neighbouring pixels of a line is free of conflicts, one across a line's end is not (14x14: 0.29 of the LDS cycles).
template <int UPW, int NBW>
__global__ __launch_bounds__(512) void conv_map_kernel(ConvParams P) {
    typedef __hip_bfloat16 T;
    typedef Frag<T> F;
    typedef F::vec vec;
    constexpr int WM = 4, WN = 2, NW = 8, NT = WN * NBW * 16, RB = 64, KC = 32, LINES = 16, PBYTES = LINES * 1024;
    constexpr int W_INSTR = 3 * NT / 16, NWI = (W_INSTR + NW - 1) / NW, WBYTES = W_INSTR * 1024, NPI = 2;

    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* const patch0 = smem;
    unsigned char* const wts0 = smem + 2 * PBYTES;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_n = wave % WN, wave_m = wave / WN;
    const int l16 = lane & 15, q = lane >> 4;
    int stream, ntile;
    decode_workgroup(P.R, stream, ntile);
    const int n0 = ntile * NT;
    const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(keep_scalar(reinterpret_cast<uintptr_t>(P.in))), 0, keep_scalar(P.in_bytes), kBufferFlags);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(keep_scalar(reinterpret_cast<uintptr_t>(P.w))), 0, keep_scalar(P.w_bytes), kBufferFlags);
    const int CinES = keep_scalar(P.Cin * 2);
    const bool packed = keep_scalar(P.w_packed) != 0;
    const int H = P.Hout, W = P.Wout;

    const int lrow = lane >> 2, lpos = lane & 3;
    uint32_t wgo[NWI];
#pragma unroll
    for (int i = 0; i < NWI; ++i) {
        const int row = (wave + i * NW) * 16 + lrow;   // tl * NT + n
        const int tl = row / NT, n = row - tl * NT;
        const int c = lpos ^ ((row / 2) % 4);
        const uint32_t off = packed ? (uint32_t)((((n0 + n) / 16 * (CinES / 64) * 9 + tl) * 16 + n % 16) * 64 + (c << 4))
                                    : (uint32_t)(((n0 + n) * 9 + tl) * CinES + (c << 4));
        wgo[i] = tl < 3 ? off : kOob;
    }
    auto issue_w = [&](int chunk, int ky, int wbuf) {
        unsigned char* dst = wts0 + wbuf * WBYTES + wave * 1024;
        const int so = packed ? (chunk * 3 + ky) * (3 * 1024) : ky * 3 * CinES + chunk * RB;
#pragma unroll
        for (int i = 0; i < NWI; ++i) {
            const uint32_t off = wgo[i];
            if ((i + 1) * NW <= W_INSTR || wave + i * NW < W_INSTR)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (__attribute__((address_space(3))) void*)(dst + i * (NW * 1024)),
                                                         16, off, so, 0, 0);
        }
    };
    issue_w(0, 0, 0);

    // patch: instruction j brings line j (row j - 1 of the map), a slot per four lanes
    uint32_t pgo[NPI];
    int iox = 0, ioy = 0, oox = 0, ooy = 0;           // tensors on a torus: the stream's origins
    {
        const size_t at = (size_t)stream * P.origin_stride;
        if (P.in_origin) { iox = P.in_origin[at]; ioy = P.in_origin[at + 1]; }
        if (P.out_origin) { oox = P.out_origin[at]; ooy = P.out_origin[at + 1]; }
    }
#pragma unroll
    for (int i = 0; i < NPI; ++i) {
        const int y = wave + i * NW - 1, x = lrow - 1;
        const bool ok = (unsigned)y < (unsigned)H && (unsigned)x < (unsigned)W;
        int iy = y, ix = x;
        if (P.in_origin && ok) { iy = torus_wrap(y, ioy, H); ix = torus_wrap(x, iox, W); }
        pgo[i] = ok ? (uint32_t)(((stream * H + iy) * W + ix) * CinES + ((lpos ^ (lrow / 4 % 2 * 2)) << 4)) : kOob;
    }
    auto issue_p = [&](int chunk, int part, int pbuf) {          // part < 0: all lines, else every third instruction
        unsigned char* dst = patch0 + pbuf * PBYTES + wave * 1024;
        const int so = chunk * RB;
#pragma unroll
        for (int i = 0; i < NPI; ++i) {
            if (part >= 0 && i % 3 != part) continue;
            const uint32_t off = pgo[i];
            if (wave + i * NW < H + 2)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(in_rsrc, (__attribute__((address_space(3))) void*)(dst + i * (NW * 1024)),
                                                         16, off, so, 0, 0);
        }
    };

    // read side: this lane's pixel of every tile of the wavefront; keep: the pixels to be stored
    int paddr[UPW][3];
    unsigned keep = 0;
#pragma unroll
    for (int u = 0; u < UPW; ++u) {
        const int p = (wave_m + u * WM) * 16 + l16;
        const bool in = p < H * W;
        const int y = in ? fast_div(p, P.pw_magic) : 0, x = in ? p - y * W : 0;
        const bool reused = in && P.umask && ((P.umask[(size_t)stream * (P.units_x * P.units_y) + (y >> 2) * P.units_x + (x >> 2)] >> ((y & 3) * 4 + (x & 3))) & 1);
        keep |= in && !reused ? 1u << u : 0u;
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
            paddr[u][kx] = (y * 16 + x + kx) * RB + ((q ^ ((x + kx) / 4 % 2 * 2)) << 4);
    }
    const int waddr = (wave_n * NBW * 16 + l16) * RB + ((q ^ ((l16 / 2) % 4)) << 4);

    floatx4 acc[UPW][NBW];
#pragma unroll
    for (int u = 0; u < UPW; ++u)
#pragma unroll
        for (int j = 0; j < NBW; ++j) acc[u][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int chan = n0 + wave_n * NBW * 16 + 4 * q;
    floatx4 bias[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j)
        bias[j] = P.bias ? *reinterpret_cast<const floatx4*>(P.bias + chan + j * 16) : floatx4{0.f, 0.f, 0.f, 0.f};

    const int n_ch = keep_scalar(P.n_chunks);
    auto issue_stage = [&](int c, int ky, int s) {     // as in conv_fast_kernel
        if (c >= n_ch) return;
        issue_w(c, ky, s & 1);
        if (ky == 0) { if (c > 0) issue_p(c, 2, c & 1); }
        else if (c + 1 < n_ch) issue_p(c + 1, ky - 1, (c + 1) & 1);
    };
    auto main_loop = [&](auto nu_tag) {
        constexpr int NU = decltype(nu_tag)::value;
        vec x[2][NU > 0 ? NU : 1], w[2][NBW];
        auto frag = [&](int pbuf, int wbuf, int ky, int kx, int b) {
            const unsigned char* xp = patch0 + pbuf * PBYTES + ky * 1024;
#pragma unroll
            for (int u = 0; u < NU; ++u) x[b][u] = *reinterpret_cast<const vec*>(xp + paddr[u][kx]);
            const unsigned char* wp = wts0 + wbuf * WBYTES + waddr + kx * (NT * RB);
#pragma unroll
            for (int j = 0; j < NBW; ++j) w[b][j] = *reinterpret_cast<const vec*>(wp + j * (16 * RB));
        };
        auto mma = [&](int b) {
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int j = 0; j < NBW; ++j) F::mma1(w[b][j], x[b][u], acc[u][j], 0);
        };
        issue_p(0, -1, 0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        issue_stage(0, 1, 1);
        frag(0, 0, 0, 0, 0);
        int sidx = 0;
        for (int c = 0; c < n_ch; ++c) {
            const int pbuf = c & 1;
#pragma unroll
            for (int ky = 0; ky < 3; ++ky, ++sidx) {
#pragma unroll
                for (int kx = 0; kx < 2; ++kx) {
                    frag(pbuf, sidx & 1, ky, kx + 1, (ky * 3 + kx + 1) & 1);
                    __builtin_amdgcn_sched_barrier(0);
                    mma((ky * 3 + kx) & 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                if (ky == 0) issue_stage(c, 2, sidx + 2);
                else issue_stage(c + 1, ky - 1, sidx + 2);
                if (ky < 2) frag(pbuf, (sidx + 1) & 1, ky + 1, 0, ((ky + 1) * 3) & 1);
                else if (c + 1 < n_ch) frag(pbuf ^ 1, (sidx + 1) & 1, 0, 0, 1);
                __builtin_amdgcn_sched_barrier(0);
                mma((ky * 3 + 2) & 1);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) x[0][u] = x[1][u];          // nine steps: the next chunk expects its first fragments in buffer 0
#pragma unroll
            for (int j = 0; j < NBW; ++j) w[0][j] = w[1][j];
        }
    };
    const int n_tiles = (H * W + 15) >> 4;
    const int n_u = keep_scalar((n_tiles - wave_m + WM - 1) / WM);
    if (n_u == UPW) main_loop(std::integral_constant<int, UPW>());
    else main_loop(std::integral_constant<int, UPW - 1>());

    const bool relu = P.relu != 0;
#pragma unroll
    for (int u = 0; u < UPW; ++u) {
        if (!((keep >> u) & 1)) continue;
        const int p = (wave_m + u * WM) * 16 + l16;
        int y = fast_div(p, P.pw_magic), x = p - y * W;
        if (P.out_origin) { y = torus_wrap(y, ooy, H); x = torus_wrap(x, oox, W); }
        T* px = reinterpret_cast<T*>(P.out) + ((stream * H + y) * W + x) * P.Cout + chan;
#pragma unroll
        for (int j = 0; j < NBW; ++j) {
            floatx4 v = acc[u][j] + bias[j];
            if (relu) activate4(v, P.relu);
            F::store4(px + j * 16, v);
        }
    }
}

// Adds the partial sums of the ks workgroups of every tile in a fixed order and applies the epilogue.
// One thread per (unit, pixel, four channels).
template <typename T>
__global__ __launch_bounds__(256) void conv_split_reduce_kernel(ConvParams P) {
    typedef Frag<T> F;
    const int c4n = P.Cout >> 2;
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int n_units = unit_count(P);
    const size_t total = (size_t)n_units * 16 * c4n;
    if (idx >= total) return;
    const int co = (int)(idx % c4n) * 4;
    const size_t pix = idx / c4n;
    const int l16 = (int)(pix & 15), u = (int)(pix >> 4);
    int stream, uy, ux, mixed = 0;
    if (P.units) {
        const TileDev t = P.units[u];
        stream = t.stream; uy = t.ty; ux = t.tx; mixed = t.reuse_mask;
    } else {
        const int per = P.units_x * P.units_y;
        stream = u / per;
        const int r = u - stream * per;
        uy = r / P.units_x; ux = r - uy * P.units_x;
    }
    const int y = uy * 4 + (l16 >> 2), x = ux * 4 + (l16 & 3);
    if (y >= P.Hout || x >= P.Wout) return;
    if ((mixed >> l16) & 1) return;   // keeps the copied value
    const size_t split_stride = (size_t)n_units * 16 * P.Cout;
    const float* p = P.partial + pix * P.Cout + co;
    floatx4 v = *reinterpret_cast<const floatx4*>(p);
    for (int s = 1; s < P.ks; ++s) v += *reinterpret_cast<const floatx4*>(p + s * split_stride);
    if (P.bias) v += *reinterpret_cast<const floatx4*>(P.bias + co);
    if (P.relu) activate4(v, P.relu);
    int yo = y, xo = x;
    if (P.out_origin) {
        xo = torus_wrap(x, P.out_origin[(size_t)stream * P.origin_stride], P.Wout);
        yo = torus_wrap(y, P.out_origin[(size_t)stream * P.origin_stride + 1], P.Hout);
    }
    T* out = reinterpret_cast<T*>(P.out) + (((size_t)stream * P.Hout + yo) * P.Wout + xo) * P.Cout + co;
    F::store4(out, v);
}

constexpr int kRegwTorusStreams = 2048;      // streams whose origins fit a kernel's LDS table (16 KB)

// ---- 3x3, 64 input channels, bf16: the weights live in registers -----------------------------
// K is only 576, so a workgroup of the kernel above spends more time on its prologue and epilogue than on its
// six stages.  Here a wavefront keeps the weights of its 32 output channels for the whole K in registers
// (9 taps x 2 K groups x 2 channel blocks = 36 fragments, 144 registers), the workgroups are persistent
// (one per CU and channel tile) and walk over the unit list; per step only the patches of the next G units
// travel (buffer_load ... lds into the other half of a double buffer) while the current ones are multiplied.
// There is no unit table in LDS: the two wavefronts that share a row of units (they differ in the channel
// half) also load exactly those units' patches, half each, so everything a wavefront needs to know about a
// unit is wavefront-uniform and lives in registers; the unit list entries are fetched two steps ahead.
//   workgroup = 8 wavefronts = 4 unit rows x 2 channel halves; step = G = 4 * UPW units x 64 channels
//   LDS       = 2 x G patches of 6 lines x 8 slots x 128 bytes (layout and swizzle of the kernel above)
struct UnitRegs {
    int in_base;    // byte offset in the input of the patch origin
    int oy, ox;     // row / column of that origin (may be negative); oy = -2^24 for a missing unit
    int out_base;   // element offset in the output of the unit's first pixel
    int kind;       // -1: missing unit, else the 16-bit mask of reusable pixels
    // tensors on a torus only (in_base and out_base are not used then): the unit's stream and the origins of that
    // stream in the input and in the output, column | row << 16
    int stream, iorg, oorg;
};

// The unit list entry of unit u (or its raster position), not yet turned into offsets: fetched two steps ahead.
__device__ __forceinline__ TileDev regw_fetch(const ConvParams& P, long u, int n_units) {
    TileDev t{0, 0, 0, -1};                 // reuse_mask -1: no such unit
    if (u >= n_units) return t;
    if (P.units) return P.units[u];
    t.stream = fast_div_any((int)u, P.npix_magic, P.units_x * P.units_y);
    const int rem = (int)u - t.stream * (P.units_x * P.units_y);
    t.ty = fast_div(rem, P.pw_magic); t.tx = rem - t.ty * P.units_x;
    t.reuse_mask = 0;
    return t;
}
// origins: the streams' origins in LDS, {input, output} as column | row << 16 (a load from memory here would depend on
// the list entry and stall every step for a round trip)
template <bool TORUS>
__device__ __forceinline__ UnitRegs regw_unit(const ConvParams& P, const TileDev& t, const int2* origins) {
    UnitRegs r;
    if (TORUS) {
        const int2 og = origins[t.stream];
        r.iorg = __builtin_amdgcn_readfirstlane(og.x);
        r.oorg = __builtin_amdgcn_readfirstlane(og.y);
        r.stream = t.stream;
    }
    const bool valid = t.reuse_mask != -1;
    const int oy = t.ty * 4 - P.p, ox = t.tx * 4 - P.p;
    r.in_base = ((t.stream * P.Hin + oy) * P.Win + ox) * P.Cin * 2;
    r.oy = valid ? oy : -(1 << 24);
    r.ox = ox;
    r.out_base = ((t.stream * P.Hout + t.ty * 4) * P.Wout + t.tx * 4) * P.Cout;
    r.kind = valid ? (t.reuse_mask & 0xffff) : -1;
    return r;
}

template <int WM, int UPW, bool TORUS>
__global__ __launch_bounds__(WM * 128) __attribute__((amdgpu_waves_per_eu(2))) void conv_regw_kernel(ConvParams P) {
    typedef Frag<__hip_bfloat16> F;
    typedef F::vec vec;
    constexpr int WN = 2, NBW = 2, G = WM * UPW;
    constexpr int RB = 128, PWP = 8, PR = 48;
    constexpr int PBYTES = G * PR * RB;

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_n = wave % WN, wave_m = wave / WN;
    const int l16 = lane & 15, q = lane >> 4;
    const int n0 = (int)blockIdx.y * 64 + wave_n * 32;          // first output channel of this wavefront
    const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(keep_scalar(reinterpret_cast<uintptr_t>(P.in))), 0, keep_scalar(P.in_bytes), kBufferFlags);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void*>(keep_scalar(reinterpret_cast<uintptr_t>(P.w))), 0, keep_scalar(P.w_bytes), kBufferFlags);

    // weights [cout][3][3][64]: fragment (tap, K group g, block j) of lane (l16, q) = 8 channels from g*32 + q*8
    vec wreg[9][2][NBW];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int j = 0; j < NBW; ++j) {
                const uint32_t off = (uint32_t)((((n0 + j * 16 + l16) * 9 + t) * 64 + g * 32 + q * 8) * 2);
                wreg[t][g][j] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, off, 0, 0));
            }
    const int chan = n0 + 4 * q;
    floatx4 bias[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j)
        bias[j] = P.bias ? *reinterpret_cast<const floatx4*>(P.bias + chan + j * 16) : floatx4{0.f, 0.f, 0.f, 0.f};
    // ReLU on the bit pattern: a float with the sign bit set is a negative integer, so max(bits, 0) as integers
    // clears exactly the negative values; without ReLU the floor is the smallest integer and changes nothing
    const int relu_floor = P.relu ? 0 : (int)0x80000000;

    // load side: of each of its units this wavefront brings lines 3 * wave_n .. 3 * wave_n + 2 (one instruction per
    // line: 8 slots x 128 bytes); the lane fills chunk position lane % 8 of slot lane / 8.  Everything that does
    // not depend on the unit is computed once: the step's address work is one add and one select per instruction.
    const int px_l = lane >> 3, lpos = lane & 7;
    const int CinES = 128;
    const int line_bytes = P.Win * CinES;
    int lane_off[3];   // on a torus without the line and the column: they depend on the stream's origin
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int py = wave_n * 3 + i;
        lane_off[i] = (TORUS ? 0 : py * line_bytes + px_l * CinES) + ((lpos ^ patch_swizzle<RB>(py, px_l)) << 4);
    }
    const int Hin = keep_scalar(P.Hin), Win = keep_scalar(P.Win);
    auto issue_p = [&](const UnitRegs (&info)[UPW], int buf) {
#pragma unroll
        for (int uu = 0; uu < UPW; ++uu) {
            // columns: slot px_l is inside the map iff 0 <= ox + px_l < Win (slots 6 and 7 are never used)
            const bool col_ok = px_l < 6 && (unsigned)(info[uu].ox + px_l) < (unsigned)Win;
            int col_off = 0;
            if (TORUS) col_off = torus_wrap(info[uu].ox + px_l, info[uu].iorg & 0xffff, Win) * CinES;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int py = wave_n * 3 + i;
                const bool row_ok = (unsigned)(info[uu].oy + py) < (unsigned)Hin;       // wavefront-uniform
                int base = info[uu].in_base;
                if (TORUS) base = (info[uu].stream * Hin + torus_wrap(info[uu].oy + py, info[uu].iorg >> 16, Hin)) * line_bytes + col_off;
                const uint32_t off = (col_ok && row_ok) ? (uint32_t)(base + lane_off[i]) : kOob;
                unsigned char* dst = smem + buf * PBYTES + ((wave_m + uu * WM) * PR + py * PWP) * RB;
                // the lanes of slots 6 and 7 sit the load out: a quarter less for the address unit, whose queue
                // is what the wavefronts of this kernel wait for when they issue their loads
                if (px_l < 6)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(in_rsrc, (__attribute__((address_space(3))) void*)dst, 16, off, 0, 0, 0);
            }
        }
    };
    // read side: byte address of this lane's row and chunk for every tap and K group
    int paddr[9][2];
    {
        const int oy = l16 >> 2, ox = l16 & 3;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int py = oy + t / 3, px = ox + t % 3;
            const int sw = patch_swizzle<RB>(py, px);
#pragma unroll
            for (int g = 0; g < 2; ++g) paddr[t][g] = (wave_m * PR + py * PWP + px) * RB + (((g * 4 + q) ^ sw) << 4);
        }
    }

    const int2* const origins = reinterpret_cast<const int2*>(smem + 2 * PBYTES);
    if (TORUS) {
        int2* const table = reinterpret_cast<int2*>(smem + 2 * PBYTES);
        for (int s = tid; s < P.n_streams; s += WM * 128) {
            const size_t at = (size_t)s * P.origin_stride;
            table[s] = int2{P.in_origin ? P.in_origin[at] | (P.in_origin[at + 1] << 16) : 0,
                            P.out_origin ? P.out_origin[at] | (P.out_origin[at + 1] << 16) : 0};
        }
        __syncthreads();
    }
    const int n_units = unit_count(P);
    const long n_groups = ((long)n_units + G - 1) / G;
    const long stride = gridDim.x;
    // Workgroup b runs on XCD b % 8.  In every pass over the list the workgroups of one XCD take consecutive
    // groups, so that the units above and below (a row of units further in the list) are in the same L2 at about
    // the same time and the halo rows are fetched from HBM once.
    const long first = (gridDim.x % 8 == 0) ? (long)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8 : (long)blockIdx.x;
    auto fetch = [&](long ug, TileDev (&raw)[UPW]) {
#pragma unroll
        for (int uu = 0; uu < UPW; ++uu) raw[uu] = regw_fetch(P, ug < n_groups ? ug * G + wave_m + uu * WM : (long)n_units, n_units);
    };
    auto decode = [&](const TileDev (&raw)[UPW], UnitRegs (&info)[UPW]) {
#pragma unroll
        for (int uu = 0; uu < UPW; ++uu) info[uu] = regw_unit<TORUS>(P, raw[uu], origins);
    };
    UnitRegs cur[UPW], nxt[UPW];
    TileDev raw[UPW];
    long ug = first;
    fetch(ug, raw); decode(raw, cur);
    fetch(ug + stride, raw); decode(raw, nxt);
    fetch(ug + 2 * stride, raw);             // decoded at the end of the first step
    issue_p(cur, 0);
    // results of the previous step, stored one step late: the wait for this step's patches at the top of the
    // loop would otherwise also wait for the stores just issued
    uintx2 pend[UPW][NBW];
    __hip_bfloat16* pend_px[UPW];
    bool pend_on[UPW];
#pragma unroll
    for (int uu = 0; uu < UPW; ++uu) pend_on[uu] = false;
    auto flush = [&]() {
#pragma unroll
        for (int uu = 0; uu < UPW; ++uu) {
            if (!pend_on[uu]) continue;
#pragma unroll
            for (int j = 0; j < NBW; ++j) *reinterpret_cast<uintx2*>(pend_px[uu] + j * 16) = pend[uu][j];
        }
    };
    for (int it = 0; ug < n_groups; ug += stride, ++it) {
        const int buf = it & 1;
        // the patches of this step have arrived; after the barrier every wavefront is done with the other buffer,
        // which the next step's patches may overwrite
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (ug + stride < n_groups) issue_p(nxt, buf ^ 1);
        flush();

        floatx4 acc[UPW][NBW];                     // start from the bias
#pragma unroll
        for (int uu = 0; uu < UPW; ++uu)
#pragma unroll
            for (int j = 0; j < NBW; ++j) acc[uu][j] = bias[j];
        const unsigned char* pbase = smem + buf * PBYTES;
        // 18 steps (tap, K group); the fragments of step s + 2 are read before the MFMAs of step s
        vec x[3][UPW];
        auto frag = [&](int st, int b) {
#pragma unroll
            for (int uu = 0; uu < UPW; ++uu)
                x[b][uu] = *reinterpret_cast<const vec*>(pbase + paddr[st / 2][st % 2] + uu * (WM * PR * RB));
        };
        frag(0, 0);
        frag(1, 1);
#pragma unroll
        for (int st = 0; st < 18; ++st) {
            if (st + 2 < 18) frag(st + 2, (st + 2) % 3);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int uu = 0; uu < UPW; ++uu)
#pragma unroll
                for (int j = 0; j < NBW; ++j) F::mma1(wreg[st / 2][st % 2][j], x[st % 3][uu], acc[uu][j], 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        // epilogue: pixel l16 of the unit, channels chan + 16 j .. + 3
#pragma unroll
        for (int uu = 0; uu < UPW; ++uu) {
            const int y = cur[uu].oy + P.p + (l16 >> 2), x = cur[uu].ox + P.p + (l16 & 3);
            pend_on[uu] = !(cur[uu].kind < 0 || y >= P.Hout || x >= P.Wout || ((cur[uu].kind >> l16) & 1));
            if (TORUS) {
                const int yw = torus_wrap(pend_on[uu] ? y : 0, cur[uu].oorg >> 16, P.Hout), xw = torus_wrap(pend_on[uu] ? x : 0, cur[uu].oorg & 0xffff, P.Wout);
                pend_px[uu] = reinterpret_cast<__hip_bfloat16*>(P.out) + ((cur[uu].stream * P.Hout + yw) * P.Wout + xw) * P.Cout + chan;
            } else
            pend_px[uu] = reinterpret_cast<__hip_bfloat16*>(P.out) + cur[uu].out_base +
                          ((l16 >> 2) * P.Wout + (l16 & 3)) * P.Cout + chan;
#pragma unroll
            for (int j = 0; j < NBW; ++j) {
                floatx4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {      // negative values (sign bit set) are negative integers
                    const int b = __float_as_int(acc[uu][j][e]);
                    v[e] = __int_as_float(b > relu_floor ? b : relu_floor);
                }
                pend[uu][j][0] = (uint32_t)F::bits(v[0]) | ((uint32_t)F::bits(v[1]) << 16);
                pend[uu][j][1] = (uint32_t)F::bits(v[2]) | ((uint32_t)F::bits(v[3]) << 16);
            }
        }
#pragma unroll
        for (int uu = 0; uu < UPW; ++uu) cur[uu] = nxt[uu];
        decode(raw, nxt);                        // the entries fetched a step ago
        fetch(ug + 3 * stride, raw);             // for the step after next
    }
    flush();
}

// dst vector idx = (((blk * nc64 + c64) * 9 + tap) * 16 + n16) * 4 + v  <-  src row (blk * 16 + n16, tap), 64-byte chunk c64
__global__ __launch_bounds__(256) void pack_weights_kernel(const uintx4* src, uintx4* dst, int nc64, size_t n_vec) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n_vec) return;
    const int v = (int)(idx % 4), n16 = (int)((idx / 4) % 16), tap = (int)((idx / 64) % 9);
    const size_t rest = idx / 576;
    const int c64 = (int)(rest % nc64);
    const size_t blk = rest / nc64;
    dst[idx] = src[((blk * 16 + n16) * 9 + tap) * ((size_t)nc64 * 4) + (size_t)c64 * 4 + v];
}

// ---- 1x1 convolutions ----------------------------------------------------------------------------
// A 1x1 layer is a plain GEMM [pixels][Cin] x [Cin][Cout] with nothing to reuse between taps, so it is bound by
// memory (large maps, small K) or by the latency of its K loop (small maps, deep K: a stage is 16 KiB of loads
// for 8 MFMAs per wavefront).  A workgroup of four wavefronts takes 4 units (64 pixels) x 64 channels and walks K
// in chunks of 128 bytes per row through a ring of up to four LDS stages that are filled three chunks ahead
// (buffer_load ... lds, one barrier per chunk); with 16 KiB per stage several workgroups share a CU and cover
// each other's waits.  With many units the tile is 8 units x 128 channels on eight wavefronts (WM = 4): half the
// bytes from L2 per multiply-add, which is what bounds the kernel then.  Rows of 128 bytes, chunk c of row r at position c ^ (r / 2) % 8: the 16 rows a fragment
// read touches spread over all banks.  Stride 1 or 2 (a strided 1x1 projection reads every second pixel).
// Weight row l16 of block j of a wavefront (NBW blocks) carries channel (l16 / 4) * 4 NBW + 4 j + l16 % 4 of its
// 16 NBW, so that a lane ends up with 4 NBW consecutive channels of one pixel and stores them in 16-byte pieces.
// Cin only has to be a whole number of 16-byte vectors (the last chunk is filled with zeros), Cout a multiple of 8.
// Workgroups are numbered so that the channel tiles of one unit group run on the same XCD at about the same time:
// the second to last of them find the input pixels in that XCD's L2; the groups go round the XCDs.
// What a short launch waits for is its chain of loads, so the list entries are fetched together with the list's length and
// the bias while the unit table is made, and no load is waited for between the stores.  The 15 layer shapes of ResNet-50 on
// 1 / 16 / 64 streams in bf16, us in all: 107.9 -> 93.2, 179.7 -> 163.4, 450.7 -> 420.9; fp32 on 1 / 6 / 16: 117.1 -> 116.2, 276.7 -> 269.9,
// 489.0 -> 477.1; no shape takes longer.  (The first weights ahead of the unit table as well: 95.9, 163.7, 426.6 and 117.2, 273.6, 484.4, with
// 56x56 64->256 in fp32 on 6 streams at 16 us for 15: they delay the patches, which take longer to come.)
//
// ADD: the layer is followed by the element-wise sum of its output with another tensor (a residual block's end), and the
// sum is written here as well: the convolution's output is rounded as it is stored and summed as the sum's own kernel
// does (ResNet-50 on one stream, frame after frame without stages: 497 -> 462 us, on 16 streams 874 -> 830).  Where a pixel is reusable its output is the copied value, fetched beside the other summand while K is walked.
// Units without work stand behind the others in the list (plan_lists_kernel); a group of them only adds.
constexpr int kPwHeaderBytes = 2048;
template <typename T, int WM, bool ADD>
__device__ __forceinline__ void conv_pw_body(const ConvParams& P, const int block) {
    typedef Frag<T> F;
    typedef typename F::vec vec;
    constexpr int ES = (int)sizeof(T), VE = F::VE;
    constexpr int RB = 128, KC = RB / ES, GPC = 2;
    constexpr int UPW = 2, NBW = WM, WN = 2, NW = WM * WN, NSTG = 4;
    constexpr int G = WM * UPW, NT = WN * NBW * 16;   // WM = 2: 4 units x 64 channels; WM = 4: 8 units x 128 channels
    constexpr int PBYTES = G * 16 * RB;             // patch rows of a stage, then the weight rows
    constexpr int STAGE = PBYTES + NT * RB;
    constexpr int D = NSTG - 1;                     // chunks in flight ahead of the one being multiplied
    static_assert(WM == 2 || WM == 4, "two patch and two weight load instructions per wavefront and stage");

    extern __shared__ __align__(16) unsigned char smem[];
    int4* const uq = reinterpret_cast<int4*>(smem);                   // [G] {stream, row, column of the unit, its reuse mask; -1: none}
    int2* const px = reinterpret_cast<int2*>(smem + 128);             // [16 G] byte offset in the input, element offset in the output
    unsigned char* const px_skip = smem + 1152;                       // [16 G] 1: not stored; 3: no such pixel
    const float* const bias_at = reinterpret_cast<const float*>(smem + 1280);     // [NT]
    unsigned char* const ring = smem + kPwHeaderBytes;
    static_assert(G <= 8 && NT <= 128, "tables");

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_n = wave % WN, wave_m = wave / WN;
    const int l16 = lane & 15, q = lane >> 4;

    const int xj = (block >> 3) / P.R, ntile = (block >> 3) - xj * P.R;
    const int ug = xj * 8 + (block & 7);
    const int n_cap = P.n_units;                    // what the launch is sized for
    if (ug * G >= n_cap) return;                    // the whole workgroup, before any barrier
    TileDev td{0, 0, 0, 0};
    if (tid < G && P.units && ug * G + tid < n_cap) td = P.units[ug * G + tid];     // (beyond the list's length: not used)
    const int n_work = unit_count(P), n_units = ADD ? n_cap : n_work;
    const bool gemm = !ADD || ug * G < n_work;      // (ADD) some unit of this group has a pixel to compute
    if (!ADD && ug * G >= n_work) return;
    const int n0 = ntile * NT;
    const int CinES = P.Cin * ES;
    const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.in), 0, P.in_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.w), 0, P.w_bytes, kBufferFlags);

    // load side: instruction j of a stage fills its LDS bytes [1024 j, 1024 j + 1024) = rows 8 j .. 8 j + 7; this
    // wavefront issues j = wave and wave + NW of the patch rows and of the weight rows
    const int lrow = lane >> 3, lpos = lane & 7;
    uint32_t pgo[2], wgo[2];
    int lch[2];                                     // first channel (within a chunk) of the vector the lane fetches
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (wave + i * NW) * 8 + lrow;
        const int c = lpos ^ ((row >> 1) & 7);
        lch[i] = c * VE;
        const int ch = n0 + row / (NBW * 16) * (NBW * 16) + ((row & 15) >> 2) * (4 * NBW) + ((row >> 4) % NBW) * 4 + (row & 3);
        wgo[i] = ch < P.Cout ? (uint32_t)(ch * CinES + (c << 4)) : kOob;
    }
    // Every unit group starts its walk over K at another chunk: rows are Cin * ES bytes apart, a power of two for
    // most layers, so workgroups that all read chunk c of their rows at the same time would all hit the few memory
    // channels those addresses map to.
    const int n_ch = P.n_chunks;
    const int start = ug % n_ch;
    auto chunk_of = [&](int c) { const int cc = start + c; return cc < n_ch ? cc : cc - n_ch; };
    // The bias goes to LDS, ahead of every other load (fetched in the epilogue it would wait for the stores before it; 16 more
    // registers leave room for two workgroups of eight wavefronts on a CU instead of three: 56x56 64->256 on 64 streams 31 -> 35 us).
    const int chan0 = n0 + wave_n * (NBW * 16) + q * (4 * NBW);
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(P.bias), 0, P.bias ? P.Cout * 4 : 0, kBufferFlags);
    if (gemm && wave < NT / 64)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, (__attribute__((address_space(3))) void*)(smem + 1280 + wave * 256), 4,
                                                 (uint32_t)((n0 + wave * 64 + lane) * 4), 0, 0, 0);
    asm volatile("" ::: "memory");

    // tables of the group's units and pixels
    if (tid < G) {
        const int u = ug * G + tid;
        int4 v{0, 0, 0, -1};
        if (u < n_units && P.units) {
            v = int4{td.stream, td.ty, td.tx, td.reuse_mask & 0xffff};
        } else if (u < n_units) {   // raster order
            v.x = fast_div_any(u, P.npix_magic, P.units_x * P.units_y);
            const int r = u - v.x * (P.units_x * P.units_y);
            v.y = fast_div(r, P.pw_magic); v.z = r - v.y * P.units_x; v.w = 0;
        }
        uq[tid] = v;
    }
    lds_barrier();
    if (tid < G * 16) {
        const int4 u = uq[tid >> 4];
        const int stream = u.x, y = u.y * 4 + ((tid >> 2) & 3), x = u.z * 4 + (tid & 3);
        const int skip = u.w < 0 || y >= P.Hout || x >= P.Wout ? 3 : (u.w >> (tid & 15)) & 1;
        int iy = y * P.s, ix = x * P.s, oy = y, ox = x;
        if ((P.in_origin || P.out_origin) && !(skip & 2)) {      // tensors on a torus (stride 1 only: the launcher sees to it)
            const size_t at = (size_t)stream * P.origin_stride;
            if (P.in_origin) { ix = torus_wrap(x, P.in_origin[at], P.Win); iy = torus_wrap(y, P.in_origin[at + 1], P.Hin); }
            if (P.out_origin) { ox = torus_wrap(x, P.out_origin[at], P.Wout); oy = torus_wrap(y, P.out_origin[at + 1], P.Hout); }
        }
        px[tid] = int2{((stream * P.Hin + iy) * P.Win + ix) * CinES, ((stream * P.Hout + oy) * P.Wout + ox) * P.Cout};
        px_skip[tid] = (unsigned char)skip;
    }
    lds_barrier();

#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (wave + i * NW) * 8 + lrow;
        const int c = lpos ^ ((row >> 1) & 7);
        pgo[i] = px_skip[row] & 2 ? kOob : (uint32_t)px[row].x + (uint32_t)(c << 4);
    }
    auto issue = [&](int chunk, int slot) {
        unsigned char* dst = ring + slot * STAGE + wave * 1024;
#pragma unroll
        for (int i = 0; i < 4; ++i) {               // the patch rows, then the weight rows
            const bool in_k = chunk * KC + lch[i % 2] < P.Cin;
            const uint32_t off = in_k ? (i < 2 ? pgo[i % 2] : wgo[i % 2]) + (uint32_t)(chunk * RB) : kOob;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(i < 2 ? in_rsrc : w_rsrc,
                                                     (__attribute__((address_space(3))) void*)(dst + i / 2 * PBYTES + i % 2 * (NW * 1024)),
                                                     16, off, 0, 0, 0);
        }
    };

    // (ADD) the other summand, and the copied values of reusable pixels: older than the patch loads, so that no count
    // of outstanding loads below includes them
    constexpr int NV = NBW * 4 / VE;                // 16-byte vectors of a lane's channels
    uintx4 other[ADD ? UPW : 1][NV], kept[ADD ? UPW : 1][NV];
    if constexpr (ADD) {
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const int row = (wave_m * UPW + u) * 16 + l16, skip = px_skip[row];
            const int at = px[row].y + chan0;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const bool in = !(skip & 2) && chan0 + v * VE < P.Cout;
                other[u][v] = kept[u][v] = uintx4{0, 0, 0, 0};
                if (in) other[u][v] = *reinterpret_cast<const uintx4*>(static_cast<const T*>(P.add_in) + at + v * VE);
                if (in && (skip & 1)) kept[u][v] = *reinterpret_cast<const uintx4*>(static_cast<const T*>(P.out) + at + v * VE);
            }
        }
        asm volatile("" ::: "memory");              // they leave now
    }

    // read side
    const int sw = (l16 >> 1) & 7;
    int xaddr[GPC], waddr[GPC];
#pragma unroll
    for (int g = 0; g < GPC; ++g) {
        xaddr[g] = (wave_m * UPW * 16 + l16) * RB + (((g * 4 + q) ^ sw) << 4);
        waddr[g] = PBYTES + (wave_n * NBW * 16 + l16) * RB + (((g * 4 + q) ^ sw) << 4);
    }
    floatx4 acc[UPW][NBW];
#pragma unroll
    for (int u = 0; u < UPW; ++u)
#pragma unroll
        for (int j = 0; j < NBW; ++j) acc[u][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    if (gemm) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < n_ch) issue(chunk_of(d), d);
    }
    for (int c = 0; gemm && c < n_ch; ++c) {
        // the loads of chunk c are complete when at most the later chunks' (4 instructions each) are outstanding
        const int ahead = n_ch - 1 - c < D - 1 ? n_ch - 1 - c : D - 1;
        if (ahead >= 2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else if (ahead == 1) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();                              // chunk c is in LDS; everyone is done with chunk c - 1
        if (c + D < n_ch) issue(chunk_of(c + D), (c + D) % NSTG);
        const unsigned char* sb = ring + (c % NSTG) * STAGE;
#pragma unroll
        for (int g = 0; g < GPC; ++g) {
            vec x[UPW], w[NBW];
#pragma unroll
            for (int u = 0; u < UPW; ++u) x[u] = *reinterpret_cast<const vec*>(sb + xaddr[g] + u * (16 * RB));
#pragma unroll
            for (int j = 0; j < NBW; ++j) w[j] = *reinterpret_cast<const vec*>(sb + waddr[g] + j * (16 * RB));
#pragma unroll
            for (int e = 0; e < F::NE; ++e)
#pragma unroll
                for (int u = 0; u < UPW; ++u)
#pragma unroll
                    for (int j = 0; j < NBW; ++j) F::mma1(w[j], x[u], acc[u][j], e);
        }
    }

    floatx4 b[NBW];
#pragma unroll
    for (int j = 0; j < NBW; ++j) b[j] = *reinterpret_cast<const floatx4*>(bias_at + (chan0 - n0) + j * 4);
    // The compiler's own waits for the early loads end here: between the stores they would wait for those too.
    if constexpr (ADD)
#pragma unroll
        for (int u = 0; u < UPW; ++u)
#pragma unroll
            for (int v = 0; v < NV; ++v) asm volatile("" : "+v"(other[u][v]), "+v"(kept[u][v]));
    // a lane holds 4 NBW consecutive channels of each of its pixels
    if (chan0 >= P.Cout) return;
    const bool relu = P.relu != 0;
#pragma unroll
    for (int u = 0; u < UPW; ++u) {
        const int row = (wave_m * UPW + u) * 16 + l16, skip = px_skip[row];
        if (ADD ? skip & 2 : skip) continue;
        const int at = px[row].y + chan0;
        T* const out = reinterpret_cast<T*>(P.out) + at;
#pragma unroll
        for (int v = 0; v < NV; ++v) {              // 16 bytes at a time: eight bf16 or four fp32 channels
            if (chan0 + v * VE >= P.Cout) break;
            uintx4 bits;
            if constexpr (sizeof(T) == 2) {
                floatx4 v0 = acc[u][2 * v] + b[2 * v], v1 = acc[u][2 * v + 1] + b[2 * v + 1];
                if (relu) { activate4(v0, P.relu); activate4(v1, P.relu); }
                bits[0] = (uint32_t)F::bits(v0[0]) | ((uint32_t)F::bits(v0[1]) << 16);
                bits[1] = (uint32_t)F::bits(v0[2]) | ((uint32_t)F::bits(v0[3]) << 16);
                bits[2] = (uint32_t)F::bits(v1[0]) | ((uint32_t)F::bits(v1[1]) << 16);
                bits[3] = (uint32_t)F::bits(v1[2]) | ((uint32_t)F::bits(v1[3]) << 16);
            } else {
                floatx4 v0 = acc[u][v] + b[v];
                if (relu) activate4(v0, P.relu);
                bits = __builtin_bit_cast(uintx4, v0);
            }
            if (!ADD || !skip) *reinterpret_cast<uintx4*>(out + v * VE) = bits;
            if constexpr (ADD) {
                if (skip) bits = kept[u][v];
                const uintx4 o = other[u][v];
                auto sum = [&](float x, float y) { const float t = x + y; return !P.add_relu || t > 0.f ? t : 0.f; };
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (sizeof(T) == 2) {
                        const float lo = sum(__uint_as_float(bits[e] << 16), __uint_as_float(o[e] << 16));
                        const float hi = sum(__uint_as_float(bits[e] & 0xffff0000u), __uint_as_float(o[e] & 0xffff0000u));
                        bits[e] = (uint32_t)F::bits(lo) | ((uint32_t)F::bits(hi) << 16);
                    } else {
                        bits[e] = __float_as_uint(sum(__uint_as_float(bits[e]), __uint_as_float(o[e])));
                    }
                }
                *reinterpret_cast<uintx4*>(static_cast<T*>(P.add_out) + at + v * VE) = bits;
            }
        }
    }
}
template <typename T, int WM>
__global__ __launch_bounds__(WM * 128) void conv_pw_kernel(ConvParams P) { conv_pw_body<T, WM, false>(P, (int)blockIdx.x); }
template <typename T, int WM>
__global__ __launch_bounds__(WM * 128) void conv_pw_add_kernel(ConvParams P) { conv_pw_body<T, WM, true>(P, (int)blockIdx.x); }
// Several 1x1 layers that read one tensor, in one launch: workgroups first[j] .. first[j + 1] - 1 are those that layer j's own launch
// would have (whole rounds of the XCDs each), so the sums are the same.  An inception module's branches have 32 to 600
// workgroups of a few us each, less than the chip holds: alone, each branch pays for a launch and for its own chain of loads.
// GoogLeNet 224x224, ten frames in bf16, 1 / 4 / 16 / 64 streams: 2458 / 2458 / 3630 / 9184 us -> 2247 / 2356 / 3341 / 8804;
// fp32, 16 streams, where the tiles fill the chip and the matrix pipes are the bound: 7839 -> 7817.
struct PwMany {
    ConvParams p[kConvBatch];
    int first[kConvBatch];
};
template <typename T, int WM>
__global__ __launch_bounds__(WM * 128) void conv_pw_many_kernel(PwMany M) {
    const int b = (int)blockIdx.x;
    int j = 0;
#pragma unroll
    for (int i = 1; i < kConvBatch; ++i) j += b >= M.first[i] ? 1 : 0;
    conv_pw_body<T, WM, false>(M.p[j], b - M.first[j]);
}
constexpr int kPwManyId = 464;        // kernel ids: + 2 for the 128 x 128 tile + bf16
constexpr int kPwAddId = 440;         // kernel ids: + 2 for the 128 x 128 tile + bf16

constexpr int kPwSplit = 4;           // wavefronts that share a tile's K
constexpr int kPwSplitId = 400;       // kernel ids: + units - 1

// ---- fp32 1x1 convolutions of few units -----------------------------------------------------------
// With few (unit group, channel tile) pairs the ring above leaves most CUs idle and the others with a serial walk over K, bound by
// the fp32 MFMAs of a lone workgroup and by what one CU fetches.  Here the WK wavefronts of a workgroup split K among
// themselves and each fetches the fragments of its part straight into registers, so every operand byte of the tile is loaded
// once, all loads of a part are in flight together and nothing waits for another wavefront before the partial tiles are added
// through LDS (in the order of the wavefronts).  Wavefront w takes the 128-byte pieces w, w + WK, ... of every row.
// Channel order within a wavefront's blocks, strides, tails and tensors on a torus as in the kernel above.
// us a call between two events with the caches emptied before, ring -> this: 14x14 1024->256 one stream 31.7 -> 15.6, 28x28
// 512->128 21.3 -> 13.0, 7x7 2048->512 53.0 -> 20.3, 56x56 64->256 12.4 -> 13.1.  Error of the sums against 64 bits, same
// layers: 3.99e-7 -> 2.06e-7, 2.84e-7 -> 1.51e-7, 5.76e-7 -> 2.90e-7, 1.03e-7 -> 0.79e-7.
// (In bf16, whose MFMAs are sixteen times as fast, the ring's workgroups wait for memory alone and whole stacks gained nothing:
// Darknet-19 416x416 on one stream took 1577 us a clip of ten frames with this kernel and 1467 without.)
template <int U, int NB, int WK>
__global__ __launch_bounds__(WK * 64) void conv_pw_split_kernel(ConvParams P) {
    typedef float T;
    typedef Frag<T> F;
    typedef typename F::vec vec;
    constexpr int ES = (int)sizeof(T), RB = 128, GPC = 2, NT = NB * 16;
    constexpr int ITEMS = U * NB / 2;                      // (unit, pair of channel blocks): what a lane stores at once
    static_assert(NB % 2 == 0, "eight channels a store");
    __shared__ __align__(16) floatx4 red[WK][U * NB][64];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, q = lane >> 4;
    const int n_units = unit_count(P);
    const int n_wg_tiles = (n_units + U - 1) / U * P.R, tiles_per_xcd = (n_wg_tiles + 7) >> 3;
    const int t = (int)(blockIdx.x & 7) * tiles_per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= tiles_per_xcd || t >= n_wg_tiles) return;    // the whole workgroup, before any barrier
    const int ug = t / P.R, ntile = t - ug * P.R;
    const int n0 = ntile * NT;
    const int CinES = P.Cin * ES;
    const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.in), 0, P.in_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.w), 0, P.w_bytes, kBufferFlags);

    uint32_t wgo[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int ch = n0 + (l16 >> 2) * (4 * NB) + 4 * j + (l16 & 3);
        wgo[j] = ch < P.Cout ? (uint32_t)(ch * CinES) : kOob;
    }
    struct Pieces { vec w[GPC][NB], x[GPC][U]; };
    uint32_t pgo[U];
    // offsets beyond a row's end, a missing pixel or channel: all beyond the tensor, the load returns zeros (both out of
    // range wrap to the start of the tensor and meet sums that are not stored)
    auto k_offset = [&](int chunk, int g) { const int kb = chunk * RB + g * 64 + q * 16; return kb < CinES ? (uint32_t)kb : kOob; };
    auto load_w = [&](Pieces& f, int chunk) {
#pragma unroll
        for (int g = 0; g < GPC; ++g) {
            const uint32_t ko = k_offset(chunk, g);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const uint32_t off = wgo[j] + ko;
                f.w[g][j] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, off, 0, 0));
            }
        }
    };
    auto load_x = [&](Pieces& f, int chunk) {
#pragma unroll
        for (int g = 0; g < GPC; ++g) {
            const uint32_t ko = k_offset(chunk, g);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t off = pgo[u] + ko;
                f.x[g][u] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(in_rsrc, off, 0, 0));
            }
        }
    };
    floatx4 acc[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[u][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](const Pieces& f) {
#pragma unroll
        for (int g = 0; g < GPC; ++g)
#pragma unroll
            for (int e = 0; e < F::NE; ++e)
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int j = 0; j < NB; ++j) F::mma1(f.w[g][j], f.x[g][u], acc[u][j], e);
    };

    Pieces a, b;
    const int n_ch = P.n_chunks;
    if (wave < n_ch) load_w(a, wave);                      // on their way while the units are looked up
    // unit u: place of the lane's pixel in the output (element offset; -1: not stored) and in the input
    int dst[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int at = ug * U + u;
        int stream = 0, uy = 0, ux = 0, mixed = 0xffff;
        if (at < n_units) {
            if (P.units) {
                const TileDev td = P.units[at];
                stream = td.stream; uy = td.ty; ux = td.tx; mixed = td.reuse_mask;
            } else {
                stream = fast_div_any(at, P.npix_magic, P.units_x * P.units_y);
                const int r = at - stream * (P.units_x * P.units_y);
                uy = fast_div(r, P.pw_magic); ux = r - uy * P.units_x; mixed = 0;
            }
        }
        const int y = uy * 4 + (l16 >> 2), x = ux * 4 + (l16 & 3);
        const bool ok = at < n_units && y < P.Hout && x < P.Wout;
        int iy = y * P.s, ix = x * P.s, oy = y, ox = x;
        if (P.in_origin || P.out_origin) {                 // tensors on a torus (stride 1 only: the launcher sees to it)
            const size_t og = (size_t)stream * P.origin_stride;
            if (P.in_origin && ok) { ix = torus_wrap(x, P.in_origin[og], P.Win); iy = torus_wrap(y, P.in_origin[og + 1], P.Hin); }
            if (P.out_origin && ok) { ox = torus_wrap(x, P.out_origin[og], P.Wout); oy = torus_wrap(y, P.out_origin[og + 1], P.Hout); }
        }
        pgo[u] = ok ? (uint32_t)(((stream * P.Hin + iy) * P.Win + ix) * CinES) : kOob;
        dst[u] = ok && !((mixed >> l16) & 1) ? ((stream * P.Hout + oy) * P.Wout + ox) * P.Cout : -1;
    }
    if (wave < n_ch) {
        load_x(a, wave);
        for (int c = wave;;) {
            if (c + WK < n_ch) { load_w(b, c + WK); load_x(b, c + WK); }
            mma(a);
            c += WK;
            if (c >= n_ch) break;
            if (c + WK < n_ch) { load_w(a, c + WK); load_x(a, c + WK); }
            mma(b);
            c += WK;
            if (c >= n_ch) break;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < NB; ++j) red[wave][u * NB + j][lane] = acc[u][j];
    __syncthreads();
    const int parts = n_ch < WK ? n_ch : WK;
#pragma unroll
    for (int i0 = 0; i0 < ITEMS; i0 += WK) {
        const int item = i0 + wave;
        if (item >= ITEMS) break;
        const int u = item / (NB / 2), j = item % (NB / 2) * 2;
        const int co = n0 + q * (4 * NB) + 4 * j;
        int at = dst[0];
#pragma unroll
        for (int v = 1; v < U; ++v) at = u == v ? dst[v] : at;
        if (co >= P.Cout || at < 0) continue;
        floatx4 v0 = red[0][u * NB + j][lane], v1 = red[0][u * NB + j + 1][lane];
#pragma unroll
        for (int w = 1; w < WK; ++w)
            if (w < parts) { v0 += red[w][u * NB + j][lane]; v1 += red[w][u * NB + j + 1][lane]; }
        if (P.bias) { v0 += *reinterpret_cast<const floatx4*>(P.bias + co); v1 += *reinterpret_cast<const floatx4*>(P.bias + co + 4); }
        if (P.relu) { activate4(v0, P.relu); activate4(v1, P.relu); }
        T* const px = reinterpret_cast<T*>(P.out) + at + co;
        F::store4(px, v0);
        F::store4(px + 4, v1);
    }
}

// ---- first layer -------------------------------------------------------------------------
// A pixel of the network input is one 16-byte vector (4 fp32 or 8 bf16 channels, the frame's three
// plus zero padding).  Four taps of a kernel row are then consecutive pixels, 64 bytes of input
// against 64 bytes of weights, which is one K group of the MFMA: a 3x3 kernel is 3 groups with
// the fourth quarter zeroed, a 7x7 kernel 14 groups with one quarter in eight zeroed.  There is
// nothing to stage: every wavefront takes one unit (16 pixels x NB 16-channel blocks), loads its
// fragments from memory directly and keeps the weights in registers while it walks over the unit
// list.  S is the stride: output pixel (y, x) reads input rows y S - p .. y S - p + K - 1.
template <typename T, int NB, int K, int S, int U>
__device__ __forceinline__ void conv_first_body(const ConvParams& P) {
    typedef Frag<T> F;
    typedef typename F::vec vec;
    constexpr bool kWide = sizeof(T) == 2 && NB >= 2;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, q = lane >> 4;
    const int n0 = blockIdx.y * (NB * 16);
    const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.in), 0, P.in_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.w), 0, P.w_bytes, kBufferFlags);

    constexpr int TG = (K + 3) / 4;                          // groups of four taps per kernel row
    vec wv[K][TG][NB];
#pragma unroll
    for (int ky = 0; ky < K; ++ky)
#pragma unroll
      for (int g = 0; g < TG; ++g)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            // bf16: row l16 of block j carries output channel (l16 / 4) * 4 NB + 4 j + l16 % 4, so that the accumulators
            // of a lane (rows 4q .. 4q+3 of every block) are 4 NB consecutive channels and leave in 16-byte stores.
            // fp32 keeps channel 16 j + l16: there a store instruction already writes 64 contiguous bytes per pixel.
            const int co = kWide ? (l16 >> 2) * (4 * NB) + j * 4 + (l16 & 3) : j * 16 + l16;
            const uint32_t off = g * 4 + q < K ? (uint32_t)(((n0 + co) * (K * K) + ky * K + g * 4 + q) * 16) : kOob;
            wv[ky][g][j] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, off, 0, 0));
        }
    constexpr int kBlockStep = kWide ? 4 : 16;               // channel distance between a lane's blocks
    const int chan = n0 + (kWide ? 4 * NB : 4) * q;
    floatx4 bias[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
        bias[j] = P.bias ? *reinterpret_cast<const floatx4*>(P.bias + chan + j * kBlockStep) : floatx4{0.f, 0.f, 0.f, 0.f};
    const bool relu = P.relu != 0;
    const int per = P.units_x * P.units_y;

    // The loop is pipelined by hand.  A wavefront takes U consecutive units per step, requests the input vectors of
    // the next step's units before it multiplies and stores the current ones, and reads the unit list two steps
    // ahead (wavefront-uniform addresses: scalar loads), so that a step waits for one memory latency at most.
    struct UnitPos { int stream, uy, ux, mixed; };     // mixed == -1: no such unit
    // Output on a torus: the streams' origins wait in LDS (P.n_streams of them; 0: too many, they are loaded from
    // memory where they are needed, a load that depends on the list entry and stalls the step)
    extern __shared__ int2 first_origins[];
    if (P.out_origin && P.n_streams > 0) {
        for (int s = threadIdx.x; s < P.n_streams; s += 256)
            first_origins[s] = int2{P.out_origin[(size_t)s * P.origin_stride], P.out_origin[(size_t)s * P.origin_stride + 1]};
        __syncthreads();
    }
    const int n_units = unit_count(P);
    auto locate = [&](int u) {
        UnitPos r{0, 0, 0, -1};
        if (u >= n_units) return r;
        if (P.units) {
            const TileDev t = P.units[u];
            r.stream = t.stream; r.uy = t.ty; r.ux = t.tx; r.mixed = t.reuse_mask & 0xffff;
        } else {
            r.stream = fast_div_any(u, P.npix_magic, P.units_x * P.units_y);
            const int rem = u - r.stream * per;
            r.uy = fast_div(rem, P.pw_magic); r.ux = rem - r.uy * P.units_x;
            r.mixed = 0;
        }
        return r;
    };
    auto load_x = [&](const UnitPos& pos, vec (&xv)[K][TG]) {
        const int y = pos.uy * 4 + (l16 >> 2), x = pos.ux * 4 + (l16 & 3);
#pragma unroll
        for (int ky = 0; ky < K; ++ky)
#pragma unroll
            for (int g = 0; g < TG; ++g) {
                const int iy = y * S - P.p + ky, ix = x * S - P.p + g * 4 + q;
                const bool ok = pos.mixed >= 0 && g * 4 + q < K && (unsigned)iy < (unsigned)P.Hin && (unsigned)ix < (unsigned)P.Win;
                const uint32_t off = ok ? (uint32_t)(((pos.stream * P.Hin + iy) * P.Win + ix) * 16) : kOob;
                xv[ky][g] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(in_rsrc, off, 0, 0));
            }
    };
    const int step = (int)gridDim.x * 4 * U;
    int u = ((int)blockIdx.x * 4 + wave) * U;
    if (u >= n_units) return;
    UnitPos pos[U], pos_next[U], pos_after[U];
    vec xv[U][K][TG], xv_next[U][K][TG];
#pragma unroll
    for (int i = 0; i < U; ++i) { pos[i] = locate(u + i); load_x(pos[i], xv[i]); }
#pragma unroll
    for (int i = 0; i < U; ++i) pos_next[i] = locate(u + step + i);
    for (;;) {
        const bool more = u + step < n_units;          // wavefront-uniform
        if (more) {
#pragma unroll
            for (int i = 0; i < U; ++i) { load_x(pos_next[i], xv_next[i]); pos_after[i] = locate(u + 2 * step + i); }
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            floatx4 acc[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[j] = bias[j];
#pragma unroll
            for (int ky = 0; ky < K; ++ky)
#pragma unroll
              for (int g = 0; g < TG; ++g)
#pragma unroll
                for (int e = 0; e < F::NE; ++e)
#pragma unroll
                    for (int j = 0; j < NB; ++j) F::mma1(wv[ky][g][j], xv[i][ky][g], acc[j], e);
            const int y = pos[i].uy * 4 + (l16 >> 2), x = pos[i].ux * 4 + (l16 & 3);
            // a reusable pixel holds the cached value
            const bool keep = pos[i].mixed >= 0 && y < P.Hout && x < P.Wout && !((pos[i].mixed >> l16) & 1);
            if (keep) {
                int yo = y, xo = x;
                if (P.out_origin) {       // the output lies on a torus
                    const int2 og = P.n_streams > 0 ? first_origins[pos[i].stream]
                                                    : int2{P.out_origin[(size_t)pos[i].stream * P.origin_stride],
                                                           P.out_origin[(size_t)pos[i].stream * P.origin_stride + 1]};
                    xo = torus_wrap(x, og.x, P.Wout);
                    yo = torus_wrap(y, og.y, P.Hout);
                }
                T* px = reinterpret_cast<T*>(P.out) + ((pos[i].stream * P.Hout + yo) * P.Wout + xo) * P.Cout + chan;
                floatx4 v[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    v[j] = acc[j];
                    if (relu) activate4(v[j], P.relu);
                }
                if constexpr (kWide) {                          // eight bf16 channels per 16-byte store
#pragma unroll
                    for (int j = 0; j < NB; j += 2) {
                        uintx4 w4;
                        w4[0] = (uint32_t)F::bits(v[j][0]) | ((uint32_t)F::bits(v[j][1]) << 16);
                        w4[1] = (uint32_t)F::bits(v[j][2]) | ((uint32_t)F::bits(v[j][3]) << 16);
                        w4[2] = (uint32_t)F::bits(v[j + 1][0]) | ((uint32_t)F::bits(v[j + 1][1]) << 16);
                        w4[3] = (uint32_t)F::bits(v[j + 1][2]) | ((uint32_t)F::bits(v[j + 1][3]) << 16);
                        *reinterpret_cast<uintx4*>(px + j * 4) = w4;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < NB; ++j) F::store4(px + j * kBlockStep, v[j]);
                }
            }
        }
        if (!more) break;
        u += step;
#pragma unroll
        for (int i = 0; i < U; ++i) {
            pos[i] = pos_next[i];
            pos_next[i] = pos_after[i];
#pragma unroll
            for (int ky = 0; ky < K; ++ky)
#pragma unroll
                for (int g = 0; g < TG; ++g) xv[i][ky][g] = xv_next[i][ky][g];
        }
    }
}

// Units per wavefront and step of the 3x3 first-layer kernel.  Measured on 64 bf16 streams at 224x224 (411 MB of output):
// 1, 2, 3, 4 units per step all take 160-180 us in full and 71 / 81 / 77 us on the bench's cached frames, so more units
// in flight buy nothing; the same kernel without its stores takes 52 us, without its loads 112 us, with neither 34 us.
constexpr int kFirstUnits = 1;
// 3x3 stride 1 (the first layer of the VGG-like stacks) and 7x7 stride 2 (the stem of the residual networks).
template <typename T, int NB>
__global__ __launch_bounds__(256) void conv_first_kernel(ConvParams P) { conv_first_body<T, NB, 3, 1, kFirstUnits>(P); }
template <typename T, int NB>
__global__ __launch_bounds__(256) void conv_stem_kernel(ConvParams P) { conv_first_body<T, NB, 7, 2, 1>(P); }
// 11x11 stride 4 (the first layer of AlexNet-style stacks): 33 weight vectors per channel block stay in registers
template <typename T>
__global__ __launch_bounds__(256) void conv_stem11_kernel(ConvParams P) { conv_first_body<T, 1, 11, 4, 1>(P); }

// ---- bf16 stems whose input pixels hold at most four channels ---------------------------------------------------
// Tensor 0 of a stack has eight channels per pixel (one 16-byte vector), of which a frame fills three or four; the rest are
// exact zeros.  In the kernels above every block of 16 or 32 channels fetches every input vector again: AlexNet's first layer
// loads 33 KiB per unit and block.  Here the unit's patch is brought into LDS once, four channels a pixel, for all channels
// of the workgroup, and a wavefront keeps the weights of 16 NB channels in registers.
//   workgroup = NU groups of two units at a time, NWC wavefronts of 16 NB channels each per group; persistent, walks the unit list
//               (one unit at a time: 96 channels on 64 streams 58.8 us for 52.8; four chains of MFMAs instead of two, and a weight
//               fragment with its zeros serves both.  The 32-channel form takes one: a wavefront brings whole patches there, and
//               the registers do not hold two.)
//   K groups  = four taps of a kernel row, one per quarter of a wavefront, row after row: those of the kernels above, in their
//               order.  Two groups share the registers of a fragment (four channels of each); the MFMA of one multiplies
//               the other's pixels by zeros, as the kernels above do with channels four to seven: the same bits.  (Both
//               in one MFMA, or MFMAs of half the K, would add in another order: measured, one value in 65 000 rounds
//               to another bf16.)  The weights with their zeros are made by two moves per two MFMAs; kept in registers for one
//               block of channels per wavefront they take longer (11x11 on 64 streams 85 us), the pixels being read twice as often.
// LDS: rows are RS bytes apart and, 11x11, column x of row y lies at x ^ 2 (y / 4 % 2): the 32 reads of half a wavefront (pixels
// of two quarters) fall into different banks.
// Channels four to seven of the weights meet zeros and are not read.
// 227x227 11x11 -> 96 on 1 / 4 / 16 / 64 streams, against the kernel above: 9.3 -> 8.4, 17.0 -> 13.6, 45.7 -> 23.2, 148.5 -> 52.4 us (37 MB
// out and 53 MB in on 64: 18 at the copy's rate); 224x224 7x7 -> 64 on 1 / 4 / 8 / 16 / 64: 6.2 -> 8.5, 11.3 -> 12.8, 17.3 -> 16.8, 28.0 -> 21.5, 92.0 -> 48.6.
// What bounds it: a step's chain of load, LDS write, barrier, reads and MFMAs at two workgroups per CU (the pixels requested
// two steps ahead, with one unit: 11x11 64 us for 58, 7x7 85 for 56: the registers cost more than the wait).
constexpr int stem4_units(int k, int nwc) { return k == 11 && nwc == 1 ? 1 : 2; }      // of a wavefront at a time
template <int K, int S, int NB, int NWC, int NU>
__global__ __launch_bounds__(NWC * NU * 64) __attribute__((amdgpu_waves_per_eu(2))) void conv_stem4_kernel(ConvParams P) {
    typedef __hip_bfloat16 T;
    typedef Frag<T> F;
    typedef F::vec vec;
    constexpr int TG = (K + 3) / 4, NG = K * TG, NP = (NG + 1) / 2;      // groups of a kernel row, all groups, pairs of them
    constexpr int UW = stem4_units(K, NWC);
    constexpr bool kSwizzle = K == 11;
    constexpr int PH = 3 * S + K, PWX = 3 * S + 4 * TG, RS = K == 11 ? 208 : 160;
    constexpr int GT = NWC * 64, NPT = (PH * PWX + GT - 1) / GT, PATCH = PH * RS;
    static_assert(PWX * 8 <= RS && (!kSwizzle || PWX % 4 == 0), "shape; a swizzled column stays in its row");

    __shared__ __align__(16) unsigned char smem[NU * UW * 2 * PATCH];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, q = lane >> 4;
    const int wave_u = wave / NWC, wave_c = wave % NWC;
    const int n0 = ((int)blockIdx.y * NWC + wave_c) * (NB * 16);
    const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.in), 0, P.in_bytes, kBufferFlags);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(P.w), 0, P.w_bytes, kBufferFlags);

    // group g, quarter q: tap 4 (g % TG) + q of kernel row g / TG; groups 2 i and 2 i + 1 in the halves of wv[i]
    uintx4 wv[NP][NB];
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            // row l16 of block j: channel (l16 / 4) * 4 NB + 4 j + l16 % 4, so that a lane ends with 4 NB consecutive ones
            const int co = n0 + (l16 >> 2) * (4 * NB) + j * 4 + (l16 & 3);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int g = 2 * i + h, tap = g % TG * 4 + q;
                const uint32_t off = g < NG && tap < K ? (uint32_t)((co * (K * K) + g / TG * K + tap) * 16) : kOob;
                const uintx2 d = __builtin_bit_cast(uintx2, __builtin_amdgcn_raw_buffer_load_b64(w_rsrc, off, 0, 0));
                wv[i][j][2 * h] = d[0]; wv[i][j][2 * h + 1] = d[1];
            }
        }
    uintx4 w_lo[NB], w_hi[NB];                       // one group's weights beside zeros
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        w_lo[j] = w_hi[j] = uintx4{0, 0, 0, 0};
        asm volatile("" : "+v"(w_lo[j]), "+v"(w_hi[j]));       // (the zeros stay in registers)
    }
    const int chan = n0 + 4 * NB * q;
    floatx4 bias[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
        bias[j] = P.bias ? *reinterpret_cast<const floatx4*>(P.bias + chan + j * 4) : floatx4{0.f, 0.f, 0.f, 0.f};
    const bool relu = P.relu != 0;

    // the pixels of a patch that this thread brings: row and column in the patch, byte offset in LDS
    const int gt = wave_c * 64 + lane;
    int ppy[NPT], ppx[NPT], ppos[NPT];
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int at = gt + i * GT;
        ppy[i] = at / PWX;
        ppx[i] = at - ppy[i] * PWX;
        ppos[i] = ppy[i] * RS + (kSwizzle ? ppx[i] ^ (ppy[i] >> 2 & 1) * 2 : ppx[i]) * 8;
    }
    const int n_units = unit_count(P), per = P.units_x * P.units_y;
    struct UnitPos { int stream, uy, ux, mixed; };     // mixed == -1: no such unit
    auto locate = [&](int u) {
        UnitPos r{0, 0, 0, -1};
        if (u >= n_units) return r;
        if (P.units) {
            const TileDev t = P.units[u];
            r.stream = t.stream; r.uy = t.ty; r.ux = t.tx; r.mixed = t.reuse_mask & 0xffff;
        } else {
            r.stream = fast_div_any(u, P.npix_magic, per);
            const int rem = u - r.stream * per;
            r.uy = fast_div(rem, P.pw_magic); r.ux = rem - r.uy * P.units_x;
            r.mixed = 0;
        }
        return r;
    };
    uintx2 px[UW][NPT];
    auto load_px = [&](int w, const UnitPos& pos) {
        const int y0 = pos.uy * (4 * S) - P.p, x0 = pos.ux * (4 * S) - P.p;
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
            const int iy = y0 + ppy[i], ix = x0 + ppx[i];
            const bool ok = pos.mixed >= 0 && (unsigned)iy < (unsigned)P.Hin && (unsigned)ix < (unsigned)P.Win;
            const uint32_t off = ok ? (uint32_t)(((pos.stream * P.Hin + iy) * P.Win + ix) * 16) : kOob;
            px[w][i] = __builtin_bit_cast(uintx2, __builtin_amdgcn_raw_buffer_load_b64(in_rsrc, off, 0, 0));
        }
    };
    // read side: this quarter's tap of group 0, for kernel rows ky with ky / 4 even and odd
    static_assert(!kSwizzle || S == 4, "line l16 / 4 of the output starts at row 4 (l16 / 4) of the patch");
    int xaddr[2];
#pragma unroll
    for (int o = 0; o < 2; ++o)
        xaddr[o] = (l16 >> 2) * (S * RS) + (l16 & 3) * (S * 8) + (kSwizzle ? q ^ (((l16 >> 2) + o) & 1) * 2 : q) * 8;

    const int step = (int)gridDim.x * (NU * UW), first = (int)blockIdx.x * (NU * UW);
    if (first >= n_units) return;                      // the whole workgroup, before any barrier
    int u = first + wave_u * UW;
    UnitPos pos[UW], pos_next[UW];
#pragma unroll
    for (int w = 0; w < UW; ++w) {
        pos[w] = locate(u + w);
        pos_next[w] = locate(u + w + step);
        load_px(w, pos[w]);
    }
    int buf = 0;
    for (int base = first;; base += step, buf ^= 1) {
        unsigned char* const patch = smem + (wave_u * 2 + buf) * (UW * PATCH);
#pragma unroll
        for (int w = 0; w < UW; ++w)
#pragma unroll
            for (int i = 0; i < NPT; ++i)
                if ((i + 1) * GT <= PH * PWX || gt + i * GT < PH * PWX) *reinterpret_cast<uintx2*>(patch + w * PATCH + ppos[i]) = px[w][i];
        if constexpr (NWC > 1) lds_barrier();      // the patches are in LDS; nobody reads the other buffer any more
        const bool more = base + step < n_units;
        UnitPos after[UW];
        if (more) {
#pragma unroll
            for (int w = 0; w < UW; ++w) {
                load_px(w, pos_next[w]);
                after[w] = locate(u + w + 2 * step);
            }
        }
        floatx4 acc[UW][NB];
#pragma unroll
        for (int w = 0; w < UW; ++w)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[w][j] = bias[j] + 0.f;      // (-0: products with the zeros may be -0 here, and +0 is what a sum of both is)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            auto read_x = [&](int w, int g) { return *reinterpret_cast<const uintx2*>(patch + w * PATCH + xaddr[g / TG >> 2 & 1] + g / TG * RS + g % TG * 32); };
            const bool two = 2 * i + 1 < NG;
            vec x[UW];
#pragma unroll
            for (int w = 0; w < UW; ++w) {
                const uintx2 lo = read_x(w, 2 * i), hi = two ? read_x(w, 2 * i + 1) : lo;
                x[w] = __builtin_bit_cast(vec, uintx4{lo[0], lo[1], hi[0], hi[1]});
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                w_lo[j][0] = wv[i][j][0]; w_lo[j][1] = wv[i][j][1];
#pragma unroll
                for (int w = 0; w < UW; ++w) F::mma1(__builtin_bit_cast(vec, w_lo[j]), x[w], acc[w][j], 0);
            }
#pragma unroll
            for (int j = 0; two && j < NB; ++j) {
                w_hi[j][2] = wv[i][j][2]; w_hi[j][3] = wv[i][j][3];
#pragma unroll
                for (int w = 0; w < UW; ++w) F::mma1(__builtin_bit_cast(vec, w_hi[j]), x[w], acc[w][j], 0);
            }
        }
#pragma unroll
        for (int w = 0; w < UW; ++w) {
            const int y = pos[w].uy * 4 + (l16 >> 2), x = pos[w].ux * 4 + (l16 & 3);
            if (pos[w].mixed >= 0 && y < P.Hout && x < P.Wout && !((pos[w].mixed >> l16) & 1)) {      // a reusable pixel holds the cached value
                int yo = y, xo = x;
                if (P.out_origin) {
                    xo = torus_wrap(x, P.out_origin[(size_t)pos[w].stream * P.origin_stride], P.Wout);
                    yo = torus_wrap(y, P.out_origin[(size_t)pos[w].stream * P.origin_stride + 1], P.Hout);
                }
                T* out = reinterpret_cast<T*>(P.out) + ((pos[w].stream * P.Hout + yo) * P.Wout + xo) * P.Cout + chan;
                uint32_t v[2 * NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    if (relu) activate4(acc[w][j], P.relu);
                    v[2 * j] = (uint32_t)F::bits(acc[w][j][0]) | ((uint32_t)F::bits(acc[w][j][1]) << 16);
                    v[2 * j + 1] = (uint32_t)F::bits(acc[w][j][2]) | ((uint32_t)F::bits(acc[w][j][3]) << 16);
                }
#pragma unroll
                for (int j = 0; j < NB; j += 2)
                    *reinterpret_cast<uintx4*>(out + j * 4) = uintx4{v[2 * j], v[2 * j + 1], v[2 * j + 2], v[2 * j + 3]};
            }
        }
        if (!more) break;
        u += step;
#pragma unroll
        for (int w = 0; w < UW; ++w) {
            pos[w] = pos_next[w];
            pos_next[w] = after[w];
        }
    }
}

// Workgroups of a launch: two per CU, which is what the registers allow (256 / 512 of them: 11x11 67 / 53 us on 64 streams, 7x7 with one
// unit a wavefront 71 / 56, and 768 66 / 60: every further one loads its weights again).
constexpr int kStem4Wgs = 512;
constexpr int kStem4Id = 432;         // kernel ids: 7x7, then 11x11 with 1, 2, 3 wavefronts a unit
// Wavefronts per unit of conv_stem4_kernel, 0: not its shape, or too few units for it: a 7x7 layer's patches are small and what
// they save has to pay for the longer start of a workgroup.  Full frames (units of 64 channels, us, the other kernel / this one): 3136
// units 11.3 / 12.8, 5488 15.6 / 14.8, 6272 17.3 / 16.8.  The units of a list lie apart, which costs the other kernel more (it fetches
// every input vector of a unit by itself): 1850 units 9.6 / 10.8, 2792 12.6 / 13.3, 3448 14.3 / 13.7, 5684 21.4 / 15.5, 11 500 36.8 / 23.8.
// Both kernels give the same bits.  Units per workgroup 1 or 4 in dc_conv_tuning choose one.
int stem4_waves(const ConvLaunch& c, long n_units, int forced) {
    if (c.dtype != DC_BF16 || c.c_frame < 1 || c.c_frame > 4 || c.Cin != 8 || forced == 1) return 0;
    if (c.k == 7 && c.s == 2) return c.Cout % 64 == 0 && (forced == 4 || n_units * (c.Cout / 64) >= (c.tiles ? 3000 : 6000)) ? 1 : 0;
    return c.k == 11 && c.s == 4 ? (c.Cout % 96 == 0 ? 3 : c.Cout % 64 == 0 ? 2 : c.Cout % 32 == 0 ? 1 : 0) : 0;
}
hipError_t stem4_launch(int k, int nwc, dim3 grid, hipStream_t st, const ConvParams& P) {
    if (k == 7) hipLaunchKernelGGL((conv_stem4_kernel<7, 2, 4, 1, 4>), grid, dim3(256), 0, st, P);
    else if (nwc == 3) hipLaunchKernelGGL((conv_stem4_kernel<11, 4, 2, 3, 1>), grid, dim3(192), 0, st, P);
    else if (nwc == 2) hipLaunchKernelGGL((conv_stem4_kernel<11, 4, 2, 2, 1>), grid, dim3(128), 0, st, P);
    else hipLaunchKernelGGL((conv_stem4_kernel<11, 4, 2, 1, 1>), grid, dim3(64), 0, st, P);
    return hipGetLastError();
}

template <typename T>
hipError_t first_launch(int k, int nb, dim3 grid, hipStream_t st, const ConvParams& P) {
    const size_t lds = P.out_origin ? (size_t)P.n_streams * sizeof(int2) : 0;      // the table of origins
    if (k == 11) hipLaunchKernelGGL((conv_stem11_kernel<T>), grid, dim3(256), lds, st, P);
    else if (k == 7) {
        if (nb == 2) hipLaunchKernelGGL((conv_stem_kernel<T, 2>), grid, dim3(256), lds, st, P);
        else hipLaunchKernelGGL((conv_stem_kernel<T, 1>), grid, dim3(256), lds, st, P);
    }
    else if (nb == 4) hipLaunchKernelGGL((conv_first_kernel<T, 4>), grid, dim3(256), lds, st, P);
    else if (nb == 2) hipLaunchKernelGGL((conv_first_kernel<T, 2>), grid, dim3(256), lds, st, P);
    else hipLaunchKernelGGL((conv_first_kernel<T, 1>), grid, dim3(256), lds, st, P);
    return hipGetLastError();
}

// ---- kernel table -----------------------------------------------------------------------
// Two wavefront arrangements (8 wavefronts each):
//   narrow: 2 x 4 wavefronts, a wavefront = up to 8 units x 16 channels, 64 channels per workgroup.  One LDS
//           read feeds four fp32 MFMAs, so fp32 is far from the LDS limit and the finest unit granularity wins.
//   wide:   4 x 2 wavefronts, a wavefront = up to 4 units x 64 channels, 128 channels per workgroup.  bf16 needs
//           one LDS read per operand per MFMA of 16 cycles: u + 4 reads for 4u MFMAs keep LDS at about half
//           of its bandwidth, where the narrow shape (u + 1 reads for u MFMAs) is bound by it.
//   wide64: 4 x 2 wavefronts, a wavefront = up to 4 units x 32 channels, 64 channels per workgroup: the bf16
//           shape for layers whose channel count is not a multiple of 128 (u + 2 reads for 2u MFMAs).
//   tall:   6 x 2 wavefronts (three per SIMD, 168 registers), a wavefront = 3 units x 64 channels, 18 units x 128
//           channels per workgroup: the same LDS reads per MFMA as wide with 3 units (7 for 12), but 18 units per
//           workgroup instead of 16.  A launch runs in rounds of 256 workgroups (one per CU: the LDS), and the last
//           round costs a whole one however few workgroups it holds; with 18 units the list of a layer often needs one
//           round less (28x28 x 64 streams: 700 workgroups instead of 784, three rounds instead of four).
struct Geom { int wm, wn, nbw, max_upw; };
constexpr int kNumGeom = 4;
constexpr Geom kGeom[kNumGeom] = {{2, 4, 1, 8}, {4, 2, 4, 4}, {4, 2, 2, 4}, {6, 2, 4, 3}};
inline int geom_nt(int geom) { return kGeom[geom].wn * kGeom[geom].nbw * 16; }

template <typename T, int KC, int U, int WM, int WN, int NBW, int KSZ = 3>
hipError_t fast_launch_one(dim3 grid, size_t lds, hipStream_t st, const ConvParams& P) {
    auto fn = conv_fast_kernel<T, KSZ, KC, U, WM, WN, NBW>;
    static std::atomic<bool> raised{false};   // per instantiation: the attribute is raised once, to the CU's whole LDS
    if (lds > 64 * 1024 && !raised.load()) {
        hipError_t a = hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
        if (a != hipSuccess) return a;
        raised.store(true);
    }
    hipLaunchKernelGGL((conv_fast_kernel<T, KSZ, KC, U, WM, WN, NBW>), grid, dim3(WM * WN * 64), lds, st, P);
    return hipGetLastError();
}
template <typename T, int KC>
hipError_t fast_launch_narrow(int upw, dim3 grid, size_t lds, hipStream_t st, const ConvParams& P) {
    switch (upw) {
        case 1: return fast_launch_one<T, KC, 1, 2, 4, 1>(grid, lds, st, P);
        case 2: return fast_launch_one<T, KC, 2, 2, 4, 1>(grid, lds, st, P);
        case 3: return fast_launch_one<T, KC, 3, 2, 4, 1>(grid, lds, st, P);
        case 4: return fast_launch_one<T, KC, 4, 2, 4, 1>(grid, lds, st, P);
        case 5: return fast_launch_one<T, KC, 5, 2, 4, 1>(grid, lds, st, P);
        case 6: return fast_launch_one<T, KC, 6, 2, 4, 1>(grid, lds, st, P);
        case 7: return fast_launch_one<T, KC, 7, 2, 4, 1>(grid, lds, st, P);
        default: return fast_launch_one<T, KC, 8, 2, 4, 1>(grid, lds, st, P);
    }
}
template <typename T, int KC>
hipError_t fast_launch_wide(int upw, dim3 grid, size_t lds, hipStream_t st, const ConvParams& P) {
    switch (upw) {
        case 1: return fast_launch_one<T, KC, 1, 4, 2, 4>(grid, lds, st, P);
        case 2: return fast_launch_one<T, KC, 2, 4, 2, 4>(grid, lds, st, P);
        case 3: return fast_launch_one<T, KC, 3, 4, 2, 4>(grid, lds, st, P);
        default: return fast_launch_one<T, KC, 4, 4, 2, 4>(grid, lds, st, P);
    }
}
template <typename T, int KC>
hipError_t fast_launch_wide64(int upw, dim3 grid, size_t lds, hipStream_t st, const ConvParams& P) {
    switch (upw) {
        case 1: return fast_launch_one<T, KC, 1, 4, 2, 2>(grid, lds, st, P);
        case 2: return fast_launch_one<T, KC, 2, 4, 2, 2>(grid, lds, st, P);
        case 3: return fast_launch_one<T, KC, 3, 4, 2, 2>(grid, lds, st, P);
        default: return fast_launch_one<T, KC, 4, 4, 2, 2>(grid, lds, st, P);
    }
}
// chunk index: KC = KG, 2 KG.  The wide arrangements are instantiated for bf16 only.
hipError_t fast_launch(bool bf16, int geom, int kci, int upw, dim3 grid, size_t lds, hipStream_t st, const ConvParams& P) {
    if (bf16 && geom == 1)
        return kci ? fast_launch_wide<__hip_bfloat16, 64>(upw, grid, lds, st, P) : fast_launch_wide<__hip_bfloat16, 32>(upw, grid, lds, st, P);
    if (bf16 && geom == 3) return fast_launch_one<__hip_bfloat16, 32, 3, 6, 2, 4>(grid, lds, st, P);   // (only this shape is built)
    if (bf16 && geom == 2)
        return kci ? fast_launch_wide64<__hip_bfloat16, 64>(upw, grid, lds, st, P) : fast_launch_wide64<__hip_bfloat16, 32>(upw, grid, lds, st, P);
    if (bf16) return kci ? fast_launch_narrow<__hip_bfloat16, 64>(upw, grid, lds, st, P) : fast_launch_narrow<__hip_bfloat16, 32>(upw, grid, lds, st, P);
    return kci ? fast_launch_narrow<float, 32>(upw, grid, lds, st, P) : fast_launch_narrow<float, 16>(upw, grid, lds, st, P);
}

// 5x5 layers (bf16): a unit's patch is 8 x 8 rows and a stage holds five taps, so the wide arrangement has room for two
// units per wavefront (145 KB) and wide64 for three.  Against the general kernel, which computes every LDS address of its
// inner loop, us per layer: 27x27 96->256 on 64 streams 182 -> 96, on 16 streams 71 -> 40, 56x56 128->128 on 8 streams
// 85 -> 46, and no smaller one measured was slower, so every such layer with whole 64-byte rows comes here.  fp32 stays on
// the general kernel (bound by the MFMA stream there, and its two half sums round less).  The sums of a stage on their own
// (SHORT) cost 3 to 6 % of a layer (27x27 96->256 on 64 streams, whole layer in bf16: 66.0 -> 68.4 us); what the fp32 sums lose
// where they cancel, rms: general kernel 8.9e-5, one chain 1.7e-4, this 4.4e-5.
hipError_t fast_launch5(int geom, int upw, dim3 grid, size_t lds, hipStream_t st, const ConvParams& P) {
    typedef __hip_bfloat16 B;
    if (geom == 1) return upw == 1 ? fast_launch_one<B, 32, 1, 4, 2, 4, 5>(grid, lds, st, P) : fast_launch_one<B, 32, 2, 4, 2, 4, 5>(grid, lds, st, P);
    return upw == 1 ? fast_launch_one<B, 32, 1, 4, 2, 2, 5>(grid, lds, st, P)
         : upw == 2 ? fast_launch_one<B, 32, 2, 4, 2, 2, 5>(grid, lds, st, P) : fast_launch_one<B, 32, 3, 4, 2, 2, 5>(grid, lds, st, P);
}
// instantiations: k = 3 or 5, arrangement, chunk index, units per wavefront
bool fast_built(int k, bool bf16, int geom, int kci, int upw) {
    if (upw < 1 || upw > kGeom[geom].max_upw || (geom != 0 && !bf16)) return false;
    if (k == 5) return bf16 && kci == 0 && ((geom == 1 && upw <= 2) || (geom == 2 && upw <= 3));
    return geom != 3 || (upw == 3 && kci == 0);      // one of the tall arrangement
}

size_t fast_lds_bytes(int k, int geom, int kci, int upw) {
    const int rpi = 16 >> kci;            // rows per load instruction: RB = 64 << kci
    return kHeaderBytes + 2 * (size_t)(kGeom[geom].wm * upw * (3 + k) * 8 / rpi) * 1024 + 2 * (size_t)(k * geom_nt(geom) / rpi) * 1024;
}

struct FastChoice { int g, ks, kci; double cost; int geom; };      // geom kDeep: conv_deep_kernel, ks its wavefronts

// Overrides of the launch model (dc_conv_tuning: tests and experiments): arrangement, units per workgroup,
// K split, channel chunk index; -1 = chosen by the model.  Process-wide; readers take a snapshot under the mutex.
std::mutex g_tune_mutex;
ConvTuning g_tune_shared{{-1, -1, -1, -1}};

// conv_deep_kernel: 256 channels per workgroup, 128 where the layer's channels are no multiple of 256.
constexpr int kDeep = 4, kDeepMinUnits = 6, kDeepMaxUnits = 8;
constexpr int kDeepId = 416;          // kernel ids: + units - 1, + 8 for two wavefronts
inline size_t deep_lds_bytes(int g) { return kHeaderBytes + 2 * (size_t)((g * 36 + 15) / 16) * 1024; }
// conv_map_kernel: tiles of 16 pixels per wavefront 1 .. 4, 64 or 128 channels per workgroup.
constexpr int kMapId = 448;           // kernel ids: + tiles per wavefront - 1, + 4 for 128 channels
constexpr size_t map_lds_bytes(int nbw) { return 2 * 16 * 1024 + 2 * (size_t)(6 * nbw) * 1024; }
// A layer the kernel can run: the map with its border fits 16 x 16 slots, and a list built elsewhere comes with the units' masks.
bool map_shape(const ConvLaunch& c) {
    return c.dtype == DC_BF16 && c.k == 3 && c.p == 1 && c.Hout == c.Hin && c.Wout == c.Win && c.Hout <= 14 && c.Wout <= 14 && c.Cout % 64 == 0 &&
           (!c.tiles || c.umask) && (long)c.n_streams * (c.Cout / 64) < 2147483647L;
}
// Blocks of 16 channels per wavefront (2 or 4) where it is the faster one, 0: it is not.  Maps of at least nine tiles (with fewer a stage
// is mostly its barrier: 14x14 256->256 on 16 streams 11 -> 18 us) that it takes at least an eighth of the rows off, by cost in
// the unit of the model below, against `other`, the cheapest of the other kernels.  The two wavefronts of a SIMD hold half of the
// tiles between them, rounded up: 288 cycles of MFMAs for two blocks of channels per tile and 32 channels.  Registers, not LDS, limit
// the variant with four blocks, and both with four tiles a wavefront, to one workgroup per CU; with two blocks and up to three tiles
// two share it, which takes 1.5 times as long as one of them.  Measured, us, model in brackets, of two blocks / four blocks / the others:
//   13x13  384->384  40 streams (one workgroup per CU) 24 (21) / 32 (30) / 29 (26);  56 (two) 33 (33) / 32 (30) / 37 (35);
//          96 (three) 50 (49) / 61 (60) / 62 (62);  128 51 (49) / 61 (60) / 81 (77);  160 (four) 64 (66) / 63 (60) / 86 (88)
//   13x13 512->1024  8 streams 26 (26) / 38 (38) / 22 (21);  16 28 (26) / 38 (38) / 33 (33);  34 63 (63) / 78 (76) / 58 (64);
//          44 63 (63) / 78 (76) / 80 (85);  80 105 (104) / 117 (113) / 125 (146)
//   14x14  512->512  28 streams 29 (29) / 41 (42) / 33 (30);  40 55 (58) / 42 (42) / 40 (39);  64 56 (58) / 47 (42) / 56 (57);
//          144 136 (144) / 130 (127) / 119 (129)
//   11x13  256->512  30 streams 15 (15) / 20 (20) / 16 (16);  40 22 (22) / 21 (20) / 20 (19);  64 23 (22) / 22 (20) / 26 (25);  160 50 (54) / 57 (60) / 53 (53)
// The model of the others is good to a tenth, so this kernel has to win by more than that can hide; for up to a workgroup per CU
// it finds the others too fast instead (14x14 256->256 on 56 streams 19.6, by the model 17.2).
int map_blocks(const ConvLaunch& c, double other) {
    const int tiles = (c.Hout * c.Wout + 15) / 16, units = ((c.Hout + 3) / 4) * ((c.Wout + 3) / 4);
    if (!map_shape(c) || tiles < 9 || tiles * 8 > units * 7) return 0;
    const int half = (tiles + 1) / 2, n_ch = c.Cin / 32;
    const long w64 = (long)c.n_streams * (c.Cout / 64), per_cu = (w64 + 255) / 256;
    const double four = c.Cout % 128 ? 1e300 : (double)((w64 / 2 + 255) / 256) * (13000 + n_ch * (576.0 * half + 460));
    const double lone = 11600 + n_ch * (326.0 * half + 600), pair = 15400 + n_ch * (576.0 * half + 750);
    const double two = tiles > 12 ? per_cu * lone : (per_cu / 2) * pair + (per_cu % 2) * (per_cu > 1 ? lone - 10000 : lone);
    if (std::min(four, two) < 0.92 * other) return four <= two ? 4 : 2;
    return per_cu == 1 && two < 1.02 * other ? 2 : 0;
}
template <int NBW>
hipError_t map_launch(int upw, dim3 grid, hipStream_t st, const ConvParams& P) {
    static std::atomic<bool> raised{false};
    if (map_lds_bytes(NBW) > 64 * 1024 && !raised.load()) {
        hipError_t a = hipSuccess;
        for (const void* fn : {reinterpret_cast<const void*>(conv_map_kernel<1, NBW>), reinterpret_cast<const void*>(conv_map_kernel<2, NBW>),
                               reinterpret_cast<const void*>(conv_map_kernel<3, NBW>), reinterpret_cast<const void*>(conv_map_kernel<4, NBW>)})
            if (a == hipSuccess) a = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)map_lds_bytes(NBW));
        if (a != hipSuccess) return a;
        raised.store(true);
    }
    if (upw == 1) hipLaunchKernelGGL((conv_map_kernel<1, NBW>), grid, dim3(512), map_lds_bytes(NBW), st, P);
    else if (upw == 2) hipLaunchKernelGGL((conv_map_kernel<2, NBW>), grid, dim3(512), map_lds_bytes(NBW), st, P);
    else if (upw == 3) hipLaunchKernelGGL((conv_map_kernel<3, NBW>), grid, dim3(512), map_lds_bytes(NBW), st, P);
    else hipLaunchKernelGGL((conv_map_kernel<4, NBW>), grid, dim3(512), map_lds_bytes(NBW), st, P);
    return hipGetLastError();
}
template <int NW>
hipError_t deep_launch(int g, dim3 grid, hipStream_t st, const ConvParams& P) {
    if (g == 8) hipLaunchKernelGGL((conv_deep_kernel<NW, 8>), grid, dim3(NW * 64), deep_lds_bytes(8), st, P);
    else if (g == 7) hipLaunchKernelGGL((conv_deep_kernel<NW, 7>), grid, dim3(NW * 64), deep_lds_bytes(7), st, P);
    else hipLaunchKernelGGL((conv_deep_kernel<NW, 6>), grid, dim3(NW * 64), deep_lds_bytes(6), st, P);
    return hipGetLastError();
}
// Cost of a launch in the unit of the model below (about 0.5 ns).  A CU holds two workgroups of four wavefronts (four of two);
// a pair of them takes the longer of its MFMAs and its weight fragments' cache look-ups (two per four lanes), a lone one
// more than half of a pair.  Measured, us, conv_fast_kernel's best -> units per workgroup 6 / 7 / 8: 56x56 256->256 64 streams
// 214 -> 212 / 175 / 181, 16 streams 60 -> 68 / 51 / 54; 28x28 512->512 64 streams 199 -> 219 / 186 / 221, 16 streams
// 60 -> 83 / 55 / 60; 112x112 128->128 64 / 28 / 20 streams 254 -> 233 / 222 / 223, 114 -> 106 / 103 / 100,
// 84 -> 83 / 80 / 73; launches of less than one workgroup per CU lose (13x13 512->1024
// 16 streams 34 -> 41 / 45 / 50), and so do few workgroups of two wavefronts (13x13 384->384 64 streams 40 -> 49 / 56 / 65;
// 52x52 128->384 8 streams, 1014 of them, 23 -> 27), hence the least number of those.
double deep_cost(const ConvLaunch& c, long n_units, int g) {
    const int nw = c.Cout % 256 ? 2 : 4, n_ch = c.Cin / 32;
    const long wgs = (n_units + g - 1) / g * (c.Cout / (64 * nw));
    if (nw == 2 && wgs < 1500) return 1e300;
    const double m = 576.0 * g * n_ch, look = 2 * 4608.0 * 1.08 * n_ch;
    const double pair = (2.6 * m > look ? 2.6 * m : look) + (nw == 2 ? 14000 : 10000), lone = 1.45 * m + 20000;
    const long per_cu = nw == 2 ? (wgs + 511) / 512 : (wgs + 255) / 256;
    return (per_cu / 2) * pair + (per_cu % 2) * lone;
}

// Cycle model of one launch.  A workgroup spends its stages (the longer of the MFMA time and the time to
// bring the stage's bytes into LDS) plus fixed costs per stage and per workgroup (decode, address set-up,
// first loads, epilogue).  A CU runs ceil(workgroups / 256) of them; as many as LDS and registers allow
// are resident together, and only the stage work of resident workgroups adds up, the fixed costs overlap.
// ks > 1 adds the reduction kernel.
// n_units: the list length to tune for; n_cap: the longest the list can be (bounds the partial sums of a K split)
FastChoice choose_fast(const ConvLaunch& c, long n_units, long n_cap, size_t scratch_bytes, int force_geom) {
    // bytes per clock and CU from L2 to LDS, fixed cycles per stage / workgroup / reduction launch (fitted to sweeps)
    constexpr double bw = 32, stage_fix = 250, wg_fix = 4500, red_fix = 13000, occ1_penalty = 1.08, lds_cap_kb = 160;
    const bool bf16 = c.dtype == DC_BF16;
    const int esz = bf16 ? 2 : 4, kg = bf16 ? 32 : 16, k = c.k;
    FastChoice best{0, 0, 0, 1e300, 0};
    for (int geom = 0; geom < kNumGeom; ++geom) {
        const Geom& G = kGeom[geom];
        const int nt = geom_nt(geom);
        if (c.Cout % nt) continue;
        if (geom != 0 && !bf16) continue;                       // not instantiated
        if (force_geom >= 0 && force_geom < kNumGeom && force_geom != geom && c.Cout % geom_nt(force_geom) == 0 && (force_geom == 0 || bf16)) continue;
        const int R = c.Cout / nt;
        for (int kci = 0; kci < 2; ++kci) {
            const int kc = kg << kci;
            if (c.Cin % kc) continue;
            const int n_chunks = c.Cin / kc, gpc = 1 << kci, rb = kc * esz;
            for (int g = 1; g <= G.wm * G.max_upw; ++g) {
                const int upw = (g + G.wm - 1) / G.wm;
                if (!fast_built(k, bf16, geom, kci, upw)) continue;
                if (fast_lds_bytes(k, geom, kci, upw) > 160 * 1024) continue;
                if (geom == 0 && !bf16 && fast_lds_bytes(k, geom, kci, upw) > (size_t)(lds_cap_kb * 1024)) continue;
                const long groups = (n_units + g - 1) / g;
                int last_cps = 0;
                for (int ks = 1; ks <= n_chunks && ks <= 64; ++ks) {
                    const int cps = (n_chunks + ks - 1) / ks;
                    if (cps == last_cps) continue;        // same split as a smaller ks
                    last_cps = cps;
                    const int ks_eff = (n_chunks + cps - 1) / cps;
                    if (ks_eff > 1 && (size_t)ks_eff * n_cap * 16 * c.Cout * 4 > scratch_bytes) continue;
                    // per stage: MFMA cycles of a SIMD (two wavefronts), LDS cycles of the CU (a 16-byte read of
                    // a wavefront takes 4), cycles to load the stage
                    // units per SIMD: the two wavefronts of a SIMD belong to wave_m groups 0/1 (narrow) or 0/2, 1/3
                    auto nu = [&](int m) { return (g - m + G.wm - 1) / G.wm; };
                    const int su = G.wm == 2 ? nu(0) + nu(1)
                                 : G.wm == 6 ? (nu(0) + nu(2) + nu(4) > nu(1) + nu(3) + nu(5) ? nu(0) + nu(2) + nu(4) : nu(1) + nu(3) + nu(5))
                                             : (nu(0) + nu(2) > nu(1) + nu(3) ? nu(0) + nu(2) : nu(1) + nu(3));
                    // (the tall arrangement needs 5 % more per unit than the wide one when both fill their rounds: measured)
                    const double mfma = (geom == 3 ? 1.18 : 1.12) * (bf16 ? 16.0 : 128.0) * su * G.nbw * k * gpc;
                    const double ldsr = (double)(G.wm * G.wn) * (upw + G.nbw) * k * gpc * 4 * 1.3;
                    const double load = ((double)g * (3 + k) * (3 + k) * rb / k + (double)k * nt * rb) / bw;
                    double stage = mfma > load ? mfma : load;
                    if (ldsr > stage) stage = ldsr;
                    const double work = cps * k * stage;
                    const double fixed = wg_fix + 400.0 * upw * G.nbw + cps * k * stage_fix;
                    const long wgs = groups * R * ks_eff;
                    const long per_cu = (wgs + 255) / 256;
                    const int vgprs = (kci ? 64 : 44) + (geom ? 10 * G.nbw * upw + 6 * G.nbw : (kci ? 18 : 16) * upw);
                    long occ = (long)(160 * 1024 / fast_lds_bytes(k, geom, kci, upw));
                    if (occ > 512 / vgprs / 2) occ = 512 / vgprs / 2;
                    if (occ > 4) occ = 4;
                    if (occ < 1) occ = 1;
                    // Workgroups that are all resident from the start share their CU to the end: the fullest CU
                    // sets the time.  With more rounds than that the dispatcher balances the CUs and only the last
                    // round is not a whole one.
                    // (measured for one workgroup per CU: 28x28 512->512 takes 179 us with 760 workgroups, 203 us with 772,
                    // 238 us with 1020 and 257 us with 1032, so up to eight rounds the last one counts as a whole one)
                    const double rounds = (wgs <= 512 || wgs <= 256 * occ || (occ == 1 && geom != 0 && wgs <= 2048)) ? (double)per_cu : wgs / 256.0 + 0.5;
                    double cost = rounds * work + (double)((per_cu + occ - 1) / occ) * fixed;
                    // a lone workgroup per CU leaves the matrix cores idle during its barriers, prologue and epilogue,
                    // and leaves no room for the workgroups of the other frame in flight (measured: 5 % per frame)
                    if (occ < 2) cost *= occ1_penalty;
                    if (ks_eff > 1) cost += red_fix + (double)(ks_eff + 1) * n_units * 16 * c.Cout * 4 / 1200.0;
                    if (cost < best.cost) best = FastChoice{g, ks_eff, kci, cost, geom};
                }
            }
        }
    }
    return best;
}

}  // namespace

// Ids 64.. name the instantiations of this file: 64 + ((bf16 * 2 + kci) * 8 + UPW - 1), 96.. the first-layer kernel,
// 110.. the wide arrangement.
bool conv_kernel_built(int id) {
    if (id >= kPwManyId) return id < kPwManyId + 4;
    if (id >= kMapId) return id < kMapId + 8;
    if (id >= kPwAddId) return id < kPwAddId + 4;
    if (id >= kStem4Id) return id < kStem4Id + 4;
    if (id >= kDeepId) return id < kDeepId + 16 && id % 8 + 1 >= kDeepMinUnits;
    return id >= kPwSplitId ? id < kPwSplitId + 2 : id >= 132 && (id - 132) / 8 < kNumGeom && fast_built(5, true, (id - 132) / 8, 0, (id - 132) % 8 + 1);
}
void conv_fast_kernel_name(int id, char* buf, size_t n) {
    if (id == 126) { snprintf(buf, n, "conv_regw_kernel<2, 2, false>"); return; }
    if (id == 130) { snprintf(buf, n, "conv_regw_kernel<2, 2, true>"); return; }      // tensors on a torus
    if (id == 129) { snprintf(buf, n, "conv_fast_kernel<__hip_bfloat16, 3, 32, 3, 6, 2, 4>"); return; }     // the tall arrangement
    if (id == 127 || id == 128 || id == 108 || id == 109) {      // 108 + bf16 (64 x 64 tile), 127 + bf16 (128 x 128): conv_pw_kernel (1x1)
        snprintf(buf, n, "conv_pw_kernel<%s, %d>", id == 109 || id == 128 ? "__hip_bfloat16" : "float", id >= 127 ? 4 : 2);
        return;
    }
    if (id >= kPwManyId) {
        snprintf(buf, n, "conv_pw_many_kernel<%s, %d>", id & 1 ? "__hip_bfloat16" : "float", id >= kPwManyId + 2 ? 4 : 2);
        return;
    }
    if (id >= kMapId) {
        snprintf(buf, n, "conv_map_kernel<%d, %d>", (id - kMapId) % 4 + 1, id >= kMapId + 4 ? 4 : 2);
        return;
    }
    if (id >= kPwAddId) {
        snprintf(buf, n, "conv_pw_add_kernel<%s, %d>", id & 1 ? "__hip_bfloat16" : "float", id >= kPwAddId + 2 ? 4 : 2);
        return;
    }
    if (id >= kStem4Id) {
        if (id == kStem4Id) snprintf(buf, n, "conv_stem4_kernel<7, 2, 4, 1, 4>");
        else snprintf(buf, n, "conv_stem4_kernel<11, 4, 2, %d, 1>", id - kStem4Id);
        return;
    }
    if (id >= kDeepId) {
        snprintf(buf, n, "conv_deep_kernel<%d, %d>", id < kDeepId + 8 ? 4 : 2, id % 8 + 1);
        return;
    }
    if (id >= kPwSplitId) {
        snprintf(buf, n, "conv_pw_split_kernel<%d, 2, %d>", id - kPwSplitId + 1, kPwSplit);
        return;
    }
    if (id >= 132) {  // 132 + arrangement * 8 + UPW - 1: 5x5 layers
        const Geom& G = kGeom[(id - 132) / 8];
        snprintf(buf, n, "conv_fast_kernel<__hip_bfloat16, 5, 32, %d, %d, %d, %d>", (id - 132) % 8 + 1, G.wm, G.wn, G.nbw);
        return;
    }
    if (id >= 110) {  // 110 + (arrangement - 1) * 8 + kci * 4 + UPW - 1: the wide bf16 arrangements
        const int v = (id - 110) % 8, wide64 = (id - 110) / 8;
        snprintf(buf, n, "conv_fast_kernel<__hip_bfloat16, 3, %d, %d, 4, 2, %d>", 32 << (v / 4), v % 4 + 1, wide64 ? 2 : 4);
        return;
    }
    if (id == 106 || id == 107) {     // 106 + bf16: conv_stem11_kernel (11x11 stride 4)
        snprintf(buf, n, "conv_stem11_kernel<%s>", id == 107 ? "__hip_bfloat16" : "float");
        return;
    }
    if (id >= 102 && id < 106) {   // 102 + bf16 * 2 + {0, 1}: conv_stem_kernel (7x7 stride 2) with 1, 2 channel blocks
        snprintf(buf, n, "conv_stem_kernel<%s, %d>", (id - 102) / 2 ? "__hip_bfloat16" : "float", 1 << ((id - 102) % 2));
        return;
    }
    if (id >= 96) {   // 96 + bf16 * 3 + {0, 1, 2}: conv_first_kernel with 1, 2, 4 channel blocks
        snprintf(buf, n, "conv_first_kernel<%s, %d>", (id - 96) / 3 ? "__hip_bfloat16" : "float", 1 << ((id - 96) % 3));
        return;
    }
    const int v = id - 64, upw = v % 8 + 1, kci = (v / 8) % 2, bf16 = v / 16;
    snprintf(buf, n, "conv_fast_kernel<%s, 3, %d, %d, 2, 4, 1>", bf16 ? "__hip_bfloat16" : "float", (bf16 ? 32 : 16) << kci, upw);
}

ConvTuning conv_tuning() {
    std::lock_guard<std::mutex> guard(g_tune_mutex);
    return g_tune_shared;
}
void conv_set_tuning(int geom, int g, int ks, int kci) {
    std::lock_guard<std::mutex> guard(g_tune_mutex);
    g_tune_shared = ConvTuning{{geom >= 0 ? geom : -1, g > 0 ? g : -1, ks > 0 ? ks : -1, kci >= 0 ? kci : -1}};
}

size_t packed_weights_bytes(int k, int s, int cin, int cout, int dtype) {
    const size_t esz = dtype_size(dtype);
    if (k != 3 || s != 1 || cout % geom_nt(0) != 0 || (cin * esz) % 64 != 0 || cin * esz == 16) return 0;
    return (size_t)cout * 9 * cin * esz;
}

hipError_t launch_pack_weights(const void* w, void* packed, int cin, int cout, int dtype, hipStream_t st) {
    const size_t esz = dtype_size(dtype);
    const size_t n_vec = (size_t)cout * 9 * cin * esz / 16;
    hipLaunchKernelGGL(pack_weights_kernel, dim3((unsigned)((n_vec + 255) / 256)), dim3(256), 0, st,
                       static_cast<const uintx4*>(w), static_cast<uintx4*>(packed), (int)(cin * esz / 64), n_vec);
    return hipGetLastError();
}

template <int WM, int UPW, bool TORUS>
hipError_t regw_launch_t(dim3 grid, hipStream_t st, const ConvParams& P) {
    const size_t lds = 2 * (size_t)(WM * UPW) * 48 * 128 + (TORUS ? (size_t)P.n_streams * sizeof(int2) : 0);
    static std::atomic<bool> raised{false};
    if (lds > 64 * 1024 && !raised.load()) {
        hipError_t a = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_regw_kernel<WM, UPW, TORUS>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
        if (a != hipSuccess) return a;
        raised.store(true);
    }
    hipLaunchKernelGGL((conv_regw_kernel<WM, UPW, TORUS>), grid, dim3(WM * 128), lds, st, P);
    return hipGetLastError();
}

// Units per workgroup of a 1x1 layer.
//   fp32: the kernel that splits K adds in another order than the ring, so the length that decides between them is the longest
//   the list can be, not the one an earlier frame had: a frame's bits do not depend on counters that may have arrived or not,
//   and the grid, which covers that length, has at most 512 workgroups.  One unit per workgroup while that makes one per CU
//   (us as above, one unit, two, ring: 14x14 1024->256 one stream 15.6, 18.2, 31.7), two up to two workgroups per CU (13x13
//   1024->512 two streams 21.0, 18.8, 32.0); four wavefronts per tile hide each other's MFMAs there.
//   128 x 128 tiles need every CU to hold several workgroups; 4096 of the smaller ones (measured in bf16: 2 % of a ResNet-50
//   frame on 64 streams).  fp32: only where K is deep as well (us, 64 x 64 -> 128 x 128: 14x14 1024->2048 32 streams 312 -> 296,
//   but 56x56 256->128 92 -> 107, 64->256 64 streams 108 -> 118).
int pw_units(const ConvLaunch& c, long n_cap, long n_units, int n_chunks, int forced) {
    if (forced == 4 || forced == 8) return forced;
    const bool bf16 = c.dtype == DC_BF16;
    const long r32 = (c.Cout + 31) / 32, small_tiles = (n_units + 3) / 4 * ((c.Cout + 63) / 64);
    if (!bf16 && n_cap * r32 <= 256) return 1;
    if (!bf16 && (n_cap + 1) / 2 * r32 <= 512) return 2;
    return small_tiles >= 4096 && c.Cout >= 128 && (bf16 || n_chunks >= 32) ? 8 : 4;
}
// The launch of a 1x1 layer; false if its shape does not qualify.
struct PwLaunch {
    ConvParams P;
    int units;            // per workgroup: 1, 2 (fp32: split K, 32 channels), 4 (64 channels), 8 (128 channels)
    int wgs;
    size_t lds;           // of the kernels with a ring
};
bool pw_prepare(const ConvLaunch& c, long n_cap, long n_units, PwLaunch& L) {
    const size_t esz = dtype_size(c.dtype);
    if ((c.in_origin || c.out_origin) && c.s != 1) return false;
    if (c.k != 1 || c.p != 0 || (c.s != 1 && c.s != 2) || (c.Cin * esz) % 16 || c.Cout % 8) return false;
    if (reinterpret_cast<uintptr_t>(c.in) % 16 || reinterpret_cast<uintptr_t>(c.w) % 16 || reinterpret_cast<uintptr_t>(c.out) % 16 ||
        (c.bias && reinterpret_cast<uintptr_t>(c.bias) % 16))
        return false;
    const int units_y = (c.Hout + 3) / 4, units_x = (c.Wout + 3) / 4;
    const int kc = (int)(128 / esz), n_chunks = (c.Cin + kc - 1) / kc;
    L.units = pw_units(c, n_cap, n_units, n_chunks, conv_tuning().v[1]);
    const int nt = L.units == 8 ? 128 : L.units == 4 ? 64 : 32, threads = L.units >= 4 ? L.units * 64 : kPwSplit * 64;
    const long R = (c.Cout + nt - 1) / nt, groups = (n_cap + L.units - 1) / L.units;
    const long tiles = (groups + 7) / 8 * 8 * R;      // (whole rounds of the XCDs)
    if ((double)c.n_streams * c.Hout * c.Wout * c.Cout >= 2147483648.0 || tiles >= 2147483647L / threads) return false;
    L.wgs = (int)tiles;
    ConvParams& P = L.P;
    P = ConvParams{};
    P.in = c.in; P.w = c.w; P.bias = c.bias; P.out = c.out;
    P.Hin = c.Hin; P.Win = c.Win; P.Cin = c.Cin; P.Hout = c.Hout; P.Wout = c.Wout; P.Cout = c.Cout;
    P.k = c.k; P.s = c.s; P.p = c.p; P.relu = c.relu;
    P.units = c.tiles; P.n_units = (int)n_cap; P.n_units_dev = c.tiles ? c.n_tiles_dev : nullptr;
    P.units_x = units_x; P.units_y = units_y;
    P.npix_magic = (uint32_t)((0x100000000ull + (uint64_t)(units_x * units_y) - 1) / (uint64_t)(units_x * units_y));
    P.pw_magic = (uint32_t)((0x100000000ull + (uint64_t)units_x - 1) / (uint64_t)units_x);
    P.in_bytes = (uint32_t)((size_t)c.n_streams * c.Hin * c.Win * c.Cin * esz);
    P.w_bytes = (uint32_t)((size_t)c.Cout * c.Cin * esz);
    P.n_chunks = n_chunks;
    P.in_origin = c.in_origin; P.out_origin = c.out_origin; P.origin_stride = c.origin_stride;
    P.R = (int)R;
    // Every kernel starts with cold caches, so a workgroup's walk over K is a chain of long-latency loads:
    // up to four chunks are in flight per workgroup, and several workgroups share a CU.
    const int stages = n_chunks < 4 ? n_chunks : 4;
    L.lds = kPwHeaderBytes + (size_t)stages * (size_t)(L.units * 4096);
    return true;
}
template <typename T, int WM>
hipError_t pw_raise() {
    static std::atomic<bool> raised{false};
    if (raised.load()) return hipSuccess;
    for (const void* f : {reinterpret_cast<const void*>(conv_pw_kernel<T, WM>), reinterpret_cast<const void*>(conv_pw_add_kernel<T, WM>),
                          reinterpret_cast<const void*>(conv_pw_many_kernel<T, WM>)}) {
        const hipError_t a = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
        if (a != hipSuccess) return a;
    }
    raised.store(true);
    return hipSuccess;
}
template <typename T, int WM>
hipError_t pw_launch_n(const PwLaunch& L, hipStream_t st) {
    if (L.lds > 64 * 1024) {
        const hipError_t a = pw_raise<T, WM>();
        if (a != hipSuccess) return a;
    }
    const dim3 grid((unsigned)L.wgs);
    if (L.P.add_out) hipLaunchKernelGGL((conv_pw_add_kernel<T, WM>), grid, dim3(WM * 128), L.lds, st, L.P);
    else hipLaunchKernelGGL((conv_pw_kernel<T, WM>), grid, dim3(WM * 128), L.lds, st, L.P);
    return hipGetLastError();
}
template <typename T>
hipError_t pw_launch(const PwLaunch& L, hipStream_t st) {
    if (L.units == 8) return pw_launch_n<T, 4>(L, st);
    if (L.units == 4) return pw_launch_n<T, 2>(L, st);
    if constexpr (sizeof(T) == 4) {
        const dim3 grid((unsigned)L.wgs);
        if (L.units == 2) hipLaunchKernelGGL((conv_pw_split_kernel<2, 2, kPwSplit>), grid, dim3(kPwSplit * 64), 0, st, L.P);
        else hipLaunchKernelGGL((conv_pw_split_kernel<1, 2, kPwSplit>), grid, dim3(kPwSplit * 64), 0, st, L.P);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}
template <typename T, int WM>
hipError_t pw_many_launch(const PwMany& M, unsigned wgs, size_t lds, hipStream_t st) {
    if (lds > 64 * 1024) {
        const hipError_t a = pw_raise<T, WM>();
        if (a != hipSuccess) return a;
    }
    hipLaunchKernelGGL((conv_pw_many_kernel<T, WM>), dim3(wgs), dim3(WM * 128), lds, st, M);
    return hipGetLastError();
}
hipError_t launch_conv_batch(const ConvBatch& b, hipStream_t st) {
    PwLaunch L[kConvBatch];
    for (int i = 0; i < b.n; ++i) {
        const ConvLaunch& c = b.c[i];
        long n_cap = 0, n_units = 0;
        L[i].units = 0;
        if (c.kw || c.dil > 1 || !conv_list_length(c, &n_cap, &n_units) || !pw_prepare(c, n_cap, n_units, L[i])) L[i].units = 0;
    }
    for (int units : {4, 8}) {
        PwMany M{};
        int of[kConvBatch], n = 0, wgs = 0;
        size_t lds = 0;
        for (int i = 0; i < b.n; ++i)
            if (L[i].units == units && b.c[i].dtype == b.c[0].dtype && wgs <= 2147483647 / 512 - L[i].wgs) {
                of[n] = i; M.p[n] = L[i].P; M.first[n++] = wgs;
                wgs += L[i].wgs; lds = std::max(lds, L[i].lds);
            }
        if (n < 2) continue;
        for (int j = n; j < kConvBatch; ++j) M.first[j] = wgs;      // (no workgroup)
        const int bf16 = b.c[0].dtype == DC_BF16 ? 1 : 0;
        hipError_t e;
        if (units == 8) e = bf16 ? pw_many_launch<__hip_bfloat16, 4>(M, (unsigned)wgs, lds, st) : pw_many_launch<float, 4>(M, (unsigned)wgs, lds, st);
        else e = bf16 ? pw_many_launch<__hip_bfloat16, 2>(M, (unsigned)wgs, lds, st) : pw_many_launch<float, 2>(M, (unsigned)wgs, lds, st);
        if (e != hipSuccess) return e;
        for (int j = 0; j < n; ++j) {
            if (b.c[of[j]].kernel_id) *b.c[of[j]].kernel_id = kPwManyId + (units == 8 ? 2 : 0) + bf16;
            L[of[j]].units = -1;
        }
    }
    for (int i = 0; i < b.n; ++i)
        if (L[i].units >= 0) {
            const hipError_t e = launch_conv(b.c[i], st);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}
// Launches the layer with the kernel of this file if its shape qualifies; returns false otherwise.
bool launch_conv_fast(const ConvLaunch& c, long n_cap, long n_units, hipStream_t st, hipError_t* err) {
    // below, n_units is the length the launch is tuned for and n_cap the length it must cover; they differ only
    // when the list is built on the GPU (then the kernels read the real length from memory)
    const int* const n_dev = c.tiles ? c.n_tiles_dev : nullptr;
    constexpr bool enabled = true;
    constexpr int g_stem_wgs = 256;      // persistent workgroups of the 7x7 / 11x11 first-layer kernels
    const ConvTuning tune = conv_tuning();
    const int* g_tune = tune.v;
    const size_t esz = dtype_size(c.dtype);
    const bool torus = c.in_origin || c.out_origin;     // only the first-layer kernels (output) and the 3x3 GEMM kernel take origins
    if (enabled && !c.in_origin && ((c.k == 3 && c.s == 1) || (c.k == 7 && c.s == 2) || (c.k == 11 && c.s == 4)) && c.Cin * esz == 16 && c.Cout % 16 == 0 &&
        reinterpret_cast<uintptr_t>(c.in) % 16 == 0 && reinterpret_cast<uintptr_t>(c.w) % 16 == 0 &&
        reinterpret_cast<uintptr_t>(c.out) % 16 == 0 && (!c.bias || reinterpret_cast<uintptr_t>(c.bias) % 16 == 0)) {
        const int units_y = (c.Hout + 3) / 4, units_x = (c.Wout + 3) / 4;
        if ((double)c.n_streams * c.Hout * c.Wout * c.Cout < 2147483648.0) {
            ConvParams P{};
            P.in = c.in; P.w = c.w; P.bias = c.bias; P.out = c.out;
            P.Hin = c.Hin; P.Win = c.Win; P.Cin = c.Cin; P.Hout = c.Hout; P.Wout = c.Wout; P.Cout = c.Cout;
            P.k = c.k; P.s = c.s; P.p = c.p; P.relu = c.relu;
            P.units = c.tiles; P.n_units = (int)n_cap; P.n_units_dev = n_dev; P.rects = c.rects; P.ranges = c.ranges;
            P.units_x = units_x; P.units_y = units_y;
            P.npix_magic = (uint32_t)((0x100000000ull + (uint64_t)(units_x * units_y) - 1) / (uint64_t)(units_x * units_y));
            P.pw_magic = (uint32_t)((0x100000000ull + (uint64_t)units_x - 1) / (uint64_t)units_x);
            P.in_bytes = (uint32_t)((size_t)c.n_streams * c.Hin * c.Win * 16);
            P.w_bytes = (uint32_t)((size_t)c.Cout * c.k * c.k * 16);
            P.out_origin = c.out_origin; P.origin_stride = c.origin_stride;
            P.n_streams = c.out_origin && c.n_streams <= kRegwTorusStreams ? c.n_streams : 0;
            // the 7x7 kernel keeps 14 weight vectors per channel block in registers: two blocks at most
            const int nb = c.k == 11 ? 1 : (c.Cout % 64 == 0 && c.k == 3 ? 4 : (c.Cout % 32 == 0 ? 2 : 1));
            // four units at a time.  3x3: at most 8 workgroups per CU.  The large kernels hold one workgroup per CU
            // (registers) and pay 28 / 33 weight loads per wavefront before the first unit, so the launch is one
            // persistent workgroup per CU and channel block, each walking its share of the units.
            const long cap = c.k == 3 ? 2048 : std::max(1L, (long)g_stem_wgs / (c.Cout / (16 * nb)));
            const long per_wg = 4 * (c.k == 3 ? kFirstUnits : 1);        // units per workgroup and step
            const long wgx = (n_cap + per_wg - 1) / per_wg < cap ? (n_cap + per_wg - 1) / per_wg : cap;
            if (c.kernel_id)
                *c.kernel_id = c.k == 11 ? 106 + (c.dtype == DC_BF16 ? 1 : 0)
                             : c.k == 7 ? 102 + (c.dtype == DC_BF16 ? 2 : 0) + (nb == 2 ? 1 : 0)
                                        : 96 + (c.dtype == DC_BF16 ? 3 : 0) + (nb == 4 ? 2 : (nb == 2 ? 1 : 0));
            if (const int nwc = stem4_waves(c, n_units, g_tune[1])) {
                const int gy = c.Cout / (c.k == 7 ? 64 : 32 * nwc);
                const long nu = (c.k == 7 ? 4 : 1) * stem4_units(c.k, nwc), wgs = std::min((n_cap + nu - 1) / nu, std::max(1L, (long)kStem4Wgs / gy));
                if (c.kernel_id) *c.kernel_id = kStem4Id + (c.k == 7 ? 0 : nwc);
                *err = stem4_launch(c.k, nwc, dim3((unsigned)wgs, (unsigned)gy), st, P);
                return true;
            }
            const dim3 grid((unsigned)wgx, (unsigned)(c.Cout / (16 * nb)));
            *err = c.dtype == DC_BF16 ? first_launch<__hip_bfloat16>(c.k, nb, grid, st, P) : first_launch<float>(c.k, nb, grid, st, P);
            return true;
        }
    }
    PwLaunch pw;
    if (pw_prepare(c, n_cap, n_units, pw)) {
        // the sum with another tensor that follows: in the kernels with a ring, of lists that name the units without work too
        if (c.add && pw.units >= 4 && !torus && (!c.tiles || n_dev) && reinterpret_cast<uintptr_t>(c.add->in) % 16 == 0 &&
            reinterpret_cast<uintptr_t>(c.add->out) % 16 == 0) {
            pw.P.add_in = c.add->in; pw.P.add_out = c.add->out; pw.P.add_relu = c.add->relu;
            c.add->done = true;
        }
        const int bf16 = c.dtype == DC_BF16 ? 1 : 0;
        if (c.kernel_id && pw.P.add_out) *c.kernel_id = kPwAddId + (pw.units == 8 ? 2 : 0) + bf16;
        else if (c.kernel_id) *c.kernel_id = (pw.units == 8 ? 127 : pw.units == 4 ? 108 : kPwSplitId + pw.units - 1) + (pw.units >= 4 ? bf16 : 0);
        *err = bf16 ? pw_launch<__hip_bfloat16>(pw, st) : pw_launch<float>(pw, st);
        return true;
    }
    if (!enabled || (c.k != 3 && !(c.k == 5 && c.dtype == DC_BF16 && !torus)) || c.s != 1 || c.Cout % geom_nt(0) != 0 || c.Cin % (64 / esz) != 0) return false;
    if (reinterpret_cast<uintptr_t>(c.in) % 16 || reinterpret_cast<uintptr_t>(c.w) % 16) return false;
    if (reinterpret_cast<uintptr_t>(c.out) % 16 || (c.bias && reinterpret_cast<uintptr_t>(c.bias) % 16)) return false;
    if ((double)c.n_streams * c.Hout * c.Wout * c.Cout >= 2147483648.0) return false;      // 32-bit output offsets
    // 64 input channels in bf16 and enough units to keep persistent workgroups busy: the weights go to registers
    if (c.dtype == DC_BF16 && c.k == 3 && c.Cin == 64 && c.relu != 2 && (!torus || c.n_streams <= kRegwTorusStreams) && (g_tune[0] == 3 || (g_tune[0] < 0 && g_tune[1] < 0 && n_units >= 4096))) {
        ConvParams P{};
        P.in = c.in; P.w = c.w; P.bias = c.bias; P.out = c.out;
        P.Hin = c.Hin; P.Win = c.Win; P.Cin = c.Cin; P.Hout = c.Hout; P.Wout = c.Wout; P.Cout = c.Cout;
        P.k = c.k; P.s = c.s; P.p = c.p; P.relu = c.relu;
        P.units = c.tiles; P.n_units = (int)n_cap; P.n_units_dev = n_dev;
        P.units_x = (c.Wout + 3) / 4; P.units_y = (c.Hout + 3) / 4;
        P.npix_magic = (uint32_t)((0x100000000ull + (uint64_t)(P.units_x * P.units_y) - 1) / (uint64_t)(P.units_x * P.units_y));
        P.pw_magic = (uint32_t)((0x100000000ull + (uint64_t)P.units_x - 1) / (uint64_t)P.units_x);
        P.in_bytes = (uint32_t)((size_t)c.n_streams * c.Hin * c.Win * c.Cin * esz);
        P.w_bytes = (uint32_t)((size_t)c.Cout * 9 * c.Cin * esz);
        P.in_origin = c.in_origin; P.out_origin = c.out_origin; P.origin_stride = c.origin_stride;
        P.n_streams = c.n_streams;
        // Two persistent workgroups of four wavefronts per CU (the registers allow two wavefronts per SIMD): they
        // drift apart, so that one's address work and epilogue overlap the other's MFMAs.
        const int R = c.Cout / 64;
        const long groups = (n_cap + 3) / 4;
        long gx = 512 / R > 0 ? 512 / R : 1;
        if (gx > groups) gx = groups;
        if (c.kernel_id) *c.kernel_id = torus ? 130 : 126;
        *err = torus ? regw_launch_t<2, 2, true>(dim3((unsigned)gx, (unsigned)R), st, P)
                     : regw_launch_t<2, 2, false>(dim3((unsigned)gx, (unsigned)R), st, P);
        return true;
    }
    size_t scratch = c.scratch && reinterpret_cast<uintptr_t>(c.scratch) % 16 == 0 ? c.scratch_bytes : 0;
    if (scratch > kConvScratchBytes) scratch = kConvScratchBytes;
    // The model costs about 2 us per call on the host; the same layers come back every frame with the same or a
    // recently seen unit count, so its answers are kept in a small direct-mapped table.
    struct Memo { int dtype, k, cin, cout, tune[4]; bool packed; long n_units, n_cap; size_t scratch; FastChoice ch; bool used; };
    static Memo memo[256];
    static std::mutex memo_mutex;
    const bool packed = c.w_packed && reinterpret_cast<uintptr_t>(c.w_packed) % 16 == 0;
    const bool deep_shape = c.dtype == DC_BF16 && c.k == 3 && c.Cout % 128 == 0;
    FastChoice ch;
    {
        std::lock_guard<std::mutex> guard(memo_mutex);
        Memo& slot = memo[((unsigned long)n_units * 2654435761ul + (unsigned)c.Cin * 40503u + (unsigned)c.Cout * 97u + (unsigned)c.dtype + (unsigned)c.k * 31u) % 256];
        if (slot.used && slot.dtype == c.dtype && slot.k == c.k && slot.packed == packed && slot.cin == c.Cin && slot.cout == c.Cout && slot.n_units == n_units && slot.n_cap == n_cap &&
            slot.scratch == scratch && slot.tune[0] == g_tune[0] && slot.tune[1] == g_tune[1] && slot.tune[2] == g_tune[2] &&
            slot.tune[3] == g_tune[3]) {
            ch = slot.ch;
        } else {
            ch = choose_fast(c, n_units, n_cap, scratch, g_tune[0] == 4 ? 3 : g_tune[0]);    // tuning 3 names another kernel
            if (deep_shape && packed && g_tune[0] < 0 && g_tune[1] < 0 && g_tune[2] < 0 && g_tune[3] < 0)
                for (int g = kDeepMaxUnits; g >= kDeepMinUnits; --g) {
                    const double cost = deep_cost(c, n_units, g);
                    if (cost < ch.cost) ch = FastChoice{g, c.Cout % 256 ? 2 : 4, 0, cost, kDeep};
                }
            if (deep_shape && g_tune[0] == 5)
                ch = FastChoice{std::min(std::max(g_tune[1], kDeepMinUnits), kDeepMaxUnits), c.Cout % 256 || g_tune[2] == 2 ? 2 : 4, 0, 0, kDeep};
            slot = Memo{c.dtype, c.k, c.Cin, c.Cout, {g_tune[0], g_tune[1], g_tune[2], g_tune[3]}, packed, n_units, n_cap, scratch, ch, true};
        }
    }
    if (g_tune[1] > 0 && ch.g > 0 && ch.geom != kDeep) {    // forced shape within the arrangement the model picked
        const int f_g = g_tune[1], f_ks = g_tune[2], f_kci = g_tune[3] < 0 ? ch.kci : g_tune[3];
        const Geom& G = kGeom[ch.geom];
        const int kc = (c.dtype == DC_BF16 ? 32 : 16) << f_kci;
        const int upw = (f_g + G.wm - 1) / G.wm;
        if (f_kci < 2 && c.Cin % kc == 0 && fast_built(c.k, c.dtype == DC_BF16, ch.geom, f_kci, upw) &&
            fast_lds_bytes(c.k, ch.geom, f_kci, upw) <= 160 * 1024) {
            const int n_chunks = c.Cin / kc;
            int ks = f_ks < 1 ? 1 : (f_ks > n_chunks ? n_chunks : f_ks);
            const int cps = (n_chunks + ks - 1) / ks;
            ks = (n_chunks + cps - 1) / cps;
            if (ks == 1 || (size_t)ks * n_cap * 16 * c.Cout * 4 <= scratch) ch = FastChoice{f_g, ks, f_kci, 0, ch.geom};
        }
    }
    if (ch.g < 1) return false;
    const bool untuned = g_tune[0] < 0 && g_tune[1] < 0 && g_tune[2] < 0 && g_tune[3] < 0;
    const int map_nbw = g_tune[0] == 6 ? (map_shape(c) ? (g_tune[1] == 4 && c.Cout % 128 == 0 ? 4 : 2) : 0)
                      : untuned && ch.kci == 0 && (ch.geom == kDeep || ch.ks == 1) && n_units * 10 >= n_cap * 9 ? map_blocks(c, ch.cost) : 0;
    const bool deep = ch.geom == kDeep;
    const int nt = deep ? 64 * ch.ks : geom_nt(ch.geom), ks = deep ? 1 : ch.ks;
    const int upw = deep ? ch.g : (ch.g + kGeom[ch.geom].wm - 1) / kGeom[ch.geom].wm;
    const int kc = (c.dtype == DC_BF16 ? 32 : 16) << ch.kci;
    const int units_y = (c.Hout + 3) / 4, units_x = (c.Wout + 3) / 4;

    ConvParams P{};
    P.in = c.in; P.w = c.w; P.bias = c.bias; P.out = c.out;
    P.Hin = c.Hin; P.Win = c.Win; P.Cin = c.Cin; P.Hout = c.Hout; P.Wout = c.Wout; P.Cout = c.Cout;
    P.k = c.k; P.s = c.s; P.p = c.p; P.relu = c.relu;
    P.units = c.tiles; P.n_units = (int)n_cap; P.n_units_dev = n_dev; P.rects = c.rects; P.ranges = c.ranges;
    P.units_x = units_x; P.units_y = units_y;
    P.ph = 3 + c.k; P.pw = 3 + c.k;
    P.npix_magic = (uint32_t)((0x100000000ull + (uint64_t)(units_x * units_y) - 1) / (uint64_t)(units_x * units_y));
    P.pw_magic = (uint32_t)((0x100000000ull + (uint64_t)units_x - 1) / (uint64_t)units_x);
    P.g_rt = ch.g;
    P.in_bytes = (uint32_t)((size_t)c.n_streams * c.Hin * c.Win * c.Cin * esz);
    P.w_bytes = (uint32_t)((size_t)c.Cout * c.k * c.k * c.Cin * esz);
    P.out_vec = 1;
    P.n_chunks = c.Cin / kc;
    P.R = c.Cout / nt;
    P.ks = ks;
    P.chunks_per_split = (P.n_chunks + ks - 1) / ks;
    P.partial = ks > 1 ? static_cast<float*>(c.scratch) : nullptr;
    P.in_origin = c.in_origin; P.out_origin = c.out_origin; P.origin_stride = c.origin_stride;
    if (c.k == 3 && packed) { P.w = c.w_packed; P.w_packed = 1; }

    if (c.kernel_id) *c.kernel_id = deep ? kDeepId + (ch.ks == 2 ? 8 : 0) + ch.g - 1 : c.k == 5 ? 132 + ch.geom * 8 + upw - 1 : ch.geom == 3 ? 129 : ch.geom ? 110 + (ch.geom - 1) * 8 + ch.kci * 4 + upw - 1 : 64 + ((c.dtype == DC_BF16 ? 2 : 0) + ch.kci) * 8 + upw - 1;
    if (map_nbw) {
        const int upw = ((c.Hout * c.Wout + 15) / 16 + 3) / 4;
        P.R = c.Cout / (32 * map_nbw); P.n_chunks = c.Cin / 32;
        P.umask = c.tiles ? c.umask : nullptr;
        P.pw_magic = (uint32_t)((0x100000000ull + (uint64_t)c.Wout - 1) / (uint64_t)c.Wout);        // pixels are divided here
        if (c.kernel_id) *c.kernel_id = kMapId + (map_nbw == 4 ? 4 : 0) + upw - 1;
        const dim3 grid((unsigned)(c.n_streams * P.R));
        *err = map_nbw == 4 ? map_launch<4>(upw, grid, st, P) : map_launch<2>(upw, grid, st, P);
        return true;
    }
    const long groups = (n_cap + ch.g - 1) / ch.g;
    const long wgx = groups * P.R;
    if (wgx > 2147483647L || ks > 65535) { *err = hipErrorInvalidValue; return true; }
    const dim3 grid((unsigned)wgx, (unsigned)ks);
    if (deep) {
        *err = ch.ks == 2 ? deep_launch<2>(ch.g, grid, st, P) : deep_launch<4>(ch.g, grid, st, P);
        return true;
    }
    const size_t lds = fast_lds_bytes(c.k, ch.geom, ch.kci, upw);
    *err = c.k == 5 ? fast_launch5(ch.geom, upw, grid, lds, st, P) : fast_launch(c.dtype == DC_BF16, ch.geom, ch.kci, upw, grid, lds, st, P);
    if (*err != hipSuccess || ks == 1) return true;
    const size_t total = (size_t)n_cap * 16 * (c.Cout / 4);
    if (c.dtype == DC_BF16)
        hipLaunchKernelGGL(conv_split_reduce_kernel<__hip_bfloat16>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, P);
    else
        hipLaunchKernelGGL(conv_split_reduce_kernel<float>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, P);
    *err = hipGetLastError();
    return true;
}

}  // namespace dc
