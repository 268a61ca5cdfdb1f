// Silhouette packing and volumetric visual-hull carving (Sec. II-B-1 over the
// whole volume, Sec. II-B-3 inside ROIs) for gfx950.
//
// A workgroup of 256 threads carves a tile of TX x TY x TZ lattice samples
// (TX * TY = 256).  The tile keeps, in LDS, the list of its samples that are
// still inside every camera tested so far.  Each pass tests the listed samples
// against the next kCamGroup cameras (independent loads, one memory round trip
// per pass) and appends the survivors to the other list, so every lane of a
// pass works on a live sample: samples outside the lattice never enter the
// list and rejected ones leave it at once.  The tile is done when a pass
// leaves no survivor or the cameras run out; the survivors are the occupied
// samples.  The occupancy is the AND over all cameras, so neither the passes
// nor the order in which samples are listed change a result.  Each test
// evaluates the full fused projection chain of the sample, bit-equal to the
// definition.
#include "fvv_internal.h"

#include <type_traits>

namespace fvv {

constexpr int kCamGroup = 2;

// ------------------------------------------------------------------ packing
// Non-zero flags of the four bytes of x as bits 0..3.  Adding 0x7f to a
// byte's low seven bits sets its high bit iff they are not all zero (no carry
// leaves the byte); ORed with the byte's own high bit, that bit says the byte
// is non-zero.  Shifted to bits 0, 8, 16, 24, the flags are gathered into bits
// 21..24 by one multiply by 1 + 2^7 + 2^14 + 2^21 (no two partial products
// share a bit there).
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t x) {
    const uint32_t f = ((((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) >> 7) & 0x01010101u;
    return ((f * 0x00204081u) >> 21) & 0xfu;
}

// Unsigned 32-bit division by a fixed divisor d >= 1 with a host-computed
// multiplier (the round-up method of Granlund and Montgomery, exact for every
// 32-bit dividend): with l = ceil(log2 d) and m = floor(2^32 (2^l - d) / d) + 1,
// n / d = (t + ((n - t) >> min(l, 1))) >> max(l - 1, 0), t = (n m) >> 32.
struct DivU32 {
    uint32_t m;
    int s1, s2;
};

DivU32 divu32_magic(uint32_t d) {
    int l = 0;
    while (l < 32 && (1ull << l) < d)
        ++l;
    const uint64_t m = (((uint64_t)1 << 32) * (((uint64_t)1 << l) - d)) / d + 1;
    return DivU32{(uint32_t)m, l < 1 ? l : 1, l > 1 ? l - 1 : 0};
}

__device__ __forceinline__ uint32_t divu32(uint32_t n, const DivU32& d) {
    const uint32_t t = __umulhi(n, d.m);
    return (t + ((n - t) >> d.s1)) >> d.s2;
}

// One lane per 32-pixel word.  Its 32 bytes are read with two 16-byte loads at
// whatever address the row's width gives them (the hardware takes any
// alignment; a wave still covers 2 KB in a row).  A row's last word, when it
// has fewer pixels, takes the row's last 32 bytes and shifts: nothing outside
// the row is read.  Only rows shorter than 32 pixels are read by bytes.  The
// nine 1279 x 719 masks (8.3 MB): 3.7 us, 17 by bytes.  k32: every word index
// fits 32 bits (row = index / wpr by multiply and shifts).
template <bool k32>
__global__ __launch_bounds__(kBlock) void pack_kernel(const uint8_t* __restrict__ masks,
                                                      uint32_t* __restrict__ sils, int n, int W,
                                                      int H, int wpr, DivU32 by_wpr) {
    const int64_t total = (int64_t)n * H * wpr;
    for (int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * kBlock) {
        int64_t row;
        if (k32)
            row = divu32((uint32_t)idx, by_wpr);
        else
            row = idx / wpr;
        const int word = (int)(idx - row * wpr);
        const uint8_t* src = masks + row * W + (int64_t)word * 32;
        uint32_t bits = 0;
        const int nb = min(32, W - word * 32);
        if (W >= 32) {
            uint32_t d[8];
            __builtin_memcpy(d, src - (32 - nb), 32);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                bits |= nonzero_bytes(d[k]) << (4 * k);
            bits >>= 32 - nb;
        } else {
            for (int b = 0; b < nb; ++b)
                bits |= (uint32_t)(src[b] != 0) << b;
        }
        sils[idx] = bits;
    }
}

hipError_t launch_pack(int n, int W, int H, const uint8_t* masks, uint32_t* sils, hipStream_t s) {
    int wpr = (W + 31) / 32;
    int64_t total = (int64_t)n * H * wpr;
    int64_t blocks = (total + kBlock - 1) / kBlock;
    if (blocks > 65536)
        blocks = 65536;
    if (blocks < 1)
        blocks = 1;
    const DivU32 dw = divu32_magic((uint32_t)wpr);
    // 32-bit indices while every index the grid-stride loop forms stays below 2^32
    if (total + (int64_t)blocks * kBlock <= ((int64_t)1 << 32))
        hipLaunchKernelGGL(pack_kernel<true>, dim3((unsigned)blocks), dim3(kBlock), 0, s, masks,
                           sils, n, W, H, wpr, dw);
    else
        hipLaunchKernelGGL(pack_kernel<false>, dim3((unsigned)blocks), dim3(kBlock), 0, s, masks,
                           sils, n, W, H, wpr, dw);
    return hipGetLastError();
}

// ------------------------------------------------------------------ tiled silhouettes
// The silhouettes in 8 x 8-pixel blocks, one uint64 per block: pixel (x, y) at
// bit 8 (y & 7) + (x & 7) of block (x / 8, y / 8); blocks row-major per camera,
// block (bx, by) of camera c at c * tpc + by * tpr + bx with tpr = ceil(W / 8)
// and tpc = tpr * ceil(H / 8).  Pixels past the image are 0.  A pixel rectangle
// of up to 9 x 9 pixels lies in at most 2 x 2 blocks.
//
// Both kernels below run one thread per block; with kAny they also OR each
// non-empty block's bit into its SilAny word (all-zero before).

// From the packed rows (whose padding bits are 0).
template <bool kAny>
__global__ __launch_bounds__(kBlock) void tile_sils_kernel(const uint32_t* __restrict__ sils,
                                                           int n, int H, int wpr, int tpr,
                                                           int tph, int bw,
                                                           uint64_t* __restrict__ tiles,
                                                           uint64_t* __restrict__ any) {
    const int64_t total = (int64_t)n * tph * tpr;
    for (int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * kBlock) {
        const int64_t cb = idx / tpr;                  // camera * tph + block row
        const int bx = (int)(idx - cb * tpr);
        const int c = (int)(cb / tph), by = (int)(cb - (int64_t)c * tph);
        const uint32_t* col = sils + (int64_t)c * H * wpr + (bx >> 2);
        const int sh = 8 * (bx & 3);
        uint64_t v = 0;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int y = 8 * by + r;
            if (y < H)
                v |= (uint64_t)((col[(int64_t)y * wpr] >> sh) & 0xffu) << (8 * r);
        }
        tiles[idx] = v;
        if (kAny && v != 0)
            atomicOr((unsigned long long*)&any[cb * bw + (bx >> 6)], 1ull << (bx & 63));
    }
}


// Both forms at once, straight from the masks, for images whose width is a
// multiple of 8: each block's thread reads its 8 rows of 8 bytes (a wave
// covers 512 contiguous bytes of each row), stores the block's word and the
// block's byte of each of its 8 packed rows (the row's last block also clears
// the padding bytes of the row's last word).  k32: every block index fits 32
// bits (split by multiply and shifts).
template <bool k32, bool kAny>
__global__ __launch_bounds__(kBlock) void pack_tiled_kernel(const uint8_t* __restrict__ masks,
                                                            int n, int W, int H, int wpr,
                                                            int tpr, int tph, int bw,
                                                            DivU32 by_tpr, DivU32 by_tph,
                                                            uint32_t* __restrict__ sils,
                                                            uint64_t* __restrict__ tiles,
                                                            uint64_t* __restrict__ any) {
    const int64_t total = (int64_t)n * tph * tpr;
    uint8_t* const rows = reinterpret_cast<uint8_t*>(sils);
    const int row_bytes = 4 * wpr;
    for (int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * kBlock) {
        int64_t cb, c;
        if (k32) {
            cb = divu32((uint32_t)idx, by_tpr);
            c = divu32((uint32_t)cb, by_tph);
        } else {
            cb = idx / tpr;
            c = cb / tph;
        }
        const int bx = (int)(idx - cb * tpr);
        const int by = (int)(cb - c * tph);
        const int y0 = 8 * by;
        const int nr = min(8, H - y0);
        const uint8_t* src = masks + ((int64_t)c * H + y0) * W + 8 * bx;
        uint8_t* dst = rows + ((int64_t)c * H + y0) * row_bytes + bx;
        uint64_t v = 0;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (r < nr) {
                const uint2 q = *reinterpret_cast<const uint2*>(src + (int64_t)r * W);
                const uint32_t b = nonzero_bytes(q.x) | (nonzero_bytes(q.y) << 4);
                v |= (uint64_t)b << (8 * r);
                dst[(int64_t)r * row_bytes] = (uint8_t)b;
                if (bx == tpr - 1)
                    for (int k = tpr; k < row_bytes; ++k)
                        dst[(int64_t)r * row_bytes + (k - bx)] = 0;
            }
        }
        tiles[idx] = v;
        if (kAny && v != 0)
            atomicOr((unsigned long long*)&any[cb * bw + (bx >> 6)], 1ull << (bx & 63));
    }
}

// The same for images whose width is a multiple of 16 (masks 16-byte
// aligned): one thread per two horizontally adjacent blocks, 16-byte loads of
// its 8 rows, the two blocks' words in one 16-byte store and two bytes of
// each packed row in one 2-byte store.  kStream, for masks so large that they
// come from memory: the 8 rows' loads are issued together, past the caches (they
// are read once, and what the frame reads next stays).  10 and 24 masks of 3840 x 2160 (83 and
// 199 MB): 22 and 51 us, 29 and 57 without; 16 of 1920 x 1080 (33 MB, the L2s'
// size, held by them and the memory-side cache): 9.9 us, 7.8 without.
template <bool k32, bool kAny, bool kStream>
__global__ __launch_bounds__(kBlock) void pack_tiled16_kernel(const uint8_t* __restrict__ masks,
                                                              int n, int W, int H, int wpr,
                                                              int tpr, int tph, int bw,
                                                              DivU32 by_tp2, DivU32 by_tph,
                                                              uint32_t* __restrict__ sils,
                                                              uint64_t* __restrict__ tiles,
                                                              uint64_t* __restrict__ any) {
    const int tp2 = tpr / 2;
    const int64_t total = (int64_t)n * tph * tp2;
    uint8_t* const rows = reinterpret_cast<uint8_t*>(sils);
    const int row_bytes = 4 * wpr;
    for (int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * kBlock) {
        int64_t cb, c;
        if (k32) {
            cb = divu32((uint32_t)idx, by_tp2);
            c = divu32((uint32_t)cb, by_tph);
        } else {
            cb = idx / tp2;
            c = cb / tph;
        }
        const int bx = 2 * (int)(idx - cb * tp2);
        const int by = (int)(cb - c * tph);
        const int y0 = 8 * by;
        const int nr = min(8, H - y0);
        const uint8_t* src = masks + ((int64_t)c * H + y0) * W + 8 * bx;
        uint8_t* dst = rows + ((int64_t)c * H + y0) * row_bytes + bx;
        uint64_t v0 = 0, v1 = 0;
        typedef uint32_t Row16 __attribute__((ext_vector_type(4)));
        Row16 rows16[8];
        if (kStream) {
#pragma unroll
            for (int r = 0; r < 8; ++r)       // (rows past the image: its last again)
                rows16[r] = __builtin_nontemporal_load(
                    reinterpret_cast<const Row16*>(src + (int64_t)min(r, nr - 1) * W));
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (r < nr) {
                const Row16 q = kStream ? rows16[r]
                                        : *reinterpret_cast<const Row16*>(src + (int64_t)r * W);
                const uint32_t b0 = nonzero_bytes(q.x) | (nonzero_bytes(q.y) << 4);
                const uint32_t b1 = nonzero_bytes(q.z) | (nonzero_bytes(q.w) << 4);
                v0 |= (uint64_t)b0 << (8 * r);
                v1 |= (uint64_t)b1 << (8 * r);
                *reinterpret_cast<uint16_t*>(dst + (int64_t)r * row_bytes) =
                    (uint16_t)(b0 | (b1 << 8));
                if (bx == tpr - 2)
                    for (int k = tpr; k < row_bytes; ++k)
                        dst[(int64_t)r * row_bytes + (k - bx)] = 0;
            }
        }
        *reinterpret_cast<ulonglong2*>(tiles + cb * tpr + bx) = make_ulonglong2(v0, v1);
        if (kAny && (v0 | v1) != 0)
            atomicOr((unsigned long long*)&any[cb * bw + (bx >> 6)],
                     (unsigned long long)((v0 ? 1ull : 0ull) | (v1 ? 2ull : 0ull)) << (bx & 63));
    }
}

// Bytes of masks from which they are streamed: 28 of 1920 x 1080 (58 MB) take
// 14.5 us so and 13.5 without, 32 (66 MB) 17.0 and 17.9, 8 of 3840 x 2160 (66 MB)
// 15.5 and 18.6.
constexpr int64_t kStreamMasks = (int64_t)60 << 20;

hipError_t launch_pack_tiled(int n, int W, int H, const uint8_t* masks, uint32_t* sils,
                             uint64_t* tiles, uint64_t* any, hipStream_t s) {
    if (W % 8 != 0 || reinterpret_cast<uintptr_t>(masks) % 8 != 0) {
        hipError_t e = launch_pack(n, W, H, masks, sils, s);
        return e == hipSuccess ? launch_tile_sils(n, W, H, sils, tiles, any, s) : e;
    }
    const int wpr = (W + 31) / 32, tpr = W / 8, tph = (H + 7) / 8, bw = sil_any_bw(W);
    if (W % 16 == 0 && reinterpret_cast<uintptr_t>(masks) % 16 == 0) {
        const int64_t total = (int64_t)n * tph * (tpr / 2);
        int64_t blocks = (total + kBlock - 1) / kBlock;
        blocks = blocks < 1 ? 1 : (blocks > 65536 ? 65536 : blocks);
        const DivU32 dx = divu32_magic((uint32_t)(tpr / 2)), dy = divu32_magic((uint32_t)tph);
        const bool k32 = total + (int64_t)blocks * kBlock <= ((int64_t)1 << 32);
        // (more blocks than 32 bits index are far more than any cache)
        const bool stream = (int64_t)n * W * H >= kStreamMasks;
        auto kernel = !k32 ? (any ? pack_tiled16_kernel<false, true, true>
                                  : pack_tiled16_kernel<false, false, true>)
                      : stream ? (any ? pack_tiled16_kernel<true, true, true>
                                      : pack_tiled16_kernel<true, false, true>)
                               : (any ? pack_tiled16_kernel<true, true, false>
                                      : pack_tiled16_kernel<true, false, false>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, masks, n, W, H,
                           wpr, tpr, tph, bw, dx, dy, sils, tiles, any);
        return hipGetLastError();
    }
    const int64_t total = (int64_t)n * tph * tpr;
    int64_t blocks = (total + kBlock - 1) / kBlock;
    blocks = blocks < 1 ? 1 : (blocks > 65536 ? 65536 : blocks);
    const DivU32 dx = divu32_magic((uint32_t)tpr), dy = divu32_magic((uint32_t)tph);
    const bool k32 = total + (int64_t)blocks * kBlock <= ((int64_t)1 << 32);
    auto kernel = k32 ? (any ? pack_tiled_kernel<true, true> : pack_tiled_kernel<true, false>)
                      : (any ? pack_tiled_kernel<false, true> : pack_tiled_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, masks, n, W, H, wpr,
                       tpr, tph, bw, dx, dy, sils, tiles, any);
    return hipGetLastError();
}


hipError_t launch_tile_sils(int n, int W, int H, const uint32_t* sils, uint64_t* tiles,
                            uint64_t* any, hipStream_t s) {
    const int wpr = (W + 31) / 32, tpr = (W + 7) / 8, tph = (H + 7) / 8, bw = sil_any_bw(W);
    const int64_t total = (int64_t)n * tph * tpr;
    int64_t blocks = (total + kBlock - 1) / kBlock;
    blocks = blocks < 1 ? 1 : (blocks > 65536 ? 65536 : blocks);
    hipLaunchKernelGGL(any ? tile_sils_kernel<true> : tile_sils_kernel<false>,
                       dim3((unsigned)blocks), dim3(kBlock), 0, s, sils, n, H, wpr, tpr, tph, bw,
                       tiles, any);
    return hipGetLastError();
}

// ------------------------------------------------------------------ carving tile
constexpr int log2_of(int v) { return v <= 1 ? 0 : 1 + log2_of(v / 2); }

// Append val to an LDS list for the lanes where pred holds (one LDS atomic
// per wave).
__device__ __forceinline__ void lds_append(bool pred, uint16_t val, uint16_t* list,
                                           uint32_t* count) {
    const uint64_t m = __ballot(pred);
    if (m == 0)
        return;
    const int leader = __ffsll((unsigned long long)m) - 1;
    uint32_t base = 0;
    if (lane_id() == leader)
        base = atomicAdd(count, (uint32_t)__popcll(m));
    base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
    if (pred)
        list[base + lane_rank(m)] = val;
}

// Where the carve also writes its occupancy as bits: nowhere, ORed into the
// labelling's row bitmap (RowBits, all-zero before), or stored into a fine
// bitmap (rows padded to words, every word of the lattice written).
constexpr int kBitsNone = 0, kBitsLabel = 1, kBitsFine = 2;

// Carve tile `tile` of lattice g.  getP(c) returns camera c's 12 floats (a
// wave-uniform address); sil_of(c) its silhouette rows.  The TX lanes of one
// tile row cover TX consecutive x inside one bitmap word (TX divides 64), so a
// tile row's bits cost one atomic (kBitsLabel, none where the row is empty)
// or one store (kBitsFine).
template <int TX, int TZ, int kBits, typename GetP, typename GetSil>
__device__ __forceinline__ void carve_tile(GetP getP, GetSil sil_of, int ncam, int W, int H,
                                           int wpr, const fvv_grid& g, uint64_t tile,
                                           uint8_t* __restrict__ out, const RowBits& rb) {
    constexpr int TY = kBlock / TX;
    constexpr int TV = TX * TY * TZ;
    constexpr int LX = log2_of(TX), LY = log2_of(TY);
    __shared__ uint16_t s_list[2][TV];
    __shared__ uint32_t s_cnt[3];
    __shared__ uint32_t s_alive[TV / 32];

    const int ntx = (g.dims[0] + TX - 1) / TX;
    const int nty = (g.dims[1] + TY - 1) / TY;
    const int bx = (int)(tile % (uint64_t)ntx);
    const uint64_t r = tile / (uint64_t)ntx;
    const int by = (int)(r % (uint64_t)nty);
    const int bz = (int)(r / (uint64_t)nty);
    const int i0 = bx * TX, j0 = by * TY, k0 = bz * TZ;

    __syncthreads();   // the previous tile of this workgroup is done with the LDS
    if (threadIdx.x < 3)
        s_cnt[threadIdx.x] = 0;
    for (int w = threadIdx.x; w < TV / 32; w += kBlock)
        s_alive[w] = 0;
    __syncthreads();
#pragma unroll
    for (int rr = 0; rr < TZ; ++rr) {
        const int s = rr * kBlock + (int)threadIdx.x;
        const int lx = s & (TX - 1), ly = (s >> LX) & (TY - 1), lz = s >> (LX + LY);
        const bool valid = i0 + lx < g.dims[0] && j0 + ly < g.dims[1] && k0 + lz < g.dims[2];
        lds_append(valid, (uint16_t)s, s_list[0], &s_cnt[0]);
    }
    __syncthreads();

    int cur = 0;
    for (int c0 = 0; c0 < ncam; c0 += kCamGroup) {
        const uint32_t n = s_cnt[cur % 3];
        if (n == 0)
            break;
        if (threadIdx.x == 0)
            s_cnt[(cur + 2) % 3] = 0;   // last read a pass ago, next appended to a pass on
        const float* P[kCamGroup];
        const uint32_t* sil[kCamGroup];
#pragma unroll
        for (int q = 0; q < kCamGroup; ++q) {
            const int c = c0 + q < ncam ? c0 + q : c0;   // wave-uniform
            P[q] = getP(c);
            sil[q] = sil_of(c);
        }
        const uint16_t* src = s_list[cur & 1];
        uint16_t* dst = s_list[(cur + 1) & 1];
        uint32_t* dcnt = &s_cnt[(cur + 1) % 3];
        // each wave takes 64 consecutive entries per round and stops as soon
        // as its next slice starts past the end of the list
        const uint32_t wave0 = (threadIdx.x / kWave) * kWave;
        for (uint32_t base = wave0; base < n; base += kBlock) {
            const uint32_t idx = base + lane_id();
            const bool act = idx < n;
            const int s = act ? src[idx] : 0;
            const int lx = s & (TX - 1), ly = (s >> LX) & (TY - 1), lz = s >> (LX + LY);
            const float X = lattice_coord(g.lo[0] + i0 + lx, g.h, g.origin[0]);
            const float Y = lattice_coord(g.lo[1] + j0 + ly, g.h, g.origin[1]);
            const float Z = lattice_coord(g.lo[2] + k0 + lz, g.h, g.origin[2]);
            // all tests of the group are issued unconditionally (a camera past
            // the last one repeats camera c0 and cannot change the result), so
            // their silhouette loads are in flight together
            const bool in = group_inside<kCamGroup>(P, X, Y, Z, sil, W, H, wpr);
            lds_append(act && in, (uint16_t)s, dst, dcnt);
        }
        __syncthreads();
        ++cur;
    }

    const uint32_t n_in = s_cnt[cur % 3];
    const uint16_t* surv = s_list[cur & 1];
    for (uint32_t base = 0; base < n_in; base += kBlock) {
        const uint32_t idx = base + threadIdx.x;
        const bool act = idx < n_in;
        const int s = act ? surv[idx] : 0;
        if (act)
            atomicOr(&s_alive[s >> 5], 1u << (s & 31));
    }
    __syncthreads();
    const uint64_t plane = (uint64_t)g.dims[0] * (uint64_t)g.dims[1];
#pragma unroll
    for (int rr = 0; rr < TZ; ++rr) {
        const int s = rr * kBlock + (int)threadIdx.x;
        const int lx = s & (TX - 1), ly = (s >> LX) & (TY - 1), lz = s >> (LX + LY);
        const int i = i0 + lx, j = j0 + ly, k = k0 + lz;
        const bool valid = i < g.dims[0] && j < g.dims[1] && k < g.dims[2];
        const uint32_t bit = (s_alive[s >> 5] >> (s & 31)) & 1u;
        if (valid)
            out[(uint64_t)k * plane + (uint64_t)j * g.dims[0] + i] = (uint8_t)bit;
        if (kBits != kBitsNone) {
            // lanes [TX*q, TX*q + TX) of the wave hold one tile row (lx = 0..TX-1)
            const uint64_t m = __ballot(valid && bit != 0u);
            const int q = lane_id() / TX;
            const uint64_t bits = TX == 64 ? m : (m >> (q * TX)) & ((1ull << (TX & 63)) - 1);
            const int64_t row = (int64_t)j + (int64_t)g.dims[1] * k;
            uint64_t* word = rb.words + row * rb.wr + (i0 >> 6);
            if (kBits == kBitsLabel && lx == 0 && bits != 0) {
                atomicOr((unsigned long long*)word, (unsigned long long)(bits << (i0 & 63)));
                atomicOr((unsigned long long*)&rb.rowmask[row >> 6], 1ull << (row & 63));
            }
            if (kBits == kBitsFine && lx == 0 && j < g.dims[1] && k < g.dims[2]) {
                if (TX == 64)
                    *word = bits;
                else if (TX == 32)
                    reinterpret_cast<uint32_t*>(word)[(i0 >> 5) & 1] = (uint32_t)bits;
                else
                    reinterpret_cast<uint16_t*>(word)[(i0 >> 4) & 3] = (uint16_t)bits;
            }
        }
    }
}

// ------------------------------------------------------------------ batched, persistent
// A job of a batched carve that the kernels can carve: 1..FVV_MAX_CAMS cameras
// of a valid image size, a non-empty lattice and non-negative offsets.
__device__ __forceinline__ bool job_ok(const fvv_job& j) {
    return j.n_cams >= 1 && j.n_cams <= FVV_MAX_CAMS && j.width >= 1 && j.height >= 1 &&
           j.width <= (1 << 16) && j.height <= (1 << 16) && j.grid.dims[0] >= 1 &&
           j.grid.dims[1] >= 1 && j.grid.dims[2] >= 1 && j.cam_base >= 0 && j.sil_base >= 0 &&
           j.out_offset >= 0;
}

// Prefix sums of the tiles over a host-given job table by one workgroup; resets
// the work counter.  counter[0] = next work item, [1] = tiles per item, [2] =
// jobs.  A job out of range gets no tiles and raises the job flag.
template <int TX, int TZ>
__global__ __launch_bounds__(kBlock) void batched_prepare_kernel(const fvv_job* __restrict__ jobs,
                                                                 uint32_t n_jobs,
                                                                 JobPrefix* __restrict__ pre,
                                                                 uint32_t* __restrict__ counter,
                                                                 uint32_t* __restrict__ status,
                                                                 uint32_t blocks) {
    __shared__ uint64_t scratch[kBlock / kWave];
    __shared__ uint64_t carry;
    if (threadIdx.x == 0)
        carry = 0;
    __syncthreads();
    for (uint32_t base = 0; base < n_jobs; base += kBlock) {
        uint32_t j = base + threadIdx.x;
        uint64_t t = 0;
        if (j < n_jobs) {
            if (job_ok(jobs[j]))
                t = tiles_of_grid(jobs[j].grid, TX, TZ);
            else
                atomicOr(status, kFlagJob);
        }
        uint64_t tot;
        const uint64_t ex = block_exclusive_sum64<kBlock>(t, scratch, &tot);
        const uint64_t c0 = carry;
        if (j < n_jobs)
            pre[j].tile_off = c0 + ex;
        __syncthreads();
        if (threadIdx.x == 0)
            carry = c0 + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        uint64_t total = carry;
        pre[n_jobs].tile_off = total;
        counter[0] = 0;
        counter[1] = grab_size(total, blocks);
        counter[2] = n_jobs;
    }
}

template <int TX, int TZ, bool kFineBits>
__global__ __launch_bounds__(kBlock) void carve_persistent_kernel(
    const fvv_job* __restrict__ jobs, const JobPrefix* __restrict__ pre,
    uint32_t* __restrict__ counter, const fvv_camera* __restrict__ cams,
    const uint32_t* __restrict__ sils, uint8_t* __restrict__ out, uint64_t* __restrict__ finebits) {
    __shared__ uint32_t s_item;
    const uint32_t nj = counter[2];
    const uint64_t per = counter[1];
    const uint64_t total = pre[nj].tile_off;
    for (;;) {
        if (threadIdx.x == 0)
            s_item = atomicAdd(&counter[0], 1u);
        __syncthreads();
        const uint64_t t0 = (uint64_t)s_item * per;
        __syncthreads();
        if (t0 >= total)
            break;
        const uint64_t t1 = t0 + per < total ? t0 + per : total;
        for (uint64_t t = t0; t < t1; ++t) {
            const int jb = upper_job([&](int m) { return pre[m].tile_off; }, (int)nj, t);
            const fvv_job job = jobs[jb];
            const int wpr = (job.width + 31) / 32;
            const int64_t cam_words = (int64_t)job.height * wpr;
            const fvv_camera* jc = cams + job.cam_base;
            const uint32_t* js = sils + job.sil_base;
            RowBits fb{};
            if (kFineBits) {
                fb.words = finebits + pre[jb].bit_off;
                fb.wr = (job.grid.dims[0] + 63) / 64;
            }
            carve_tile<TX, TZ, kFineBits ? kBitsFine : kBitsNone>(
                [&](int c) { return &jc[c].P[0]; }, [&](int c) { return js + c * cam_words; },
                job.n_cams, job.width, job.height, wpr, job.grid, t - pre[jb].tile_off,
                out + job.out_offset, fb);
        }
    }
}

// ------------------------------------------------------------------ frame fine carve, culled
// The fine carve of a frame classifies cameras per box of lattice samples
// before testing samples.  The projections of a box's samples lie in the
// convex hull of its eight corner projections (w > 0 over the whole lattice
// box wherever the rounding pad is finite), and the pad bounds how far a
// sample's floored quotient and the corners' rcp quotients can be from the
// real projections; so every sample's pixel lies in the corners' pixel
// rectangle widened by the pad.  If that rectangle holds no foreground pixel
// of the image, the camera rejects every sample of the box; if it lies inside
// the image and is all foreground, it accepts every sample.  Otherwise the
// camera is mixed for the box and its samples are tested one by one.  A tile
// (TX x TY x 4) is classified as 16 sub-blocks of 4 x 4 x 4 samples, one
// (sub-block, camera) pair per thread; one wave then carves one sub-block,
// lane = sample, testing only the sub-block's mixed cameras.  Results are
// identical to testing every camera: the skipped tests are decided by the
// rectangles.
constexpr int kCullMixed = 0, kCullAccept = 1, kCullReject = 2;

// Pixel rectangle from the corner quotient bounds [x0, x1] x [y0, y1] of a
// box: widened by the rounding pad, clamped a little outside the image (which
// keeps the conversions exact) and then to the image.  Returns kCullMixed when
// no pad bound holds, kCullReject when the rectangle misses the image, else -1
// with the clamped rectangle [cx0, cx1] x [cy0, cy1] and whether the unclamped
// one lies inside the image.
__device__ __forceinline__ int rect_of_bounds(float x0, float x1, float y0, float y1, float pad,
                                              int Wi, int Hi, int& cx0, int& cx1, int& cy0,
                                              int& cy1, bool& inside) {
    if (!(pad < 1.0f))
        return kCullMixed;
    const float W = (float)Wi, H = (float)Hi;
    const int px0 = (int)__builtin_floorf(__builtin_amdgcn_fmed3f(x0 - pad, -2.0f, W + 1.0f));
    const int px1 = (int)__builtin_floorf(__builtin_amdgcn_fmed3f(x1 + pad, -2.0f, W + 1.0f));
    const int py0 = (int)__builtin_floorf(__builtin_amdgcn_fmed3f(y0 - pad, -2.0f, H + 1.0f));
    const int py1 = (int)__builtin_floorf(__builtin_amdgcn_fmed3f(y1 + pad, -2.0f, H + 1.0f));
    inside = px0 >= 0 && py0 >= 0 && px1 < Wi && py1 < Hi;
    cx0 = max(px0, 0);
    cx1 = min(px1, Wi - 1);
    cy0 = max(py0, 0);
    cy1 = min(py1, Hi - 1);
    if (cx0 > cx1 || cy0 > cy1)
        return kCullReject;                    // every sample projects off the image
    return -1;
}

// Quotients of camera P at one corner of the box lo, hi (bit a of `corner`
// picks hi on axis a), with an rcp-based division.
__device__ __forceinline__ void corner_quotients(const float* P, const float* lo, const float* hi,
                                                 int corner, float& qa, float& qb) {
    const float X = (corner & 1) ? hi[0] : lo[0];
    const float Y = (corner & 2) ? hi[1] : lo[1];
    const float Z = (corner & 4) ? hi[2] : lo[2];
    const float a = __builtin_fmaf(P[2], Z, __builtin_fmaf(P[1], Y, __builtin_fmaf(P[0], X, P[3])));
    const float b = __builtin_fmaf(P[6], Z, __builtin_fmaf(P[5], Y, __builtin_fmaf(P[4], X, P[7])));
    const float w =
        __builtin_fmaf(P[10], Z, __builtin_fmaf(P[9], Y, __builtin_fmaf(P[8], X, P[11])));
    const float r = __builtin_amdgcn_rcpf(w);
    qa = a * r;
    qb = b * r;
}

// Pixel rectangle of camera c over the box of samples with world corners lo,
// hi (see rect_of_bounds).
template <class Cams>
__device__ __forceinline__ int box_rect(const Cams& cams, int c, const float* lo, const float* hi,
                                        int& cx0, int& cx1, int& cy0, int& cy1, bool& inside) {
    const float pad = cams.padc(c);
    if (!(pad < 1.0f))
        return kCullMixed;
    const float* P = cams.Pc(c);
    float x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        float qa, qb;
        corner_quotients(P, lo, hi, k, qa, qb);
        x0 = fminf(x0, qa);
        x1 = fmaxf(x1, qa);
        y0 = fminf(y0, qb);
        y1 = fmaxf(y1, qb);
    }
    return rect_of_bounds(x0, x1, y0, y1, pad, cams.W, cams.H, cx0, cx1, cy0, cy1, inside);
}

// Lane permutations within aligned groups of 8 lanes (DPP): swap neighbours,
// swap pairs, swap quads.
template <int kCtrl>
__device__ __forceinline__ float dpp_f32(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, false));
}

__device__ __forceinline__ float min8(float v) {
    v = fminf(v, dpp_f32<0xB1>(v));    // quad_perm [1,0,3,2]
    v = fminf(v, dpp_f32<0x4E>(v));    // quad_perm [2,3,0,1]
    return fminf(v, dpp_f32<0x141>(v));  // row_half_mirror
}

__device__ __forceinline__ float max8(float v) {
    v = fmaxf(v, dpp_f32<0xB1>(v));
    v = fmaxf(v, dpp_f32<0x4E>(v));
    return fmaxf(v, dpp_f32<0x141>(v));
}

// Foreground test of row y of silhouette `sil` over columns [cx0, cx1], at
// most kWords words from word w0: any / all of the pixels set.
template <int kWords>
__device__ __forceinline__ void row_any_all(const uint32_t* __restrict__ row, int cx0, int cx1,
                                            bool on, bool& any, bool& all) {
    const int w0 = cx0 >> 5, w1 = cx1 >> 5;
#pragma unroll
    for (int q = 0; q < kWords; ++q) {
        const int wq = w0 + q;
        const bool won = on && wq <= w1;
        const uint32_t lo_m = wq == w0 ? ~0u << (cx0 & 31) : ~0u;
        const uint32_t hi_m = wq == w1 ? (~0u >> (31 - (cx1 & 31))) : ~0u;
        const uint32_t m = won ? (lo_m & hi_m) : 0u;
        uint32_t v = 0;
        if (won)
            v = row[wq];
        any |= (v & m) != 0u;
        all &= (v & m) == m;
    }
}

// Classification of camera c for the box of samples with world corners lo,
// hi: rectangles of more than kRows rows or kWords silhouette words count as
// mixed.
template <int kRows, int kWords, class Cams>
__device__ __forceinline__ int classify_box(const Cams& cams, int c,
                                            const uint32_t* __restrict__ sil, const float* lo,
                                            const float* hi) {
    int cx0, cx1, cy0, cy1;
    bool inside;
    const int r0 = box_rect(cams, c, lo, hi, cx0, cx1, cy0, cy1, inside);
    if (r0 >= 0)
        return r0;
    if (cy1 - cy0 >= kRows || (cx1 >> 5) - (cx0 >> 5) >= kWords)
        return kCullMixed;
    bool any = false, all = true;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const bool row_on = r <= cy1 - cy0;
        row_any_all<kWords>(sil + (row_on ? cy0 + r : cy0) * cams.wpr, cx0, cx1, row_on, any,
                            all);
    }
    if (!any)
        return kCullReject;
    return (inside && all) ? kCullAccept : kCullMixed;
}

// Classification of every camera for the box lo, hi by one wave, four cameras
// per pass: the 16 lanes of camera cb + l/16 project one corner each (lanes
// l%8) and reduce the corner bounds over 8 lanes, then test row l%16 of the
// rectangle (rectangles of more than 16 rows or kWords words count as mixed).
// Returns, uniform over the wave, the cameras that reject every sample of the
// box and those that are mixed; the others accept every sample.  kStop: leave
// after the first pass with a rejecting camera (mixed is then incomplete).
template <int kWords, bool kStop = false, class Cams>
__device__ __forceinline__ void classify_box_wave(const Cams& cams,
                                                  const uint32_t* __restrict__ sils,
                                                  int64_t cam_words, const float* lo,
                                                  const float* hi, uint32_t& reject,
                                                  uint32_t& mixed) {
    const int lane = lane_id(), r = lane & 15, grp = lane >> 4;
    reject = 0;
    mixed = 0;
    for (int cb = 0; cb < cams.n; cb += 4) {
        const int c = cb + grp;
        const bool cam_on = c < cams.n;
        const int cc = cam_on ? c : cb;
        float qa, qb;
        corner_quotients(cams.Pc(cc), lo, hi, lane & 7, qa, qb);
        const float x0 = min8(qa), x1 = max8(qa), y0 = min8(qb), y1 = max8(qb);
        int cx0, cx1, cy0, cy1;
        bool inside = false;
        int st = rect_of_bounds(x0, x1, y0, y1, cams.padc(cc), cams.W, cams.H, cx0, cx1, cy0, cy1,
                                inside);
        if (st < 0 && (cy1 - cy0 >= 16 || (cx1 >> 5) - (cx0 >> 5) >= kWords))
            st = kCullMixed;
        bool any = false, all = true;
        if (cam_on && st < 0) {
            const bool row_on = r <= cy1 - cy0;
            row_any_all<kWords>(sils + cc * cam_words + (row_on ? cy0 + r : cy0) * cams.wpr, cx0,
                                cx1, row_on, any, all);
        }
        const uint32_t gany = (uint32_t)(__ballot(any) >> (16 * grp)) & 0xffffu;
        const uint32_t gall = (uint32_t)(__ballot(all) >> (16 * grp)) & 0xffffu;
        const bool rej = cam_on && (st == kCullReject || (st < 0 && gany == 0));
        const bool acc = cam_on && st < 0 && gany != 0 && inside && gall == 0xffffu;
        const uint64_t rb = __ballot(r == 0 && rej), mb = __ballot(r == 0 && cam_on && !rej && !acc);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            reject |= (uint32_t)((rb >> (16 * g)) & 1u) << (cb + g);
            mixed |= (uint32_t)((mb >> (16 * g)) & 1u) << (cb + g);
        }
        if (kStop && reject != 0u)
            return;
    }
}

// World corners of the samples [i0, i1] x [j0, j1] x [k0, k1] of lattice g.
__device__ __forceinline__ void box_corners(const fvv_grid& g, int i0, int i1, int j0, int j1,
                                            int k0, int k1, float* lo, float* hi) {
    lo[0] = lattice_coord(g.lo[0] + i0, g.h, g.origin[0]);
    hi[0] = lattice_coord(g.lo[0] + i1, g.h, g.origin[0]);
    lo[1] = lattice_coord(g.lo[1] + j0, g.h, g.origin[1]);
    hi[1] = lattice_coord(g.lo[1] + j1, g.h, g.origin[1]);
    lo[2] = lattice_coord(g.lo[2] + k0, g.h, g.origin[2]);
    hi[2] = lattice_coord(g.lo[2] + k1, g.h, g.origin[2]);
}

// Tile t of lattice g (x fastest, then y, then z): its first sample.
template <int TX>
__device__ __forceinline__ void tile_origin(const fvv_grid& g, uint64_t tile, int& i0, int& j0,
                                            int& k0) {
    constexpr int TY = kBlock / TX;
    const int ntx = (g.dims[0] + TX - 1) / TX;
    const int nty = (g.dims[1] + TY - 1) / TY;
    int bx, by, bz;
    if ((tile >> 32) == 0) {                    // 32-bit index arithmetic where it fits
        const uint32_t t32 = (uint32_t)tile, rq = t32 / (uint32_t)ntx;
        bx = (int)(t32 - rq * (uint32_t)ntx);
        by = (int)(rq % (uint32_t)nty);
        bz = (int)(rq / (uint32_t)nty);
    } else {
        const uint64_t rq = tile / (uint64_t)ntx;
        bx = (int)(tile - rq * (uint64_t)ntx);
        by = (int)(rq % (uint64_t)nty);
        bz = (int)(rq / (uint64_t)nty);
    }
    i0 = bx * TX;
    j0 = by * TY;
    k0 = bz * 4;
}

// ------------------------------------------------------------------ one lattice
template <int TX, int TZ, bool kRows>
__global__ __launch_bounds__(kBlock) void carve_kernel(const CamSet cams,
                                                       const uint32_t* __restrict__ sils,
                                                       const fvv_grid g, uint8_t* __restrict__ occ,
                                                       const RowBits rb) {
    const int64_t cam_words = (int64_t)cams.H * cams.wpr;
    carve_tile<TX, TZ, kRows ? kBitsLabel : kBitsNone>([&](int c) { return &cams.P[c][0]; },
                              [&](int c) { return sils + c * cam_words; }, cams.n, cams.W, cams.H,
                              cams.wpr, g, blockIdx.x, occ, rb);
}

// Large lattices, most of whose samples lie far from every silhouette, in two
// passes over boxes of 8 x 8 x 4 samples (compact boxes project to small
// rectangles, so more of them are rejected whole than flat tiles of the same
// size): carve_reject_kernel zeroes the occupancy and marks the boxes that no
// camera rejects whole; carve_kept_kernel carves the marked boxes.
constexpr int kRejRows = 16;   // block rows of a rectangle read for a rejection

// Whether the camera cam (P, then the rounding pad) sees no foreground pixel
// in the padded rectangle of the box lo, hi (then no sample of the box is
// occupied), by one lane: the bounds of the 8 corners' quotients, then the
// silhouette's non-empty 8 x 8-pixel blocks under the rectangle (sb: this
// camera's block rows), eight rows at a time until one is non-empty.  A
// rectangle of more than kRejRows block rows or two words of blocks rejects
// nothing.
__device__ __forceinline__ bool cam_rejects_box(const float* cam, int W, int H,
                                                const uint64_t* __restrict__ sb, int bw,
                                                const float* lo, const float* hi) {
    float x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        // the (y, z) partial sums, shared by the two corners on x
        const float Y = (k & 1) ? hi[1] : lo[1], Z = (k & 2) ? hi[2] : lo[2];
        const float ayz = __builtin_fmaf(cam[2], Z, __builtin_fmaf(cam[1], Y, cam[3]));
        const float byz = __builtin_fmaf(cam[6], Z, __builtin_fmaf(cam[5], Y, cam[7]));
        const float wyz = __builtin_fmaf(cam[10], Z, __builtin_fmaf(cam[9], Y, cam[11]));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float X = e ? hi[0] : lo[0];
            const float a = __builtin_fmaf(cam[0], X, ayz);
            const float b = __builtin_fmaf(cam[4], X, byz);
            const float w = __builtin_fmaf(cam[8], X, wyz);
            const float r = __builtin_amdgcn_rcpf(w);
            x0 = fminf(x0, a * r);
            x1 = fmaxf(x1, a * r);
            y0 = fminf(y0, b * r);
            y1 = fmaxf(y1, b * r);
        }
    }
    int cx0, cx1, cy0, cy1;
    bool inside;
    const int st = rect_of_bounds(x0, x1, y0, y1, cam[12], W, H, cx0, cx1, cy0, cy1, inside);
    if (st >= 0)
        return st == kCullReject;
    const int by0 = cy0 >> 3, nby = (cy1 >> 3) - by0 + 1;
    const int bx0 = cx0 >> 3, bx1 = cx1 >> 3, w0 = bx0 >> 6;
    if (nby > kRejRows || (bx1 >> 6) - w0 > 1)
        return false;
    const bool two = (bx1 >> 6) != w0;
    const uint64_t m0 = (~0ull << (bx0 & 63)) & (two ? ~0ull : ~0ull >> (63 - (bx1 & 63)));
    const uint64_t m1 = two ? ~0ull >> (63 - (bx1 & 63)) : 0ull;
    // each batch's loads in bounds and issued at once: rows past the
    // rectangle repeat its last row, the second word repeats the first where
    // there is none
    const uint64_t* row = sb + (int64_t)by0 * bw + w0;
    const int w1 = two ? 1 : 0;
    uint64_t acc = 0ull;
    for (int r0 = 0; r0 < nby && acc == 0ull; r0 += 8) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const uint64_t* rr = row + (int64_t)min(r0 + r, nby - 1) * bw;
            acc |= (rr[0] & m0) | (rr[w1] & m1);
        }
    }
    return acc == 0ull;
}

// The boxes of the two-pass carve: nbx x nby x nbz boxes of 8 x 8 x 4 samples,
// x fastest; with the divisions by nbx and nby.
struct RejBoxes {
    uint32_t n, nbx, nby;
    DivU32 by_nbx, by_nby;
};


__device__ __forceinline__ void rej_box_origin(const RejBoxes& bx, uint32_t b, int& i0, int& j0,
                                               int& k0) {
    const uint32_t q = divu32(b, bx.by_nbx), bz = divu32(q, bx.by_nby);
    i0 = 8 * (int)(b - q * bx.nbx);
    j0 = 8 * (int)(q - bz * bx.nby);
    k0 = 4 * (int)bz;
}

// Zeros over the whole occupancy (16-byte stores between the first and the
// last 16-byte boundary), then one thread per (box, camera): a workgroup
// takes per_wg = min(256 / cameras, 64) boxes (cam_of: division by the camera
// count), each camera that rejects a box marks it in LDS, and the
// boxes no camera rejects are appended to list (one atomic on *count per
// workgroup that keeps any; *count is 0 before, order unspecified).
__global__ __launch_bounds__(kBlock) void carve_reject_kernel(const CamSet cams,
                                                              const SilAny sa, const fvv_grid g,
                                                              uint8_t* __restrict__ occ,
                                                              const RejBoxes boxes, int per_wg,
                                                              DivU32 cam_of,
                                                              uint32_t* __restrict__ list,
                                                              uint32_t* __restrict__ count) {
    __shared__ float s_cam[FVV_MAX_CAMS][13];
    __shared__ uint32_t s_rej[kBlock];
    for (int i = threadIdx.x; i < cams.n * 13; i += kBlock) {
        const int c = i / 13, e = i - 13 * c;
        s_cam[c][e] = e < 12 ? cams.P[c][e] : cams.pad[c];
    }
    s_rej[threadIdx.x] = 0u;
    const uint64_t V = (uint64_t)g.dims[0] * (uint64_t)g.dims[1] * (uint64_t)g.dims[2];
    const uint64_t tid = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    const uint64_t nth = (uint64_t)gridDim.x * kBlock;
    const uint64_t mis = (16u - (uint32_t)(reinterpret_cast<uintptr_t>(occ) & 15u)) & 15u;
    const uint64_t head = mis < V ? mis : V;
    const uint64_t n16 = (V - head) >> 4, tail0 = head + (n16 << 4);
    uint4* const body = reinterpret_cast<uint4*>(occ + head);
    for (uint64_t i = tid; i < n16; i += nth)
        body[i] = make_uint4(0u, 0u, 0u, 0u);
    if (tid < head)
        occ[tid] = 0;
    if (tid < V - tail0)
        occ[tail0 + tid] = 0;
    __syncthreads();

    const uint32_t bl = divu32(threadIdx.x, cam_of);
    const int c = (int)(threadIdx.x - bl * (uint32_t)cams.n);
    const uint32_t b = blockIdx.x * (uint32_t)per_wg + bl;
    if (bl < (uint32_t)per_wg && b < boxes.n) {
        int i0, j0, k0;
        rej_box_origin(boxes, b, i0, j0, k0);
        float lo[3], hi[3];
        box_corners(g, i0, min(i0 + 8, g.dims[0]) - 1, j0, min(j0 + 8, g.dims[1]) - 1, k0,
                    min(k0 + 4, g.dims[2]) - 1, lo, hi);
        if (cam_rejects_box(s_cam[c], cams.W, cams.H, sa.bits + (int64_t)c * sa.tph * sa.bw,
                            sa.bw, lo, hi))
            s_rej[bl] = 1u;
    }
    __syncthreads();
    if (threadIdx.x < kWave) {   // per_wg <= 64: the first wave holds every box's flag
        const uint32_t bb = blockIdx.x * (uint32_t)per_wg + threadIdx.x;
        const bool kept = threadIdx.x < (unsigned)per_wg && bb < boxes.n && !s_rej[threadIdx.x];
        const uint64_t km = __ballot(kept);
        if (km) {
            uint32_t at = 0u;
            if (threadIdx.x == 0)
                at = atomicAdd(count, (uint32_t)__popcll(km));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
            if (kept)
                list[at + lane_rank(km)] = bb;
        }
    }
}

// One z layer (8 x 8 samples) of a kept box by one wave: lane (x, y) = (l % 8,
// l / 8) holds one sample, tested against 16 cameras at a time in one call
// (cam: matrices and pads in LDS; a camera past the last repeats the last)
// until it is out or the cameras are; then its occupancy byte and, with
// kRows, the labelling's row bits (a box row's 8 bits ORed into its word).
template <bool kRows>
__device__ __forceinline__ void carve_box_layer(const float (*cam)[13],
                                                const uint32_t* __restrict__ sils,
                                                int64_t cam_words, int ncam, int W, int H,
                                                int wpr, const fvv_grid& g, int i0, int j0, int k,
                                                uint8_t* __restrict__ out, const RowBits& rb) {
    const int lane = lane_id();
    const int i = i0 + (lane & 7), j = j0 + (lane >> 3);
    bool alive = i < g.dims[0] && j < g.dims[1] && k < g.dims[2];
    const bool valid = alive;
    const float X = lattice_coord(g.lo[0] + i, g.h, g.origin[0]);
    const float Y = lattice_coord(g.lo[1] + j, g.h, g.origin[1]);
    const float Z = lattice_coord(g.lo[2] + k, g.h, g.origin[2]);
    for (int c0 = 0; c0 < ncam && __ballot(alive) != 0ull; c0 += 16) {
        const float* P[16];
        const uint32_t* S[16];
        float Xs[16], Ys[16], Zs[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int c = min(c0 + q, ncam - 1);
            P[q] = cam[c];
            S[q] = sils + c * cam_words;
            Xs[q] = X;
            Ys[q] = Y;
            Zs[q] = Z;
        }
        alive = alive && multi_inside<16>(P, Xs, Ys, Zs, S, W, H, wpr) == 0xffffu;
    }
    if (valid)
        out[(uint64_t)k * g.dims[0] * (uint64_t)g.dims[1] + (uint64_t)j * g.dims[0] + i] =
            alive ? 1 : 0;
    if (kRows) {
        const uint64_t bits = (__ballot(alive) >> (8 * (lane >> 3))) & 0xffull;
        if ((lane & 7) == 0 && bits != 0) {
            const int64_t row = (int64_t)j + (int64_t)g.dims[1] * k;
            atomicOr((unsigned long long*)(rb.words + row * rb.wr + (i0 >> 6)),
                     (unsigned long long)(bits << (i0 & 63)));
            atomicOr((unsigned long long*)&rb.rowmask[row >> 6], 1ull << (row & 63));
        }
    }
}

// The kept boxes (list, *count of them): workgroup w of G carves entries w, w +
// G, ... with its four waves, one z layer each; any_bits (any_words words)
// zeroed.
template <bool kRows>
__global__ __launch_bounds__(kBlock) void carve_kept_kernel(const CamSet cams,
                                                            const uint32_t* __restrict__ sils,
                                                            const fvv_grid g,
                                                            uint8_t* __restrict__ occ,
                                                            const RowBits rb,
                                                            const uint32_t* __restrict__ list,
                                                            const uint32_t* __restrict__ count,
                                                            const RejBoxes boxes,
                                                            uint64_t* __restrict__ any_bits,
                                                            int64_t any_words) {
    __shared__ float s_cam[FVV_MAX_CAMS][13];
    for (int i = threadIdx.x; i < cams.n * 13; i += kBlock) {
        const int c = i / 13, e = i - 13 * c;
        s_cam[c][e] = e < 12 ? cams.P[c][e] : cams.pad[c];
    }
    // the non-empty blocks, read by the first pass, cleared for the next frame
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < any_words;
         i += (int64_t)gridDim.x * kBlock)
        any_bits[i] = 0ull;
    __syncthreads();
    const int64_t cam_words = (int64_t)cams.H * cams.wpr;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t n = min(*count, boxes.n);
    for (uint32_t q = blockIdx.x; q < n; q += gridDim.x) {
        int i0, j0, k0;
        rej_box_origin(boxes, list[q], i0, j0, k0);
        carve_box_layer<kRows>(s_cam, sils, cam_words, cams.n, cams.W, cams.H, cams.wpr, g, i0,
                               j0, k0 + wave, occ, rb);
    }
}

// Camera classification of a whole culled tile (TX x TY x 4 samples from
// i0, j0, k0) by one wave: rejecting and mixed cameras, uniform over the wave.
template <int TX, int kWords = 2, bool kStop = false, class Cams>
__device__ __forceinline__ void classify_tile(const Cams& cams, const uint32_t* __restrict__ sils,
                                              const fvv_grid& g, int i0, int j0, int k0,
                                              uint32_t& reject, uint32_t& mixed) {
    constexpr int TY = kBlock / TX;
    float lo[3], hi[3];
    box_corners(g, i0, min(i0 + TX, g.dims[0]) - 1, j0, min(j0 + TY, g.dims[1]) - 1, k0,
                min(k0 + 4, g.dims[2]) - 1, lo, hi);
    classify_box_wave<kWords, kStop>(cams, sils, (int64_t)cams.H * cams.wpr, lo, hi, reject, mixed);
}

// One culled tile (first sample i0, j0, k0).  tile_off (uniform): a camera
// rejects the whole tile, which
// is written as zeros with no other work; tile_mixed: the cameras left to
// classify per sub-block (cameras outside it accept the whole tile).  rb:
// nothing (words null), a fine bitmap (rows of whole words written), or the
// labelling's row bitmap (rowmask set: bits ORed in, rows marked).  Every
// LDS read of a tile happens before its last barrier except the s_occ reads
// of the output pass, and the next tile writes s_occ only after two barriers,
// so consecutive tiles need no barrier between them.
template <int TX, class Cams>
__device__ __forceinline__ void carve_tile_culled(const Cams& cams,
                                                  const uint32_t* __restrict__ sils,
                                                  const fvv_grid& g, int i0, int j0, int k0,
                                                  uint8_t* __restrict__ out, const RowBits& rb,
                                                  bool tile_off = false,
                                                  uint32_t tile_mixed = ~0u) {
    constexpr int TY = kBlock / TX, TZ = 4;
    constexpr int TV = TX * TY * TZ;
    constexpr int SBX = TX / 4;                 // sub-blocks along x (16 in all)
    constexpr int LX = log2_of(TX), LY = log2_of(TY);
    __shared__ uint8_t s_occ[TV];
    __shared__ uint32_t s_mixed[16];
    __shared__ uint32_t s_reject;
    const int64_t cam_words = (int64_t)cams.H * cams.wpr;
    const int tk1 = min(k0 + TZ, g.dims[2]) - 1;
    const int wave = threadIdx.x / kWave, lane = lane_id();

    if (!tile_off) {
        if (threadIdx.x < 16)
            s_mixed[threadIdx.x] = 0;
        if (threadIdx.x == 0)
            s_reject = 0;
        __syncthreads();
        for (int p = threadIdx.x; p < 16 * cams.n; p += kBlock) {
            const int b = p & 15, c = p >> 4;
            const int si0 = i0 + (b % SBX) * 4, sj0 = j0 + (b / SBX) * 4;
            if (si0 >= g.dims[0] || sj0 >= g.dims[1] || !((tile_mixed >> c) & 1u))
                continue;
            float lo[3], hi[3];
            box_corners(g, si0, min(si0 + 4, g.dims[0]) - 1, sj0, min(sj0 + 4, g.dims[1]) - 1,
                        k0, tk1, lo, hi);
            const int cl = classify_box<6, 2>(cams, c, sils + c * cam_words, lo, hi);
            if (cl == kCullReject)
                atomicOr(&s_reject, 1u << b);
            else if (cl == kCullMixed)
                atomicOr(&s_mixed[b], 1u << c);
        }
        __syncthreads();
        // one wave per sub-block, lane = sample (x fastest, then y, then z)
        for (int b = wave; b < 16; b += kBlock / kWave) {
            const int lx = (b % SBX) * 4 + (lane & 3);
            const int ly = (b / SBX) * 4 + ((lane >> 2) & 3);
            const int lz = lane >> 4;
            const bool valid = i0 + lx < g.dims[0] && j0 + ly < g.dims[1] && k0 + lz < g.dims[2];
            bool alive = valid && !((s_reject >> b) & 1u);
            if (__ballot(alive) != 0) {
                const float X = lattice_coord(g.lo[0] + i0 + lx, g.h, g.origin[0]);
                const float Y = lattice_coord(g.lo[1] + j0 + ly, g.h, g.origin[1]);
                const float Z = lattice_coord(g.lo[2] + k0 + lz, g.h, g.origin[2]);
                // wave-uniform: the sub-block's mixed cameras, two per pass
                uint32_t rest = s_mixed[b];
                while (rest && __ballot(alive) != 0) {
                    const int ca = __ffs(rest) - 1;
                    rest &= rest - 1;
                    if (rest) {
                        const int cb = __ffs(rest) - 1;
                        rest &= rest - 1;
                        const float* P2[2] = {cams.Pc(ca), cams.Pc(cb)};
                        const uint32_t* S2[2] = {sils + ca * cam_words,
                                                 sils + cb * cam_words};
                        alive = alive &&
                                group_inside<2>(P2, X, Y, Z, S2, cams.W, cams.H, cams.wpr);
                    } else {
                        const float* P1[1] = {cams.Pc(ca)};
                        const uint32_t* S1[1] = {sils + ca * cam_words};
                        alive = alive &&
                                group_inside<1>(P1, X, Y, Z, S1, cams.W, cams.H, cams.wpr);
                    }
                }
            }
            s_occ[lx + TX * (ly + TY * lz)] = alive ? 1 : 0;
        }
        __syncthreads();
    }
    // output: thread (lx, ly) writes sample row ly, column lx of every z layer
    const uint64_t plane = (uint64_t)g.dims[0] * (uint64_t)g.dims[1];
    const int lx = threadIdx.x & (TX - 1), ly = threadIdx.x >> LX;
    const int i = i0 + lx, j = j0 + ly;
    const bool vxy = i < g.dims[0] && j < g.dims[1];
    uint8_t* const o = out + ((uint64_t)k0 * plane + (uint64_t)j * (uint64_t)g.dims[0] + i);
    if (tile_off && (!rb.words || rb.rowmask)) {   // zeros; a label bitmap gets no bits
        const int nzr = min(TZ, g.dims[2] - k0);
        if (vxy)
            for (int rr = 0; rr < nzr; ++rr)
                o[rr * plane] = 0;
        return;
    }
#pragma unroll
    for (int rr = 0; rr < TZ; ++rr) {
        const int k = k0 + rr;
        const bool valid = vxy && k < g.dims[2];
        const uint8_t bit = tile_off ? 0 : s_occ[rr * kBlock + threadIdx.x];
        if (valid)
            o[rr * plane] = bit;
        // fine bitmap: lanes [TX*q, TX*q + TX) of the wave hold one tile row
        const uint64_t m = __ballot(valid && bit != 0);
        const int q = lane_id() / TX;
        const uint64_t bits = TX == 64 ? m : (m >> (q * TX)) & ((1ull << (TX & 63)) - 1);
        if (rb.words && lx == 0 && j < g.dims[1] && k < g.dims[2]) {
            const int64_t row = (int64_t)j + (int64_t)g.dims[1] * k;
            uint64_t* word = rb.words + row * rb.wr + (i0 >> 6);
            if (rb.rowmask) {
                // the labelling's row bitmap (all-zero before the carve): OR in
                // the set bits and mark the row
                if (bits) {
                    atomicOr((unsigned long long*)word, (unsigned long long)(bits << (i0 & 63)));
                    atomicOr((unsigned long long*)&rb.rowmask[row >> 6], 1ull << (row & 63));
                }
            } else if (TX == 64) {
                *word = bits;
            } else if (TX == 32) {
                reinterpret_cast<uint32_t*>(word)[(i0 >> 5) & 1] = (uint32_t)bits;
            } else {
                reinterpret_cast<uint16_t*>(word)[(i0 >> 4) & 3] = (uint16_t)bits;
            }
        }
    }
}

// One lattice with camera culling (tiles of depth 4): one tile per workgroup,
// the whole-tile classification by the first wave, then the sub-block culling
// of carve_tile_culled.  The camera set's rounding pads must hold over the
// lattice's box (infinite pads leave every camera mixed).
template <int TX>
__global__ __launch_bounds__(kBlock) void carve_culled_kernel(const CamSet cams,
                                                              const uint32_t* __restrict__ sils,
                                                              const fvv_grid g,
                                                              uint8_t* __restrict__ occ,
                                                              const RowBits rb) {
    __shared__ uint32_t s_cls[2];
    int i0, j0, k0;
    tile_origin<TX>(g, blockIdx.x, i0, j0, k0);
    if (threadIdx.x < kWave) {
        uint32_t rej, mix;
        classify_tile<TX>(cams, sils, g, i0, j0, k0, rej, mix);
        if (threadIdx.x == 0) {
            s_cls[0] = rej;
            s_cls[1] = mix;
        }
    }
    __syncthreads();
    const uint32_t rej = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_cls[0]);
    const uint32_t mix = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_cls[1]);
    carve_tile_culled<TX>(cams, sils, g, i0, j0, k0, occ, rb, rej != 0, mix);
}

// Any and all of the pixels [cx0, cx1] x [cy0, cy1] (inside the image) of one
// camera's tiled silhouette tc, when the rectangle lies in at most 2 x 2
// blocks; false (nothing examined) when it spans more.
__device__ __forceinline__ bool rect_any_all_tiled(const uint64_t* __restrict__ tc, int tpr,
                                                   int cx0, int cx1, int cy0, int cy1, bool& any,
                                                   bool& all) {
    const int bx0 = cx0 >> 3, bx1 = cx1 >> 3, by0 = cy0 >> 3, by1 = cy1 >> 3;
    if (bx1 - bx0 > 1 || by1 - by0 > 1)
        return false;
    uint64_t v[4], m[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int bx = bx0 + (d & 1), by = by0 + (d >> 1);
        const bool on = bx <= bx1 && by <= by1;
        // the rectangle's columns and rows within the block (already inside
        // [0, 7] for a block the rectangle touches; clamped for the others)
        const int c0 = min(max(cx0 - 8 * bx, 0), 7), c1 = min(max(cx1 - 8 * bx, 0), 7);
        const int r0 = min(max(cy0 - 8 * by, 0), 7), r1 = min(max(cy1 - 8 * by, 0), 7);
        const uint64_t cols = (uint64_t)((2u << c1) - (1u << c0)) * 0x0101010101010101ull;
        const uint64_t rows = (~0ull >> (8 * (7 - r1))) & (~0ull << (8 * r0));
        m[d] = on ? cols & rows : 0ull;
        v[d] = 0;
        if (on)
            v[d] = tc[(int64_t)by * tpr + bx];
    }
    any = false;
    all = true;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        any |= (v[d] & m[d]) != 0ull;
        all &= (v[d] & m[d]) == m[d];
    }
    return true;
}

// Classification of one camera for the box of samples with world corners lo,
// hi: reject (no foreground pixel in the padded rectangle), accept (inside the
// image and all foreground) or mixed (also for rectangles of more than 2 x 2
// tiled blocks).  cam: P (12 floats) and the rounding pad.  The corners'
// projection rows are the chains of three fmas in the order z, y, x (the
// rounding pad bounds a chain's error in any order), so the (y, z) partial
// sums are shared by the two corners on x.
__device__ __forceinline__ int classify_box_tiled(const float* cam, int W, int H,
                                                  const uint64_t* __restrict__ tc, int tpr,
                                                  const float* lo, const float* hi) {
    const float pad = cam[12];
    if (!(pad < 1.0f))
        return kCullMixed;
    float x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float Y = (k & 1) ? hi[1] : lo[1], Z = (k & 2) ? hi[2] : lo[2];
        const float ayz = __builtin_fmaf(cam[1], Y, __builtin_fmaf(cam[2], Z, cam[3]));
        const float byz = __builtin_fmaf(cam[5], Y, __builtin_fmaf(cam[6], Z, cam[7]));
        const float wyz = __builtin_fmaf(cam[9], Y, __builtin_fmaf(cam[10], Z, cam[11]));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float X = e ? hi[0] : lo[0];
            const float a = __builtin_fmaf(cam[0], X, ayz);
            const float b = __builtin_fmaf(cam[4], X, byz);
            const float w = __builtin_fmaf(cam[8], X, wyz);
            const float r = __builtin_amdgcn_rcpf(w);
            const float qa = a * r, qb = b * r;
            x0 = fminf(x0, qa);
            x1 = fmaxf(x1, qa);
            y0 = fminf(y0, qb);
            y1 = fmaxf(y1, qb);
        }
    }
    int cx0, cx1, cy0, cy1;
    bool inside;
    const int r0 = rect_of_bounds(x0, x1, y0, y1, pad, W, H, cx0, cx1, cy0, cy1, inside);
    if (r0 >= 0)
        return r0;
    bool any, all;
    if (!rect_any_all_tiled(tc, tpr, cx0, cx1, cy0, cy1, any, all))
        return kCullMixed;
    if (!any)
        return kCullReject;
    return (inside && all) ? kCullAccept : kCullMixed;
}

// The pixel of camera P (12 floats) for the point (X, Y, Z) as the occupancy
// test floors it (sil_test up to the silhouette word): px, py, and whether
// w > 0 and the pixel lies in the W x H image.
__device__ __forceinline__ bool point_pixel_exact(const float* __restrict__ P, float X, float Y,
                                                  float Z, int W, int H, int& px, int& py) {
    const float a = __builtin_fmaf(P[2], Z, __builtin_fmaf(P[1], Y, __builtin_fmaf(P[0], X, P[3])));
    const float b = __builtin_fmaf(P[6], Z, __builtin_fmaf(P[5], Y, __builtin_fmaf(P[4], X, P[7])));
    const float w =
        __builtin_fmaf(P[10], Z, __builtin_fmaf(P[9], Y, __builtin_fmaf(P[8], X, P[11])));
    const float r = __builtin_amdgcn_rcpf(w);
    float qa = a * r, qb = b * r;
    const bool tiny = w > 0.0f && w < 0x1p-64f;
    if (__builtin_expect(__ballot(tiny) != 0, 0)) {
        if (tiny) {
            qa = a / w;
            qb = b / w;
        }
    }
    qa = __builtin_amdgcn_fmed3f(qa, -4.0f, (float)W + 4.0f);
    qb = __builtin_amdgcn_fmed3f(qb, -4.0f, (float)H + 4.0f);
    px = exact_floor(a, w, qa);
    py = exact_floor(b, w, qb);
    return (w > 0.0f) & ((unsigned)px < (unsigned)W) & ((unsigned)py < (unsigned)H);
}

// The pixels of the rectangle [cx0, cx0 + 7] x [cy0, cy0 + 7] of one camera's
// tiled silhouette tc as one 64-bit window, bit 8 r + c = pixel (cx0 + c,
// cy0 + r), from the up to 2 x 2 blocks around its corner (nx, ny: whether the
// rectangle's last column / row, cx1 / cy1, lie in the next block; pixels past
// the image are 0).  Rows are shifted up by cy0 % 8, then each row's pixels
// right by cx0 % 8 with the next block's pixels shifted in.
__device__ __forceinline__ uint64_t tiled_window(const uint64_t* __restrict__ tc, int tpr,
                                                 int cx0, int cy0, bool nx, bool ny, bool on) {
    const uint64_t* tb = tc + (int64_t)(cy0 >> 3) * tpr + (cx0 >> 3);
    uint64_t b0 = 0, b1 = 0, b2 = 0, b3 = 0;
    if (on)
        b0 = tb[0];
    if (on && nx)
        b1 = tb[1];
    if (on && ny)
        b2 = tb[tpr];
    if (on && nx && ny)
        b3 = tb[tpr + 1];
    const int ox = cx0 & 7, oy = 8 * (cy0 & 7);
    const uint64_t t0 = oy ? (b0 >> oy) | (b2 << (64 - oy)) : b0;
    const uint64_t t1 = oy ? (b1 >> oy) | (b3 << (64 - oy)) : b1;
    const uint64_t lo = (uint64_t)(0xffu >> ox) * 0x0101010101010101ull;
    return ((t0 >> ox) & lo) | (ox ? (t1 << (8 - ox)) & ~lo : 0ull);
}

// Wave-uniform values read from LDS, into scalar registers.
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}
__device__ __forceinline__ fvv_grid uniform(const fvv_grid& v) {
    fvv_grid g;
    for (int a = 0; a < 3; ++a) {
        g.origin[a] = uniform(v.origin[a]);
        g.lo[a] = uniform(v.lo[a]);
        g.dims[a] = uniform(v.dims[a]);
    }
    g.h = uniform(v.h);
    return g;
}

// A (sub-block, camera) pair's window as the tests read it: the pixels, and
// the window's corner pixel (x | y << 16), or kNoWindow when the camera's
// rectangle is larger than 8 x 8 pixels (its tests then load packed words).
constexpr uint32_t kNoWindow = 0xffffffffu;

struct PairWindow {
    uint64_t bits;
    uint32_t org;
    uint32_t pad_;
};

// One 16 x 4 x 4 block of a fine lattice by one wave (first sample bi0, bj0,
// k0; bi0 is a multiple of 16), without workgroup barriers:
//   1. classification: lane (q, c) = (lane / 16, lane % 16) classifies camera
//      cb + c for the 4 x 4 x 4 sub-block q of the block.  The rectangle
//      [floor(c - r), floor(c + r)] around the rcp quotient c of the
//      sub-block's centre, with the job's radius r for the camera (which
//      bounds how far any point of a 4 x 4 x 4 box moves from its centre's
//      projection, widened by the rounding pad), holds the pixel of every
//      sample of the sub-block.  Clamped to the image: no pixel left -> the
//      camera rejects every sample; otherwise, at most 8 x 8 pixels, the
//      rectangle's pixels as a window from the tiled silhouettes: none set ->
//      reject; all set and the rectangle inside the image -> accept; else
//      mixed, the window kept for the tests.  Larger rectangles are tested
//      from the tiled blocks when they span at most 2 x 2 of them (no
//      window), else count as mixed.
//   2. tests: lane = sample (x, y, z) = (lane % 4, lane / 4 % 4, lane / 16)
//      of each sub-block no camera rejects; each pass tests one mixed camera
//      for each of the four sub-blocks (uniform branches), the pixel's bit
//      read from the pair's window (every in-image sample pixel lies in the
//      clamped rectangle) or, without one, from the packed rows.
//   3. output: the occupancy bytes, and the block's 16 bits of each fine-bitmap
//      row word.
// cam_lds: per camera P and the rounding pad; rho: the job's radii per camera
// (kRhoPer floats); win: this wave's LDS windows [4][FVV_MAX_CAMS].  kSome:
// only n_sel cameras are left to look at, number r in lane r's `sel`, the
// others accept every sample of the block; and the output is zero before, so
// that an empty block writes nothing.  Returns
// the number of test passes, and in the high half the (sub-block, camera)
// tests they made (wave-uniform counts, for measurement builds).
template <bool kSome>
__device__ __forceinline__ uint32_t carve_block16(const CamSet& cams, int n_sel, int sel,
                                                  const float (*cam_lds)[13],
                                              const float* __restrict__ rho,
                                              PairWindow (*win)[FVV_MAX_CAMS],
                                              const uint32_t* __restrict__ sils,
                                              const uint64_t* __restrict__ tiles, int tpr,
                                              int64_t tpc, const fvv_grid& g, int bi0, int bj0,
                                              int k0, uint8_t* __restrict__ out,
                                              const RowBits& fb) {
    const int nx = g.dims[0], ny = g.dims[1], nz = g.dims[2];
    if (bj0 >= ny)
        return 0u;                                 // no row of the block is in the lattice
    uint32_t n_pass = 0u, n_test = 0u;
    const int lane = lane_id();
    const int lx = lane & 3, ly = (lane >> 2) & 3, lz = lane >> 4;
    const int64_t cam_words = (int64_t)cams.H * cams.wpr;
    uint64_t occ[4] = {0ull, 0ull, 0ull, 0ull};
    if (bi0 < nx) {
        // 1. classification
        const int q = lane >> 4, cl = lane & 15;
        const int si0 = bi0 + 4 * q;
        const bool sb_on = si0 < nx;
        float lo[3], hi[3];
        box_corners(g, min(si0, nx - 1), min(si0 + 3, nx - 1), bj0, min(bj0 + 3, ny - 1), k0,
                    min(k0 + 3, nz - 1), lo, hi);
        const float Xc = 0.5f * (lo[0] + hi[0]), Yc = 0.5f * (lo[1] + hi[1]);
        const float Zc = 0.5f * (lo[2] + hi[2]);
        uint32_t rej[4] = {0u, 0u, 0u, 0u}, mix[4] = {0u, 0u, 0u, 0u};
        const int n_look = kSome ? n_sel : cams.n;
        for (int cb = 0; cb < n_look; cb += 16) {
            // c: the camera (kSome: its number among those left)
            const int c = cb + cl;
            const bool on = sb_on && c < n_look;
            const int named = kSome ? __shfl(sel, c & 63) : c;   // (from every lane)
            const int cc = on ? named : 0;
            const float* P = cam_lds[cc];
            const float rx = rho[cc * kRhoPer + 0], ry = rho[cc * kRhoPer + 1];
            const float a = __builtin_fmaf(P[2], Zc, __builtin_fmaf(P[1], Yc, __builtin_fmaf(P[0], Xc, P[3])));
            const float b = __builtin_fmaf(P[6], Zc, __builtin_fmaf(P[5], Yc, __builtin_fmaf(P[4], Xc, P[7])));
            const float w = __builtin_fmaf(P[10], Zc, __builtin_fmaf(P[9], Yc, __builtin_fmaf(P[8], Xc, P[11])));
            const float r = __builtin_amdgcn_rcpf(w);
            const float W = (float)cams.W, H = (float)cams.H;
            const float qa = __builtin_amdgcn_fmed3f(a * r, -8.0f, W + 8.0f);
            const float qb = __builtin_amdgcn_fmed3f(b * r, -8.0f, H + 8.0f);
            const bool bounded = rx < 64.0f && ry < 64.0f;   // (INFINITY: no bound)
            const int x0 = (int)__builtin_floorf(qa - (bounded ? rx : 0.0f));
            const int x1 = (int)__builtin_floorf(qa + (bounded ? rx : 0.0f));
            const int y0 = (int)__builtin_floorf(qb - (bounded ? ry : 0.0f));
            const int y1 = (int)__builtin_floorf(qb + (bounded ? ry : 0.0f));
            const bool inside = x0 >= 0 && y0 >= 0 && x1 < cams.W && y1 < cams.H;
            const int cx0 = max(x0, 0), cx1 = min(x1, cams.W - 1);
            const int cy0 = max(y0, 0), cy1 = min(y1, cams.H - 1);
            const bool off = cx0 > cx1 || cy0 > cy1;
            const bool small = bounded && !off && cx1 - cx0 <= 7 && cy1 - cy0 <= 7;
            const uint64_t* tc = tiles + cc * tpc;
            const uint64_t wv = tiled_window(tc, tpr, small ? cx0 : 0, small ? cy0 : 0,
                                             (cx1 >> 3) != (cx0 >> 3), (cy1 >> 3) != (cy0 >> 3),
                                             on && small);
            const uint64_t cols = (uint64_t)((2u << (cx1 - cx0 & 7)) - 1u) * 0x0101010101010101ull;
            const uint64_t m = cols & (~0ull >> (8 * (7 - (cy1 - cy0 & 7))));
            bool any = (wv & m) != 0ull, all = (wv & m) == m;
            bool known = small;
            if (__ballot(on && bounded && !off && !small) != 0ull) {
                // rectangles past a window: any / all from the tiled blocks
                bool a2 = false, l2 = true;
                const bool ok2 = on && bounded && !off && !small &&
                                 rect_any_all_tiled(tc, tpr, cx0, cx1, cy0, cy1, a2, l2);
                if (ok2) {
                    any = a2;
                    all = l2;
                    known = true;
                }
            }
            int cls = kCullMixed;
            if (bounded && off)
                cls = kCullReject;
            else if (known)
                cls = !any ? kCullReject : ((inside && all) ? kCullAccept : kCullMixed);
            if (on && cls == kCullMixed) {
                PairWindow pw;
                pw.bits = wv;
                pw.org = small ? ((uint32_t)cx0 | ((uint32_t)cy0 << 16)) : kNoWindow;
                pw.pad_ = 0;
                win[q][c] = pw;
            }
            const uint64_t rb = __ballot(on && cls == kCullReject);
            const uint64_t mb = __ballot(on && cls == kCullMixed);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                rej[s] |= (uint32_t)(rb >> (16 * s)) & 0xffffu;
                mix[s] |= ((uint32_t)(mb >> (16 * s)) & 0xffffu) << cb;
            }
            // no sub-block left for the next cameras
            if (cb + 16 < n_look && rej[0] != 0u && (rej[1] != 0u || bi0 + 4 >= nx) &&
                (rej[2] != 0u || bi0 + 8 >= nx) && (rej[3] != 0u || bi0 + 12 >= nx))
                break;
        }
        wave_lds_sync();   // the windows, written above, are read below by every lane
        // 2. tests
        const bool vyz = bj0 + ly < ny && k0 + lz < nz;
        const float Y = lattice_coord(g.lo[1] + bj0 + ly, g.h, g.origin[1]);
        const float Z = lattice_coord(g.lo[2] + k0 + lz, g.h, g.origin[2]);
        float X[4];
        bool alive[4];
        uint32_t rest[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int i = bi0 + 4 * s + lx;
            X[s] = lattice_coord(g.lo[0] + i, g.h, g.origin[0]);
            alive[s] = vyz && i < nx && rej[s] == 0u;
            rest[s] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(rej[s] == 0u ? mix[s] : 0u));
        }
        while ((rest[0] | rest[1] | rest[2] | rest[3]) != 0u) {
            ++n_pass;
            n_test += (rest[0] != 0u) + (rest[1] != 0u) + (rest[2] != 0u) + (rest[3] != 0u);
            int px[4], py[4];
            bool ok[4], act[4];
            uint32_t word[4], org[4];
            uint64_t wbits[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                act[s] = rest[s] != 0u;
                if (act[s]) {
                    const int c = __ffs(rest[s]) - 1;
                    rest[s] &= rest[s] - 1u;
                    const PairWindow pw = win[s][c];
                    const int cam = kSome ? __builtin_amdgcn_readlane(sel, c) : c;
                    org[s] = (uint32_t)__builtin_amdgcn_readfirstlane((int)pw.org);
                    wbits[s] = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(pw.bits >> 32)) << 32) |
                               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)pw.bits);
                    ok[s] = point_pixel_exact(cams.Pc(cam), X[s], Y, Z, cams.W, cams.H, px[s],
                                              py[s]);
                    word[s] = 0u;
                    if (org[s] == kNoWindow && ok[s])
                        word[s] = sils[cam * cam_words + py[s] * cams.wpr + (px[s] >> 5)];
                }
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (act[s]) {
                    bool in;
                    if (org[s] != kNoWindow) {
                        const int ox = (int)(org[s] & 0xffffu), oy = (int)(org[s] >> 16);
                        in = ok[s] && ((wbits[s] >> ((8 * (py[s] - oy) + (px[s] - ox)) & 63)) & 1ull);
                    } else {
                        in = ok[s] && ((word[s] >> (px[s] & 31)) & 1u);
                    }
                    alive[s] = alive[s] && in;
                    if (__ballot(alive[s]) == 0ull)
                        rest[s] = 0u;
                }
            }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
            occ[s] = __ballot(alive[s]);
        wave_lds_sync();   // the next block rewrites the windows
    }
    if (kSome && (occ[0] | occ[1] | occ[2] | occ[3]) == 0ull)
        return n_pass | (n_test << 16);
    // 3. output: bytes, lane -> (x, y) = (lane % 16, lane / 16), every z
    const uint64_t plane = (uint64_t)nx * (uint64_t)ny;
    {
        const int x = lane & 15, y = lane >> 4;
        const int i = bi0 + x, j = bj0 + y;
        const int s = x >> 2;
        const uint64_t oq = s == 0 ? occ[0] : s == 1 ? occ[1] : s == 2 ? occ[2] : occ[3];
        if (i < nx && j < ny) {
            uint8_t* o = out + ((uint64_t)k0 * plane + (uint64_t)j * (uint64_t)nx + i);
#pragma unroll
            for (int z = 0; z < 4; ++z)
                if (k0 + z < nz)
                    o[z * plane] = (uint8_t)((oq >> ((x & 3) + 4 * y + 16 * z)) & 1ull);
        }
    }
    // fine bitmap: lane r < 16 -> row (y, z) = (r % 4, r / 4); the block's 16
    // samples along x are bits (bi0 & 63) .. + 15 of the row's word
    if (lane < 16) {
        const int y = lane & 3, z = lane >> 2;
        const int j = bj0 + y, k = k0 + z;
        if (j < ny && k < nz) {
            uint32_t b = 0;
#pragma unroll
            for (int s = 0; s < 4; ++s)
                b |= (uint32_t)((occ[s] >> (4 * y + 16 * z)) & 0xfull) << (4 * s);
            const int64_t row = (int64_t)j + (int64_t)ny * k;
            reinterpret_cast<uint16_t*>(fb.words + row * fb.wr + (bi0 >> 6))[(bi0 & 63) >> 4] =
                (uint16_t)b;
        }
    }
    return n_pass | (n_test << 16);
}

// A brick: kFineBrickX x kFineBrickYZ x kFineBrickYZ samples, four blocks.
constexpr int kFineBrickX = 16, kFineBrickYZ = 8;

// Classification of every camera for two bricks side by side along x (the first
// one's first sample i0, j0, k0) by one wave, lane = (brick l / 32, camera l %
// 32; four bricks of 16 lanes for rigs of up to 16 cameras, compiled in beside
// it, spilled registers): the rectangle around
// the rcp quotient of the brick's centre, its half-widths the sums of the job's
// edge radii (each of half a spacing, so 15, 7 and 7 of them span the brick's
// half-extents), as in carve_block16; read from up to 4 x 4 tiled blocks
// (larger: mixed).  Returns the ballot of the cameras that reject every sample
// of their brick, and in mixed that of those that neither reject nor accept all
// of them (bricks past the lattice have neither).
__device__ __forceinline__ uint64_t classify_bricks(const CamSet& cams, const float (*cam_lds)[13],
                                                    const float* __restrict__ rho,
                                                    const uint64_t* __restrict__ tiles, int tpr,
                                                    int64_t tpc, const fvv_grid& g, int i0, int j0,
                                                    int k0, uint64_t& mixed) {
    const int lane = lane_id(), ib = i0 + (lane >> 5) * kFineBrickX;
    const bool on = (lane & 31) < cams.n && ib < g.dims[0];
    const int c = on ? lane & 31 : 0;
    float lo[3], hi[3];
    box_corners(g, min(ib, g.dims[0] - 1), min(ib + kFineBrickX, g.dims[0]) - 1, j0,
                min(j0 + kFineBrickYZ, g.dims[1]) - 1, k0, min(k0 + kFineBrickYZ, g.dims[2]) - 1, lo, hi);
    const float Xc = 0.5f * (lo[0] + hi[0]), Yc = 0.5f * (lo[1] + hi[1]);
    const float Zc = 0.5f * (lo[2] + hi[2]);
    const float* P = cam_lds[c];
    const float* r = rho + c * kRhoPer;
    constexpr float ex = kFineBrickX - 1, eyz = kFineBrickYZ - 1;
    const float rx = ex * r[2] + eyz * (r[4] + r[6]), ry = ex * r[3] + eyz * (r[5] + r[7]);
    const float a = __builtin_fmaf(P[2], Zc, __builtin_fmaf(P[1], Yc, __builtin_fmaf(P[0], Xc, P[3])));
    const float b = __builtin_fmaf(P[6], Zc, __builtin_fmaf(P[5], Yc, __builtin_fmaf(P[4], Xc, P[7])));
    const float w = __builtin_fmaf(P[10], Zc, __builtin_fmaf(P[9], Yc, __builtin_fmaf(P[8], Xc, P[11])));
    const float q = __builtin_amdgcn_rcpf(w);
    const float W = (float)cams.W, H = (float)cams.H;
    const bool bounded = rx < 32.0f && ry < 32.0f;   // (wider: more than 4 blocks)
    const float sx = bounded ? rx : 0.0f, sy = bounded ? ry : 0.0f;
    const float qa = __builtin_amdgcn_fmed3f(a * q, -64.0f, W + 64.0f);
    const float qb = __builtin_amdgcn_fmed3f(b * q, -64.0f, H + 64.0f);
    const int x0 = (int)__builtin_floorf(qa - sx), x1 = (int)__builtin_floorf(qa + sx);
    const int y0 = (int)__builtin_floorf(qb - sy), y1 = (int)__builtin_floorf(qb + sy);
    const bool inside = x0 >= 0 && y0 >= 0 && x1 < cams.W && y1 < cams.H;
    const int cx0 = max(x0, 0), cx1 = min(x1, cams.W - 1);
    const int cy0 = max(y0, 0), cy1 = min(y1, cams.H - 1);
    const bool off = cx0 > cx1 || cy0 > cy1;
    const int bx0 = cx0 >> 3, by0 = cy0 >> 3, nbx = (cx1 >> 3) - bx0, nby = (cy1 >> 3) - by0;
    const bool known = on && bounded && !off && nbx < 4 && nby < 4;
    bool any = false, all = true;
    if (known) {
        const uint64_t* t = tiles + c * tpc + (int64_t)by0 * tpr + bx0;
        uint64_t cols[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int x = 8 * (bx0 + d), c0 = max(cx0 - x, 0), c1 = max(min(cx1 - x, 7), 0);
            cols[d] = d <= nbx ? (uint64_t)((2u << c1) - (1u << c0)) * 0x0101010101010101ull : 0ull;
        }
        // (a block row at a time: all sixteen blocks at once spill registers)
#pragma unroll 1
        for (int e = 0; e <= nby; ++e) {
            const int y = 8 * (by0 + e), r0 = max(cy0 - y, 0), r1 = min(cy1 - y, 7);
            const uint64_t rows = (~0ull >> (8 * (7 - r1))) & (~0ull << (8 * r0));
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint64_t m = cols[d] & rows;
                const uint64_t v = t[(int64_t)e * tpr + min(d, nbx)];
                any |= (v & m) != 0ull;
                all &= (v & m) == m;
            }
        }
    }
    const bool rej = on && bounded && (off || (known && !any));
    mixed = __ballot(on && !rej && !(known && inside && all));
    return __ballot(rej);
}

// A brick whose samples are all occupied: its occupancy bytes and its 16 bits of
// each fine-bitmap row word (the bits past nx clear), lane = row (y, z) = (l % 8,
// l / 8).
__device__ __forceinline__ void fill_brick(const fvv_grid& g, int i0, int j0, int k0,
                                           uint8_t* __restrict__ out, const RowBits& fb) {
    const int lane = lane_id(), j = j0 + (lane & 7), k = k0 + (lane >> 3);
    if (j >= g.dims[1] || k >= g.dims[2])
        return;
    const int64_t row = (int64_t)j + (int64_t)g.dims[1] * k;
    const int n = min(g.dims[0] - i0, 16);
    uint8_t* o = out + row * g.dims[0] + i0;
    const uint32_t v[4] = {0x01010101u, 0x01010101u, 0x01010101u, 0x01010101u};
    if (n == 16)
        __builtin_memcpy(o, v, 16);
    else
        for (int x = 0; x < n; ++x)
            o[x] = 1;
    reinterpret_cast<uint16_t*>(fb.words + row * fb.wr + (i0 >> 6))[(i0 & 63) >> 4] =
        (uint16_t)((1u << n) - 1u);
}

// Zero n bytes from p by one wave: 16-byte stores between the first and the
// last 16-byte boundary, byte stores at the ends.
__device__ __forceinline__ void wave_zero_span(uint8_t* p, int64_t n) {
    const int lane = lane_id();
    const int64_t head = (int64_t)((16 - ((uintptr_t)p & 15)) & 15);
    const int64_t h = head < n ? head : n;
    const int64_t n16 = (n - h) / 16, tail0 = h + 16 * n16;
    uint4* q = reinterpret_cast<uint4*>(p + h);
    for (int64_t i = lane; i < n16; i += kWave)
        q[i] = make_uint4(0u, 0u, 0u, 0u);
    if (lane < h)
        p[lane] = 0;
    if (lane < n - tail0)
        p[tail0 + lane] = 0;
}

// Measurement builds (FVV_CARVE_PROBE defined) record, for the first
// kProbeWaves waves of the frame's fine carve, the real-time clock (100 MHz)
// at the wave's entry and exit, its block count and the time its workgroup's
// tables took (entry to the barrier after them), and for its first
// kProbeIters blocks their start, end, test passes and tests.
#ifdef FVV_CARVE_PROBE
constexpr int kProbeWaves = 16384, kProbeIters = 4;
__device__ uint64_t carve_probe_blocks[kProbeWaves * kProbeIters][3];
__device__ uint64_t carve_probe_waves[kProbeWaves][3];
#endif

// The fine carve of a frame: the tiles of all carried ROIs dealt out to the
// workgroups in turn (tile t to workgroup t mod grid, then t + grid, ...), so
// every XCD gets an even share of the costly tiles near the surfaces (this
// measured faster than contiguous tile ranges per XCD, which keep each L2's
// share of the silhouettes smaller but leave some XCDs with more work).  A
// workgroup takes whole tiles (TX x TY x 4 samples);
// each of its four waves owns one 16 x 4 x 4 block of the tile (x offset
// 16 (w mod TX/16), y offset 4 (w div TX/16)) and carves it on its own, with
// no workgroup barrier (carve_block16).  Job tables of up to kJobLds ROIs and
// the cameras' matrices and rounding pads are kept in LDS.
//
// A large frame (at least kGroupTiles tiles of 1024 samples, its jobs in LDS)
// goes by groups of bricks side by side along x instead: most of its blocks lie
// well outside or inside, and 16-byte pieces of rows are what its time goes to.
// A workgroup zeroes a group's output while it classifies the cameras for the
// bricks; the bricks that no camera rejects go into a list in LDS, from which
// the waves take one block after the other (carve_block16 for the brick's mixed
// cameras) or a whole brick to fill.  From kWideGroupTiles on a group spans up
// to 64 bricks (whole rows: each layer's zeros are one span); below, 8, so that
// there are several groups per workgroup.  4.3e8 samples in 24 cameras: 1500 us
// by tiles, 850 by bricks each written on its own (680 of them for the writes
// alone), 380 by groups; whole frames of 8, 13, 24, 28 and 30e6 samples (16 to
// 24 cameras) 176, 285, 298, 330 and 297 us against 176, 298, 330, 353 and 367.
// Smaller ones lose by it (5e6 samples of 56 ROIs: 267 against 255, a frame of
// 4e6: the carve 49 against 42).  A large frame of more than kJobLds ROIs goes by
// tiles: 8.4e7 samples of 82 ROIs in 16 cameras take the carve 403 us, where 5.9e7
// of 57 take 200 (1.4 times as long per sample).
constexpr int kJobLds = 64;
constexpr int kGroupBricks = 64;
constexpr uint64_t kGroupTiles = 12288, kWideGroupTiles = 65536;

// A group: `bricks` bricks side by side along x.  What is left of it: the bricks
// that no camera rejects, by place along x and mixed cameras (none: all full),
// their count and the next block to take, of this group and of the next (par:
// whose turn); and the group itself, read back per block so that the block loop
// keeps little of it in registers (kept in scalar registers, it spilled a
// hundred of them).
struct GroupList {
    uint16_t brick[kGroupBricks];
    uint32_t mixed[kGroupBricks];
    uint32_t left[2], next[2];
    uint64_t t;
    int32_t jb, i0, j0, k0, par;
};

__device__ __forceinline__ uint64_t fine_groups(const fvv_grid& g, int bricks) {
    const int x = bricks * kFineBrickX;
    return (uint64_t)((g.dims[0] + x - 1) / x) *
           (uint64_t)((g.dims[1] + kFineBrickYZ - 1) / kFineBrickYZ) *
           (uint64_t)((g.dims[2] + kFineBrickYZ - 1) / kFineBrickYZ);
}

template <int TX>
__global__ __launch_bounds__(kBlock, 7) void carve_frame_kernel(const fvv_job* __restrict__ jobs,
                                                             const JobPrefix* __restrict__ pre,
                                                             const uint32_t* __restrict__ counter,
                                                             const CamSet cams,
                                                             const uint32_t* __restrict__ sils,
                                                             const uint64_t* __restrict__ tiles,
                                                             const float* __restrict__ rho,
                                                             uint8_t* __restrict__ out,
                                                             uint64_t* __restrict__ finebits,
                                                             int job_lds, LabelWrite lw) {
    // the workgroups past the carve's write the coarse labels and filtered
    // occupancy and clear the labelling's row bitmap (they start as the
    // carve's tail frees the CUs)
    if (blockIdx.x >= lw.carve_blocks) {
        const int64_t stride = (int64_t)(gridDim.x - lw.carve_blocks) * kBlock;
        const int64_t t0 = (int64_t)(blockIdx.x - lw.carve_blocks) * kBlock + threadIdx.x;
        label_write_samples(lw, t0, stride);
        label_write_clear(lw, t0, stride);
        return;
    }
#ifdef FVV_CARVE_PROBE
    const uint64_t probe_entry = __builtin_amdgcn_s_memrealtime();
    uint32_t probe_blocks = 0;
#endif
    constexpr int BXN = TX / 16;                     // blocks of a tile along x
    __shared__ PairWindow s_win[kBlock / kWave][4][FVV_MAX_CAMS];
    __shared__ uint64_t s_tile_off[kJobLds + 1];
    __shared__ uint64_t s_bit_off[kJobLds];
    __shared__ int64_t s_out[kJobLds];
    __shared__ fvv_grid s_grid[kJobLds];
    __shared__ float s_cam[FVV_MAX_CAMS][13];        // P, then the rounding pad
    __shared__ GroupList s_list;
    // the job tables of the first job_lds jobs (every job the output can hold,
    // up to kJobLds), loaded without waiting for the frame's job count
    for (int j = threadIdx.x; j <= job_lds; j += kBlock) {
        s_tile_off[j] = pre[j].tile_off;
        if (j < job_lds) {
            s_bit_off[j] = pre[j].bit_off;
            s_out[j] = jobs[j].out_offset;
            s_grid[j] = jobs[j].grid;
        }
    }
    const int nj = (int)counter[2];
    const bool lds = nj <= job_lds;
    for (int i = threadIdx.x; i < cams.n * 13; i += kBlock) {
        const int c = i / 13, e = i - 13 * c;
        s_cam[c][e] = e < 12 ? cams.P[c][e] : cams.pad[c];
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int xo = 16 * (wave % BXN), yo = 4 * (wave / BXN);
    const int tpr = (cams.W + 7) / 8;
    const int64_t tpc = (int64_t)tpr * ((cams.H + 7) / 8);
#ifdef FVV_CARVE_PROBE
    const uint64_t probe_tables = __builtin_amdgcn_s_memrealtime();
    // a block from t_a to now, and its counts, into the wave's records
    auto probe_block = [&](uint64_t t_a, uint32_t passes_tests) {
        const uint64_t t_b = __builtin_amdgcn_s_memrealtime();
        const uint32_t pw = blockIdx.x * (kBlock / kWave) + wave;
        if (lane_id() == 0 && pw < (uint32_t)kProbeWaves && probe_blocks < (uint32_t)kProbeIters) {
            uint64_t* r = carve_probe_blocks[pw * kProbeIters + probe_blocks];
            r[0] = t_a;
            r[1] = t_b;
            r[2] = passes_tests;
        }
        ++probe_blocks;
    };
#endif
    // the tiles' loop, once with the job tables in LDS and once without (two
    // copies, so that neither reads its tables through generic pointers)
    auto tiles_loop = [&](auto in_lds) {
    uint64_t total;
    if constexpr (decltype(in_lds)::value)
        total = s_tile_off[nj];
    else
        total = pre[nj].tile_off;
    const XcdSlice xs{0, total, blockIdx.x, lw.carve_blocks};
    for (uint64_t t = xs.begin + xs.slot; t < xs.end; t += xs.stride) {
        int jb;
        fvv_grid g;
        int64_t out_off;
        uint64_t tile0, bit_off;
        if constexpr (decltype(in_lds)::value) {
            jb = upper_job([&](int m) { return s_tile_off[m]; }, nj, t);
            g = s_grid[jb];
            out_off = s_out[jb];
            tile0 = s_tile_off[jb];
            bit_off = s_bit_off[jb];
        } else {
            jb = upper_job([&](int m) { return pre[m].tile_off; }, nj, t);
            g = jobs[jb].grid;
            out_off = jobs[jb].out_offset;
            tile0 = pre[jb].tile_off;
            bit_off = pre[jb].bit_off;
        }
        RowBits fb{};
        fb.words = finebits + bit_off;
        fb.wr = (g.dims[0] + 63) / 64;
        int i0, j0, k0;
        tile_origin<TX>(g, t - tile0, i0, j0, k0);
#ifdef FVV_CARVE_PROBE
        const uint64_t t_a = __builtin_amdgcn_s_memrealtime();
#endif
        const uint32_t passes_tests =
            carve_block16<false>(cams, 0, 0, s_cam, rho + (int64_t)jb * FVV_MAX_CAMS * kRhoPer,
                                 s_win[wave],
                          sils, tiles, tpr, tpc, g, i0 + xo, j0 + yo, k0, out + out_off, fb);
#ifdef FVV_CARVE_PROBE
        probe_block(t_a, passes_tests);
#else
        (void)passes_tests;
#endif
    }
    };
    if (lds && s_tile_off[nj] >= kGroupTiles) {
        // the groups' prefix over the jobs, in the tiles' place
        const int bricks = s_tile_off[nj] >= kWideGroupTiles ? kGroupBricks : 8;
        __syncthreads();
        if (threadIdx.x < kWave) {
            const uint64_t n = (int)threadIdx.x < nj ? fine_groups(s_grid[threadIdx.x], bricks) : 0ull;
            const uint64_t inc = wave_inclusive_sum64(n);
            if ((int)threadIdx.x < nj)
                s_tile_off[threadIdx.x + 1] = inc;
            if (threadIdx.x == 0) {
                s_tile_off[0] = 0ull;
                s_list.left[0] = s_list.next[0] = 0u;
            }
        }
        __syncthreads();
        GroupList& list = s_list;
        const int lane = lane_id();
        uint64_t t = blockIdx.x;
        int par = 0;
        while (t < uniform(s_tile_off[nj])) {
            // 1. the group's output zeroed, and the cameras classified for its
            // bricks, two per wave at once
            {
                const int jb = uniform(upper_job([&](int m) { return s_tile_off[m]; }, nj, t));
                const fvv_grid g = uniform(s_grid[jb]);
                const uint64_t q = t - uniform(s_tile_off[jb]);
                const uint32_t ngx = (uint32_t)((g.dims[0] + bricks * kFineBrickX - 1) /
                                                (bricks * kFineBrickX));
                const uint32_t ngy = (uint32_t)((g.dims[1] + kFineBrickYZ - 1) / kFineBrickYZ);
                const uint64_t qy = q / ngx;
                const int i0 = (int)(q - qy * ngx) * bricks * kFineBrickX;
                const int j0 = (int)(qy % ngy) * kFineBrickYZ, k0 = (int)(qy / ngy) * kFineBrickYZ;
                {
                    const int nr = min(kFineBrickYZ, g.dims[1] - j0);
                    const int rows = nr * min(kFineBrickYZ, g.dims[2] - k0);
                    const int n = min(g.dims[0] - i0, bricks * kFineBrickX);
                    const int wr = (g.dims[0] + 63) / 64, np = (n + 15) / 16, nw = (n + 63) / 64;
                    uint8_t* const o = out + uniform((uint64_t)s_out[jb]) + i0;
                    uint64_t* const words = finebits + uniform(s_bit_off[jb]) + (i0 >> 6);
                    const uint32_t z[4] = {0u, 0u, 0u, 0u};
                    if (n == g.dims[0]) {      // whole rows: one span per layer
                        for (int l = wave; l * nr < rows; l += kBlock / kWave)
                            wave_zero_span(o + ((int64_t)j0 + (int64_t)g.dims[1] * (k0 + l)) * n,
                                           (int64_t)nr * n);
                    } else for (int e = threadIdx.x; e < rows * np; e += kBlock) {
                        const int rw = e / np, x = 16 * (e - rw * np);
                        const int64_t row = (int64_t)(j0 + rw % nr) + (int64_t)g.dims[1] * (k0 + rw / nr);
                        uint8_t* const p = o + row * g.dims[0] + x;
                        if (x + 16 <= n)
                            __builtin_memcpy(p, z, 16);
                        else
                            for (int b = 0; b < n - x; ++b)
                                p[b] = 0;
                    }
                    for (int e = threadIdx.x; e < rows * nw; e += kBlock) {
                        const int rw = e / nw;
                        const int64_t row = (int64_t)(j0 + rw % nr) + (int64_t)g.dims[1] * (k0 + rw / nr);
                        words[row * wr + (e - rw * nw)] = 0ull;
                    }
                }
                const int nb = min((g.dims[0] - i0 + kFineBrickX - 1) / kFineBrickX, bricks);
                for (int b0 = 2 * wave; b0 < nb; b0 += 2 * (kBlock / kWave)) {
                    uint64_t mixed;
                    const uint64_t rej =
                        classify_bricks(cams, s_cam, rho + (int64_t)jb * FVV_MAX_CAMS * kRhoPer,
                                        tiles, tpr, tpc, g, i0 + b0 * kFineBrickX, j0, k0, mixed);
                    const int b = lane >> 5;
                    if ((lane & 31) == 0 && b0 + b < nb && (uint32_t)(rej >> (32 * b)) == 0u) {
                        const uint32_t at = atomicAdd(&list.left[par], 1u);
                        list.brick[at] = (uint16_t)(b0 + b);
                        list.mixed[at] = (uint32_t)(mixed >> (32 * b));
                    }
                }
                if (threadIdx.x == 0) {
                    list.t = t;
                    list.jb = jb;
                    list.i0 = i0;
                    list.j0 = j0;
                    list.k0 = k0;
                    list.par = par;
                    list.left[par ^ 1] = list.next[par ^ 1] = 0u;
                }
            }
            __syncthreads();           // the list is complete, the zeros are written
            // 2. the blocks of the bricks that no camera rejects, one after the
            // other by whichever wave is free
            for (;;) {
                const int p = uniform(list.par);
                uint32_t item = 0u;
                if (lane == 0)
                    item = atomicAdd(&list.next[p], 1u);
                item = (uint32_t)uniform((int)item);
                if (item >= 4u * (uint32_t)uniform((int)list.left[p]))
                    break;
                const int jb = uniform(list.jb);
                const fvv_grid g = uniform(s_grid[jb]);
                const int i0 = uniform(list.i0) + kFineBrickX * uniform((int)list.brick[item >> 2]);
                const uint32_t mix = (uint32_t)uniform((int)list.mixed[item >> 2]);
                const int j0 = uniform(list.j0), k0 = uniform(list.k0), b = (int)(item & 3u);
                const int jy = j0 + 4 * (b & 1), kz = k0 + 4 * (b >> 1);
                RowBits fb{};
                fb.words = finebits + uniform(s_bit_off[jb]);
                fb.wr = (g.dims[0] + 63) / 64;
                uint8_t* const o = out + uniform((uint64_t)s_out[jb]);
                if (mix == 0u) {
                    if (b == 0)
                        fill_brick(g, i0, j0, k0, o, fb);
                    continue;
                }
                if (jy >= g.dims[1] || kz >= g.dims[2])
                    continue;
                // lane r: the r-th mixed camera
                const int rank = __popc(mix & (uint32_t)lanes_below_mask());
                const int sel = __builtin_amdgcn_ds_permute(
                    4 * (lane < 32 && ((mix >> (lane & 31)) & 1u) ? rank : 63), lane);
#ifdef FVV_CARVE_PROBE
                const uint64_t t_a = __builtin_amdgcn_s_memrealtime();
#endif
                const uint32_t passes_tests = carve_block16<true>(
                    cams, __popc(mix), sel, s_cam, rho + (int64_t)jb * FVV_MAX_CAMS * kRhoPer,
                    s_win[wave], sils, tiles, tpr, tpc, g, i0, jy, kz, o, fb);
#ifdef FVV_CARVE_PROBE
                probe_block(t_a, passes_tests);
#else
                (void)passes_tests;
#endif
            }
            t = uniform(list.t) + lw.carve_blocks;
            par = uniform(list.par) ^ 1;
            __syncthreads();           // the list is free
        }
    } else if (lds) {
        tiles_loop(std::true_type{});
    } else {
        tiles_loop(std::false_type{});
    }
#ifdef FVV_CARVE_PROBE
    const uint32_t pw = blockIdx.x * (kBlock / kWave) + wave;
    if (lane_id() == 0 && pw < (uint32_t)kProbeWaves) {
        carve_probe_waves[pw][0] = probe_entry;
        carve_probe_waves[pw][1] = __builtin_amdgcn_s_memrealtime();
        // blocks carved, and (high half) the ticks from entry to the tables'
        // barrier
        carve_probe_waves[pw][2] = probe_blocks | ((probe_tables - probe_entry) << 32);
    }
#endif
}

// ------------------------------------------------------------------ batched carve, culled
// Most of a large batch is empty (98.6 % on 64 frames x 12 ROIs of two
// ellipsoids), so what it cannot do without is writing zeros.  Three passes:
//   1. batched_zero_kernel zeroes every job's output, each workgroup a
//      contiguous part of a job; its first workgroups write the prefixes and
//      the rounding pads.
//   2. batched_mark_kernel classifies the cameras for units (kUnitY sample
//      rows x 4 layers, all along x), a wave per kUnitGroup of them, the group
//      as a whole first, and then for the tiles (16 samples along x) of a unit
//      that no camera rejects, 16 at a time.  Such a unit's tiles get a mark
//      in their first byte: kLiveMark, or kDeadMark where a camera rejects the
//      tile.  A small batch it carves itself (carve_strips).
//   3. carve_batched_culled_kernel carves the live tiles of the marked units,
//      a wave each.
// The units and tiles go to the XCDs in a static partition; each job's cameras
// come from the device table.  64 frames x 12 ROIs (2.9e9 samples, 4 cameras)
// take 530 + 103 + 201 us (a plain fill of as many bytes 415); one pass that
// classified and wrote a row of tiles per workgroup and step took 1258 us.  A
// first pass that zeroed the rejected units itself took 636 us whatever it
// classified: its 2.5 KB spans at odd addresses reach 4.2 TB/s.
constexpr int kBatchedJobLds = 1024;
constexpr int kGroup = kBlock / kWave;
constexpr int kRowRectWords = 8;   // silhouette words per row of a unit's rectangle
constexpr uint8_t kLiveMark = 0xff, kDeadMark = 0xfe;   // no occupancy values

// The units of a culled batched carve: kUnitY sample rows of 4 layers, all
// along x, y fastest, the rows padded to groups of kUnitGroup units.
constexpr int kUnitY = 16, kUnitGroup = 4;

__device__ __forceinline__ uint64_t units_of_grid(const fvv_grid& g) {
    constexpr uint32_t kRows = kUnitY * kUnitGroup;   // (unsigned: a side may be near 2^31)
    return kUnitGroup * (uint64_t)(((uint32_t)g.dims[1] + kRows - 1u) / kRows) *
           (uint64_t)((g.dims[2] + 3) / 4);
}

// The jobs' prefixes of units, or with kStrips of strips, in LDS (kLds) or from
// the table.
template <bool kLds, bool kStrips>
struct JobOffsets {
    const uint64_t* lds;
    const JobPrefix* pre;
    __device__ uint64_t operator()(int m) const {
        return kLds ? lds[m] : kStrips ? pre[m].bit_off : pre[m].tile_off;
    }
};

template <bool kLds, bool kStrips = false>
__device__ __forceinline__ JobOffsets<kLds, kStrips> load_offsets(
    const JobPrefix* __restrict__ pre, int nj, uint64_t* lds) {
    if (kLds) {
        for (int j = threadIdx.x; j <= nj; j += kBlock)
            lds[j] = kStrips ? pre[j].bit_off : pre[j].tile_off;
        __syncthreads();
    }
    return JobOffsets<kLds, kStrips>{lds, pre};
}

// A small batch (kStripTiles tiles of 64 x 4 x 4 samples, 48 per CU; those of a few
// cameras count twice) is carved by strips instead, kStripY sample rows of 4
// layers, all along x, y fastest, in the marking's place (the third pass finds no
// units): with so few units the marks cost a launch's latency and leave most of
// the chip idle, the more so the more cameras a unit waits for.  32 tight ROIs of
// 2e6 samples in all (3385 tiles) in 4, 16 and 32 cameras: 32, 50 and 113 us, by
// marks 38, 91 and 191; 6 ROIs of 6.6e5: 21.4 and 26.6; nearly empty ones of 6e6
// (10190 tiles) in 12 and 32 cameras: 60 and 81, by marks 85 and 126.  Above, 32
// tight ROIs of 5.6e6 in 4 cameras (8079 tiles, counted twice): 47 and 42 by
// marks; 128 nearly empty ones of 1e7 in 8 cameras (15397): 64 and 59.
constexpr int kStripY = 4;
constexpr uint64_t kStripTiles = 12288;
constexpr int kFewCams = 6;

__device__ __forceinline__ uint64_t strips_of_grid(const fvv_grid& g) {
    return (uint64_t)(((uint32_t)g.dims[1] + kStripY - 1u) / kStripY) *
           (uint64_t)((g.dims[2] + 3) / 4);
}

// Unit u of a job: whether it has rows in the lattice (padding units do not), its
// first row and layer, and the place of its first byte.
struct BatchedUnit {
    bool on;
    int j0, k0;
    int64_t at;
};

__device__ __forceinline__ BatchedUnit batched_unit(const fvv_job& job, uint32_t u) {
    constexpr uint32_t kRows = kUnitY * kUnitGroup;
    const uint32_t nuy = kUnitGroup * (((uint32_t)job.grid.dims[1] + kRows - 1u) / kRows);
    BatchedUnit b;
    const uint32_t j0 = u % nuy * kUnitY;
    b.on = j0 < (uint32_t)job.grid.dims[1];
    b.j0 = b.on ? (int)j0 : 0;
    b.k0 = (int)(u / nuy) * 4;
    b.at = job.out_offset +
           ((int64_t)b.k0 * job.grid.dims[1] + b.j0) * (int64_t)job.grid.dims[0];
    return b;
}

__device__ __forceinline__ JobCams job_cams(const fvv_job& job, int j,
                                            const fvv_camera* __restrict__ cams,
                                            const float* __restrict__ job_pad) {
    return JobCams{cams + job.cam_base, job_pad + (int64_t)j * FVV_MAX_CAMS, job.n_cams,
                   job.width, job.height, (job.width + 31) / 32};
}

// A job's cameras staged in LDS: P, then the rounding pad.
struct LdsCams {
    const float (*cam)[13];
    int32_t n, W, H, wpr;
    __device__ const float* Pc(int c) const { return cam[c]; }
    __device__ float padc(int c) const { return cam[c][12]; }
};

// The zeroing pass's steps: a job's output in pieces of kZeroStep bytes, cut at
// the address's multiples of it (lines are written whole but at a job's ends).
constexpr uint64_t kZeroStep = kBlock * 16;

struct JobBytes {
    uintptr_t p0, p1;
    __device__ uint64_t steps() const { return (p1 - 1) / kZeroStep - p0 / kZeroStep + 1; }
};

__device__ __forceinline__ JobBytes job_bytes(const fvv_job& j, const uint8_t* out) {
    const uintptr_t p0 = (uintptr_t)(out + j.out_offset);
    return JobBytes{p0, p0 + (uintptr_t)((uint64_t)j.grid.dims[0] * (uint64_t)j.grid.dims[1] *
                                         (uint64_t)j.grid.dims[2])};
}

// A table's prefixes go kPrefixJobs jobs per thread (their loads in flight
// together): a workgroup takes 1024 jobs at once.
constexpr int kPrefixJobs = 4;
static_assert(kBlock * kPrefixJobs == kBatchedJobLds, "an LDS table in one step");

// Workgroup 0: the prefixes of units (tile_off; no units in all where the batch
// goes by strips) and of strips (bit_off); a job out of range has none and raises
// the job flag.  The next: the rounding pad of every (job, camera) pair over the
// job's lattice box, job_pad[j * FVV_MAX_CAMS + c].
__device__ __forceinline__ void batched_table(uint32_t block, const fvv_job* __restrict__ jobs,
                                              uint32_t n_jobs, const fvv_camera* __restrict__ cams,
                                              float* __restrict__ job_pad,
                                              JobPrefix* __restrict__ pre,
                                              uint32_t* __restrict__ counter,
                                              uint32_t* __restrict__ status) {
    if (block == 0) {
        __shared__ uint64_t scratch[kBlock / kWave];
        uint64_t units = 0, strips = 0, tiles = 0;
        for (uint32_t base = 0; base < n_jobs; base += kBatchedJobLds) {
            const uint32_t j0 = base + kPrefixJobs * threadIdx.x;
            uint64_t u[kPrefixJobs], r[kPrefixJobs], us = 0, rs = 0;
#pragma unroll
            for (int e = 0; e < kPrefixJobs; ++e) {
                u[e] = r[e] = 0;
                if (j0 + e < n_jobs) {
                    const fvv_job& j = jobs[j0 + e];
                    if (job_ok(j)) {
                        u[e] = units_of_grid(j.grid);
                        r[e] = strips_of_grid(j.grid);
                        tiles += r[e] * (((uint32_t)j.grid.dims[0] + 63u) / 64u) *
                                 (j.n_cams <= kFewCams ? 2u : 1u);
                    } else {
                        atomicOr(status, kFlagJob);
                    }
                }
                us += u[e];
                rs += r[e];
            }
            uint64_t ut, rt;
            uint64_t ua = units + block_exclusive_sum64<kBlock>(us, scratch, &ut);
            uint64_t ra = strips + block_exclusive_sum64<kBlock>(rs, scratch, &rt);
#pragma unroll
            for (int e = 0; e < kPrefixJobs; ++e)
                if (j0 + e < n_jobs) {
                    pre[j0 + e].tile_off = ua;
                    pre[j0 + e].bit_off = ra;
                    ua += u[e];
                    ra += r[e];
                }
            units += ut;
            strips += rt;
        }
        uint64_t all;
        block_exclusive_sum64<kBlock>(tiles, scratch, &all);
        if (threadIdx.x == 0) {
            pre[n_jobs].tile_off = all <= kStripTiles ? 0ull : units;
            pre[n_jobs].bit_off = strips;
            counter[2] = n_jobs;
        }
        return;
    }
    const uint64_t p = (uint64_t)(block - 1) * kBlock + threadIdx.x;
    if (p >= (uint64_t)n_jobs * FVV_MAX_CAMS)
        return;
    const fvv_job& j = jobs[p / FVV_MAX_CAMS];
    const int c = (int)(p % FVV_MAX_CAMS);
    if (!job_ok(j) || c >= j.n_cams)
        return;
    double lo[3], hi[3];
    grid_box(j.grid, lo, hi);
    job_pad[p] = rounding_pad(cams[j.cam_base + c].P, j.width, j.height, lo, hi);
}

// Zero steps [q, end) of a job's output by the workgroup.
__device__ __forceinline__ void zero_steps(const JobBytes& b, uint64_t q, uint64_t end) {
    uintptr_t at = (b.p0 & ~(uintptr_t)(kZeroStep - 1)) + q * kZeroStep + 16 * threadIdx.x;
    for (; q < end; ++q, at += kZeroStep) {
        if (at >= b.p0 && at + 16 <= b.p1) {
            *reinterpret_cast<uint4*>(at) = make_uint4(0u, 0u, 0u, 0u);
        } else {
            for (int k = 0; k < 16; ++k)
                if (at + k >= b.p0 && at + k < b.p1)
                    *reinterpret_cast<uint8_t*>(at + k) = 0;
        }
    }
}

// Zeros all jobs' outputs.  Workgroups [0, table): batched_table's work.  The
// next `shared`: what jobs are longer than parts * kPartSteps steps, in equal
// shares over 1024 jobs at a time, whatever the jobs' sizes.  The rest, `parts`
// per job: the job's first parts * kPartSteps steps.  (Without the shared ones a
// batch took as long as its largest job's few workgroups: 3147 us for 767 small
// ROIs and one of 1e9 samples, 481 now; parts of 256 and 512 steps: 486, 502.  All
// steps in equal shares over the table need a sum over the table in every
// workgroup: 5 to 20 us more for 768 jobs.)
constexpr uint64_t kPartSteps = 128;
constexpr uint64_t kMostZero = 1 << 20;   // workgroups of one launch (they loop beyond)

__global__ __launch_bounds__(kBlock, 8) void batched_zero_kernel(
    const fvv_job* __restrict__ jobs, uint32_t n_jobs, const fvv_camera* __restrict__ cams,
    float* __restrict__ job_pad, JobPrefix* __restrict__ pre, uint32_t* __restrict__ counter,
    uint32_t* __restrict__ status, uint32_t table, uint32_t shared, uint32_t parts,
    uint8_t* __restrict__ out) {
    if (blockIdx.x < table) {
        batched_table(blockIdx.x, jobs, n_jobs, cams, job_pad, pre, counter, status);
        return;
    }
    const uint64_t most = (uint64_t)parts * kPartSteps;
    if (blockIdx.x >= table + shared) {
        const uint64_t n = (uint64_t)n_jobs * parts;
        for (uint64_t z = blockIdx.x - table - shared; z < n; z += gridDim.x - table - shared) {
            const uint32_t jn = (uint32_t)(z / parts), part = (uint32_t)(z - (uint64_t)jn * parts);
            if (!job_ok(jobs[jn]))
                continue;
            const JobBytes b = job_bytes(jobs[jn], out);
            const uint64_t all = b.steps(), steps = all < most ? all : most;
            zero_steps(b, steps * part / parts, steps * (part + 1) / parts);
        }
        return;
    }
    __shared__ uint64_t s_step[kBatchedJobLds + 1];
    __shared__ uint64_t scratch[kBlock / kWave];
    for (uint32_t base = 0; base < n_jobs; base += kBatchedJobLds) {
        const uint32_t j0 = kPrefixJobs * threadIdx.x;
        uint64_t z[kPrefixJobs], zs = 0, total;
#pragma unroll
        for (int e = 0; e < kPrefixJobs; ++e) {
            z[e] = 0;
            if (base + j0 + e < n_jobs && job_ok(jobs[base + j0 + e])) {
                const uint64_t all = job_bytes(jobs[base + j0 + e], out).steps();
                z[e] = all > most ? all - most : 0ull;
            }
            zs += z[e];
        }
        uint64_t at = block_exclusive_sum64<kBlock>(zs, scratch, &total);
        if (total == 0)
            continue;
#pragma unroll
        for (int e = 0; e < kPrefixJobs; ++e) {
            s_step[j0 + e] = at;
            at += z[e];
        }
        if (threadIdx.x == 0)
            s_step[kBatchedJobLds] = total;
        __syncthreads();
        uint64_t q = total * (blockIdx.x - table) / shared;
        const uint64_t q1 = total * (blockIdx.x - table + 1) / shared;
        auto off = [&](int m) { return s_step[m]; };
        int jn = upper_job(off, kBatchedJobLds, q);
        while (q < q1) {
            while (off(jn + 1) <= q)      // (most jobs have nothing left)
                ++jn;
            const uint64_t first = off(jn), end = off(jn + 1) < q1 ? off(jn + 1) : q1;
            zero_steps(job_bytes(jobs[base + jn], out), most + (q - first), most + (end - first));
            q = end;
        }
        __syncthreads();
    }
}

// Pixels [x0, x0 + 31] of a silhouette row of wpr words, bit b = pixel x0 + b
// (pixels past the row are 0): the two words around x0, kept inside the row.
__device__ __forceinline__ uint32_t row_window(const uint32_t* __restrict__ row, int wpr, int x0) {
    const int w = min(x0 >> 5, max(wpr - 2, 0));
    uint64_t v = row[w];
    if (wpr > 1)
        v |= (uint64_t)row[w + 1] << 32;
    return (uint32_t)(v >> (x0 - 32 * w));
}

// Classification of camera c for the box of samples with world corners lo, hi
// by one lane, from the packed rows of its silhouette: rectangles of more than
// 16 x 32 pixels are mixed; win: the first 8 x 8 pixels of the rectangle, bit
// 8 r + x, org: its corner (x | y << 16) where it fits those, else kNoWindow.
template <class Cams>
__device__ __forceinline__ int classify_small(const Cams& cams, int c,
                                              const uint32_t* __restrict__ sil, const float* lo,
                                              const float* hi, uint64_t& win, uint32_t& org) {
    int cx0, cx1, cy0, cy1;
    bool inside;
    const int st = box_rect(cams, c, lo, hi, cx0, cx1, cy0, cy1, inside);
    win = 0ull;
    org = kNoWindow;
    if (st >= 0)
        return st;
    if (cy1 - cy0 >= 16 || cx1 - cx0 >= 32)
        return kCullMixed;
    const uint32_t m = ~0u >> (31 - (cx1 - cx0));
    uint32_t any = 0u, all = m;
#pragma unroll
    for (int r = 0; r < 8; ++r) {     // rows past the last repeat it
        const uint32_t v =
            row_window(sil + (int64_t)min(cy0 + r, cy1) * cams.wpr, cams.wpr, cx0);
        any |= v & m;
        all &= v;
        win |= (uint64_t)(v & 0xffu) << (8 * r);
    }
    if (cy1 - cy0 >= 8) {
#pragma unroll
        for (int r = 8; r < 16; ++r) {
            const uint32_t v =
                row_window(sil + (int64_t)min(cy0 + r, cy1) * cams.wpr, cams.wpr, cx0);
            any |= v & m;
            all &= v;
        }
    }
    if (cy1 - cy0 < 8 && cx1 - cx0 < 8)
        org = (uint32_t)cx0 | ((uint32_t)cy0 << 16);
    if (any == 0u)
        return kCullReject;
    return inside && all == m ? kCullAccept : kCullMixed;
}

// The four cameras' bits of a ballot over lanes (b, c) = (l % 16, l / 16), ORed.
__device__ __forceinline__ uint32_t any_camera16(uint64_t m) {
    return (uint32_t)((m | (m >> 16) | (m >> 32) | (m >> 48)) & 0xffffull);
}

// A small batch in one pass, a workgroup per strip: the cameras classified for
// four tiles of 64 samples along x at once, a wave each, then those that no
// camera rejects carved by the workgroup (the output is zero before).
template <bool kLds>
__device__ __forceinline__ void carve_strips(const fvv_job* __restrict__ jobs, int nj,
                                             const JobPrefix* __restrict__ pre,
                                             const fvv_camera* __restrict__ cams,
                                             const float* __restrict__ job_pad,
                                             const uint32_t* __restrict__ sils,
                                             uint8_t* __restrict__ out, uint64_t* lds) {
    constexpr uint32_t TX = kBlock / kStripY;
    __shared__ int32_t s_cls[kGroup][2];      // rejecting, mixed cameras
    const auto off = load_offsets<kLds, true>(pre, nj, lds);
    const XcdSlice xs = xcd_slice(off(nj));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (uint64_t strip = xs.begin + xs.slot; strip < xs.end; strip += xs.stride) {
        const int j = __builtin_amdgcn_readfirstlane(upper_job(off, nj, strip));
        const fvv_job& job = jobs[j];
        const fvv_grid g = job.grid;
        const JobCams jc = job_cams(job, j, cams, job_pad);
        const uint32_t r = (uint32_t)(strip - off(j));
        const uint32_t nty = ((uint32_t)g.dims[1] + kStripY - 1u) / kStripY;
        const int j0 = (int)(r % nty) * kStripY, k0 = (int)(r / nty) * 4;
        for (uint32_t x0 = 0; x0 < (uint32_t)g.dims[0]; x0 += TX * kGroup) {
            __syncthreads();                  // the last tiles are done with s_cls
            if (x0 + TX * wave < (uint32_t)g.dims[0]) {
                uint32_t rej, mix;
                classify_tile<TX, kRowRectWords, true>(jc, sils + job.sil_base, g, (int)(x0 + TX * wave),
                                                 j0, k0, rej, mix);
                if (lane_id() == 0) {
                    s_cls[wave][0] = (int32_t)rej;
                    s_cls[wave][1] = (int32_t)mix;
                }
            }
            __syncthreads();
            for (int w = 0; w < kGroup && x0 + TX * w < (uint32_t)g.dims[0]; ++w)
                if (uniform(s_cls[w][0]) == 0)
                    carve_tile_culled<TX>(jc, sils + job.sil_base, g, (int)(x0 + TX * w), j0, k0,
                                          out + job.out_offset, RowBits{}, false,
                                          (uint32_t)uniform(s_cls[w][1]));
        }
    }
}

template <bool kLds>
__global__ __launch_bounds__(kBlock, 8) void batched_mark_kernel(
    const fvv_job* __restrict__ jobs, const JobPrefix* __restrict__ pre,
    const uint32_t* __restrict__ counter, const fvv_camera* __restrict__ cams,
    const float* __restrict__ job_pad, const uint32_t* __restrict__ sils,
    uint8_t* __restrict__ out) {
    __shared__ uint64_t s_off[kLds ? kBatchedJobLds + 1 : 1];
    const int nj = (int)counter[2];
    if (pre[nj].tile_off == 0) {
        carve_strips<kLds>(jobs, nj, pre, cams, job_pad, sils, out, s_off);
        return;
    }
    const auto off = load_offsets<kLds>(pre, nj, s_off);
    // units one by one (a wave waits for two classifications each) until there is
    // a group for every wave, then group by group (most groups are rejected with
    // one): 64 nearly empty ROIs of 2.9e7 samples in 11 and 32 cameras (1e4 units)
    // take the call 64 and 125 us one by one, 83 and 183 in groups; 192 of 2.3e8 in
    // 4 cameras (4e4 units) 99 and 93
    const uint64_t total = off(nj);
    const int per = total <= (uint64_t)gridDim.x * kGroup * kUnitGroup ? 1 : kUnitGroup;
    const XcdSlice xs = xcd_slice(total / per);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint64_t step = (uint64_t)xs.stride * kGroup;
    uint64_t grp = xs.begin + (uint64_t)xs.slot * kGroup + wave;
    int jb = 0;
    if (grp < xs.end)
        jb = upper_job(off, nj, grp * per);
    for (; grp < xs.end; grp += step) {
        const uint64_t unit = grp * per;
        while (jb + 1 < nj && off(jb + 1) <= unit)   // units ascend
            ++jb;
        const int j = __builtin_amdgcn_readfirstlane(jb);
        const fvv_job& job = jobs[j];
        const fvv_grid g = job.grid;
        const JobCams jc = job_cams(job, j, cams, job_pad);
        const BatchedUnit u = batched_unit(job, (uint32_t)(unit - off(j)));
        auto rejected = [&](int j0, int rows) {
            float lo[3], hi[3];
            box_corners(g, 0, g.dims[0] - 1, j0, j0 + min(rows, g.dims[1] - j0) - 1, u.k0,
                        min(u.k0 + 4, g.dims[2]) - 1, lo, hi);
            uint32_t rej, mix;
            classify_box_wave<kRowRectWords, true>(jc, sils + job.sil_base,
                                                   (int64_t)jc.H * jc.wpr, lo, hi, rej, mix);
            return rej != 0u;
        };
        if (!u.on || (per > 1 && rejected(u.j0, kUnitY * kUnitGroup)))
            continue;
        for (int q = 0; q < per; ++q) {
            if (q * kUnitY >= g.dims[1] - u.j0)
                break;
            const int j0 = u.j0 + q * kUnitY;
            if (rejected(j0, kUnitY))
                continue;
            // its tiles, 16 at a time: lane (b, c) = (tile, camera of four)
            const int lane = lane_id(), b = lane & 15, cl = lane >> 4;
            const uint32_t nx = (uint32_t)g.dims[0];   // (unsigned: the steps go past nx)
            for (uint32_t x = 16 * b; __ballot(x < nx) != 0ull; x += 256) {
                float lo[3], hi[3];
                const int i0 = (int)min(x, nx - 1u);
                box_corners(g, i0, i0 + min(16, g.dims[0] - i0) - 1, j0,
                            j0 + min(kUnitY, g.dims[1] - j0) - 1, u.k0, min(u.k0 + 4, g.dims[2]) - 1,
                            lo, hi);
                uint32_t live = (uint32_t)(__ballot(x < nx) & 0xffffull);
                for (int cb = 0; cb < jc.n && live != 0u; cb += 4) {
                    const int c = cb + cl;
                    int cls = kCullMixed;
                    uint64_t win;
                    uint32_t org;
                    if (c < jc.n && ((live >> b) & 1u))
                        cls = classify_small(jc, c, sils + job.sil_base + (int64_t)c * jc.H * jc.wpr,
                                             lo, hi, win, org);
                    live &= ~any_camera16(__ballot(cls == kCullReject));
                }
                if (lane < 16 && x < nx)
                    out[u.at + (int64_t)q * kUnitY * g.dims[0] + i0] =
                        (live >> b) & 1u ? kLiveMark : kDeadMark;
            }
        }
    }
}

// A tile of 16 x 16 x 4 samples (from i0, j0, k0) by one wave, without
// workgroup barriers.  Four cameras at a time:
//   1. lane (b, c) = (lane % 16, lane / 16) classifies camera cb + c for the
//      tile's 4 x 4 x 4 sub-block b from its padded corner rectangle, if that
//      is at most 16 x 32 pixels (else mixed); a mixed rectangle of at most
//      8 x 8 pixels stays in the lane as a 64-bit window;
//   2. the mixed (sub-block, camera) pairs of the sub-blocks no camera rejected
//      are tested with lane = sample, the pixel from the pair's window or,
//      without one, from the packed rows.
// Returns in lane b < 16 the occupancy of sub-block b, sample (x, y, z) at bit
// x + 4 y + 16 z, for the sub-blocks in the mask `sub`, else 0 (the lanes past
// them hold nothing of use).
template <class Cams>
__device__ __forceinline__ uint64_t carve_tile16(const Cams& cams,
                                                 const uint32_t* __restrict__ sils,
                                                 const fvv_grid& g, int i0, int j0, int k0,
                                                 uint32_t sub) {
    const int lane = lane_id(), b = lane & 15, cl = lane >> 4;
    const int64_t cam_words = (int64_t)cams.H * cams.wpr;
    const int nx = g.dims[0], ny = g.dims[1], nz = g.dims[2];
    const int si = i0 + 4 * (b & 3), sj = j0 + 4 * (b >> 2);
    const bool sb_on = si < nx && sj < ny && ((sub >> b) & 1u);
    float lo[3], hi[3];
    const int bi = min(si, nx - 1), bj = min(sj, ny - 1);
    box_corners(g, bi, bi + min(4, nx - bi) - 1, bj, bj + min(4, ny - bj) - 1, k0,
                min(k0 + 4, nz) - 1, lo, hi);
    // sample masks of the sub-block's x, y and z inside the lattice
    uint64_t occ = 0ull;
    if (sb_on) {
        const uint64_t mx = 0xfull >> (4 - min(nx - si, 4)), my = (1ull << (4 * min(ny - sj, 4))) - 1ull;
        const uint64_t row = (mx * 0x1111ull) & my;
        const int mz = min(nz - k0, 4);
        occ = (row * 0x0001000100010001ull) & (~0ull >> (16 * (4 - mz)));
    }
    const float Z = lattice_coord(g.lo[2] + k0 + (lane >> 4), g.h, g.origin[2]);
    for (int cb = 0; cb < cams.n; cb += 4) {
        const uint32_t live = (uint32_t)(__ballot(occ != 0ull) & 0xffffull);
        if (live == 0u)
            break;
        const int c = cb + cl;
        int cls = kCullAccept;
        uint64_t win = 0ull;
        uint32_t org = kNoWindow;
        if (c < cams.n && ((live >> b) & 1u))
            cls = classify_small(cams, c, sils + c * cam_words, lo, hi, win, org);
        const uint32_t rej = any_camera16(__ballot(cls == kCullReject));
        if ((rej >> b) & 1u)
            occ = 0ull;
        const uint64_t mb = __ballot(cls == kCullMixed);
        // camera after camera (its matrix stays in scalar registers), its mixed
        // sub-blocks that are still alive, two at a time (independent chains)
        for (int q = 0; q < 4; ++q) {
            uint32_t todo = (uint32_t)(mb >> (16 * q)) & (uint32_t)__ballot(occ != 0ull) & 0xffffu;
            if (todo == 0u)
                continue;
            const int cc = cb + q;
            float P[12];
#pragma unroll
            for (int e = 0; e < 12; ++e)
                P[e] = cams.Pc(cc)[e];
            while (todo != 0u) {
                uint64_t left[2];
                int sb[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int t = __ffs(todo) - 1, src = 16 * q + t;
                    if (k == 1 || (todo & (todo - 1u)) != 0u)
                        todo &= todo - 1u;   // (the last one again where there is no second)
                    sb[k] = t;
                    const float X = lattice_coord(g.lo[0] + i0 + 4 * (t & 3) + (lane & 3), g.h,
                                                  g.origin[0]);
                    const float Y = lattice_coord(g.lo[1] + j0 + 4 * (t >> 2) + ((lane >> 2) & 3),
                                                  g.h, g.origin[1]);
                    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)org, src);
                    const uint64_t w =
                        ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(win >> 32), src) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)win, src);
                    int px, py;
                    const bool ok = point_pixel_exact(P, X, Y, Z, cams.W, cams.H, px, py);
                    bool in = (w >> ((8 * (py - (int)(o >> 16)) + px - (int)(o & 0xffffu)) & 63)) & 1ull;
                    if (o == kNoWindow) {
                        uint32_t v = 0u;
                        if (ok)
                            v = sils[cc * cam_words + (int64_t)py * cams.wpr + (px >> 5)];
                        in = (v >> (px & 31)) & 1u;
                    }
                    left[k] = __ballot(ok && in);
                }
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (lane == sb[k])
                        occ &= left[k];
            }
        }
    }
    return occ;
}

// Four occupancy bits as bytes.
__device__ __forceinline__ uint32_t nibble_bytes(uint32_t n) {
    return (n * 0x00204081u) & 0x01010101u;
}

// The 16 samples along x of row y, layer z of a tile from carve_tile16's
// lanes: lane = y + 16 z gets bit x.
__device__ __forceinline__ uint32_t tile16_row(uint64_t occ) {
    const int lane = lane_id(), y = lane & 15, z = lane >> 4;
    const int sh = 4 * (y & 3) + 16 * (z & 1);
    uint32_t bits = 0u;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int src = 4 * (y >> 2) + s;
        const uint32_t l = (uint32_t)__shfl((int)(uint32_t)occ, src);
        const uint32_t h = (uint32_t)__shfl((int)(uint32_t)(occ >> 32), src);
        bits |= (((z >> 1) ? h : l) >> sh & 0xfu) << (4 * s);
    }
    return bits;
}

// Store a row's 16 bytes (the first n of them) at o, at any alignment.
__device__ __forceinline__ void store_row16(uint8_t* o, uint32_t bits, int n) {
    uint32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        v[k] = nibble_bytes((bits >> (4 * k)) & 0xfu);
    if (n >= 16)
        __builtin_memcpy(o, v, 16);
    else
        for (int x = 0; x < n; ++x)
            o[x] = (uint8_t)((bits >> x) & 1u);
}

template <bool kLds>
__global__ __launch_bounds__(kBlock, 6) void carve_batched_culled_kernel(
    const fvv_job* __restrict__ jobs, const JobPrefix* __restrict__ pre,
    const uint32_t* __restrict__ counter, const fvv_camera* __restrict__ cams,
    const float* __restrict__ job_pad, const uint32_t* __restrict__ sils,
    uint8_t* __restrict__ out) {
    __shared__ uint64_t s_off[kLds ? kBatchedJobLds + 1 : 1];
    __shared__ float s_cam[FVV_MAX_CAMS][13];
    // the marks as the first wave read them, by turns (a turn's readers have
    // passed the next one's barrier before it is written again).  All waves go by
    // these: another workgroup may be writing the same bytes, where two jobs share
    // output, and waves that each read them could disagree about the tiles and the
    // barriers.  (852.9 us for 64 frames x 12 ROIs, 845.0 with each reading them;
    // units read 64 at a time without barriers between spilled registers: 896.)
    __shared__ uint64_t s_todo[2], s_live[2];
    const int nj = (int)counter[2];
    const auto off = load_offsets<kLds>(pre, nj, s_off);
    const XcdSlice xs = xcd_slice(off(nj));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = lane_id();
    int staged = -1, todo_turn = 0, live_turn = 0;
    // the marks of 64 of the workgroup's units at a time, then the marked ones
    for (uint64_t base = xs.begin + xs.slot; base < xs.end; base += (uint64_t)xs.stride * kWave) {
        const uint64_t mine = base + (uint64_t)xs.stride * lane;
        int jl = 0;
        bool kept = false;
        if (mine < xs.end) {
            jl = upper_job(off, nj, mine);
            const BatchedUnit u = batched_unit(jobs[jl], (uint32_t)(mine - off(jl)));
            kept = wave == 0 && u.on && out[u.at] >= kDeadMark;
        }
        const uint64_t marked = __ballot(kept);
        if (threadIdx.x == 0)
            s_todo[todo_turn] = marked;
        __syncthreads();   // the marks are read; the carve overwrites them
        uint64_t todo = uniform(s_todo[todo_turn]);
        todo_turn ^= 1;
        for (; todo != 0ull; todo &= todo - 1ull) {
            const int bit = __ffsll((unsigned long long)todo) - 1;
            const int j = __builtin_amdgcn_readlane(jl, bit);
            const fvv_job& job = jobs[j];
            const fvv_grid g = job.grid;
            const LdsCams jc{s_cam, job.n_cams, job.width, job.height, (job.width + 31) / 32};
            const BatchedUnit u =
                batched_unit(job, (uint32_t)(base + (uint64_t)xs.stride * bit - off(j)));
            uint8_t* const p = out + u.at;
            // the job's cameras: a tile reads each several times in a row of
            // dependent steps
            if (j != staged) {
                __syncthreads();   // the previous job's tiles are done with them
                for (int i = threadIdx.x; i < jc.n * 13; i += kBlock) {
                    const int c = i / 13, e = i - 13 * c;
                    s_cam[c][e] = e < 12 ? cams[job.cam_base + c].P[e]
                                         : job_pad[(int64_t)j * FVV_MAX_CAMS + c];
                }
                staged = j;
            }
            const uint32_t nx = (uint32_t)g.dims[0];   // (unsigned: the steps go past nx)
            for (uint32_t x0 = 0; x0 < nx; x0 += 16 * kWave) {
                // 64 tiles' marks; a dead tile is zero but for its mark
                if (wave == 0) {
                    const uint32_t x = x0 + 16 * lane;
                    const uint8_t mark = x < nx ? p[x] : 0;
                    const uint64_t marked = __ballot(mark == kLiveMark);
                    if (lane == 0)
                        s_live[live_turn] = marked;
                    if (mark == kDeadMark)
                        p[x] = 0;
                }
                __syncthreads();   // the marks are read; the cameras are staged
                uint64_t live = uniform(s_live[live_turn]);
                live_turn ^= 1;
                // a tile per wave; one or two tiles are shared out in 4 or 2
                // parts of 4 or 8 rows (the waves would idle)
                const int nl = __popcll(live);
                const int parts = nl == 1 ? 4 : nl == 2 ? 2 : 1, rows = 16 / parts;
                const int part = wave % parts;
                const uint32_t sub = parts == 1 ? 0xffffu : ((1u << rows) - 1u) << (part * rows);
                for (int q = 0; live != 0ull; live &= live - 1ull, ++q) {
                    if (q % (kGroup / parts) != wave / parts)
                        continue;
                    const int i0 = (int)x0 + 16 * (__ffsll((unsigned long long)live) - 1);
                    const uint32_t row =
                        tile16_row(carve_tile16(jc, sils + job.sil_base, g, i0, u.j0, u.k0, sub));
                    const int y = lane & 15, z = lane >> 4;
                    if (y < g.dims[1] - u.j0 && u.k0 + z < g.dims[2] && y / rows == part)
                        store_row16(p + ((int64_t)z * g.dims[1] + y) * g.dims[0] + i0, row,
                                    min(16, g.dims[0] - i0));
                }
            }
        }
    }
}

hipError_t launch_carve_frame(fvv_ctx* ctx, const fvv_job* jobs, int max_jobs,
                              const CamSet& cams, const uint32_t* sils, const uint64_t* tiles,
                              uint8_t* out, uint64_t* finebits, TileShape t, int blocks,
                              const fvv_grid& coarse, uint8_t* occ_coarse, int32_t* labels,
                              hipStream_t s, hipEvent_t k_start, hipEvent_t k_stop) {
    if (t.tz != 4) {
        // the persistent carve: the events bracket its launch; the labels'
        // write pass goes first
        hipError_t e = launch_label_write(ctx, coarse, occ_coarse, labels, s);
        if (e == hipSuccess && k_start)
            e = hipEventRecord(k_start, s);
        if (e == hipSuccess)
            e = launch_carve_batched(ctx, jobs, 0, ctx->d_cams, sils, out, finebits, t, blocks,
                                     true, s);
        if (e == hipSuccess && k_stop)
            e = hipEventRecord(k_stop, s);
        return e;
    }
    blocks = (blocks + kXcds - 1) / kXcds * kXcds;
    // the coarse labels' write pass rides in the same launch, in workgroups
    // after the carve's: eight samples or more per thread, at most 16
    // workgroups per CU (2.3e7 samples: 58, 48, 40, 40, 41 us with 1, 2, 8, 16
    // and 32; 40 to 45 with them first)
    LabelWrite lw = label_write_args(ctx, coarse, occ_coarse, labels);
    lw.carve_blocks = (uint32_t)blocks;
    const int64_t lw_blocks = (lw.V + 8 * kBlock - 1) / (8 * kBlock);
    const int extra = (int)(lw_blocks < 1 ? 1 : (lw_blocks > 16 * ctx->n_cus ? 16 * ctx->n_cus
                                                                              : lw_blocks));
    // jobs: max_jobs entries; the prefix table holds at least max_jobs + 1
    const int job_lds = max_jobs < kJobLds ? max_jobs : kJobLds;
#define X(TXV)                                                                                 \
    if (t.tx == TXV) {                                                                         \
        hipExtLaunchKernelGGL((carve_frame_kernel<TXV>), dim3(blocks + extra), dim3(kBlock), 0, \
                              s, k_start, k_stop, 0, jobs, ctx->d_prefix, ctx->d_counter, cams, \
                              sils, tiles, ctx->d_rho, out, finebits, job_lds, lw);            \
        return hipGetLastError();                                                              \
    }
    X(64) X(32) X(16)
#undef X
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------ dispatch
#define FVV_TILE_CASES(X)                                                                  \
    X(64, 1) X(64, 2) X(64, 4) X(64, 8) X(32, 1) X(32, 2) X(32, 4) X(32, 8) X(16, 1)     \
    X(16, 2) X(16, 4) X(16, 8)

hipError_t launch_carve(const CamSet& cams, const uint32_t* sils, const fvv_grid& g, TileShape t,
                        uint8_t* occ, const RowBits* rows, hipStream_t s,
                        const CarveReject* rej) {
    const uint64_t tiles = tiles_of_grid(g, t.tx, t.tz);
    if (tiles == 0)
        return hipSuccess;
    if (tiles > 0x7fffffffull)
        return hipErrorInvalidValue;
    const RowBits rb = rows ? *rows : RowBits{};
    if (t.tz == 4) {                      // camera culling per tile and per 4x4x4 sub-block
#define X(TXV)                                                                                \
        if (t.tx == TXV) {                                                                    \
            hipLaunchKernelGGL((carve_culled_kernel<TXV>), dim3((unsigned)tiles), dim3(kBlock), \
                               0, s, cams, sils, g, occ, rb);                                 \
            return hipGetLastError();                                                         \
        }
        X(64)
        X(32)
        X(16)
#undef X
        return hipErrorInvalidValue;
    }
    const uint64_t V = (uint64_t)g.dims[0] * (uint64_t)g.dims[1] * (uint64_t)g.dims[2];
    if (rej && V >= kRejectMinSamples) {
        RejBoxes boxes;
        boxes.nbx = (uint32_t)((g.dims[0] + 7) / 8);
        boxes.nby = (uint32_t)((g.dims[1] + 7) / 8);
        const uint64_t nb = (uint64_t)boxes.nbx * boxes.nby * (uint64_t)((g.dims[2] + 3) / 4);
        if (nb > 0x7fffffffull)
            return hipErrorInvalidValue;
        boxes.n = (uint32_t)nb;
        boxes.by_nbx = divu32_magic(boxes.nbx);
        boxes.by_nby = divu32_magic(boxes.nby);
        const int per_wg = kBlock / cams.n < kWave ? kBlock / cams.n : kWave;
        const unsigned rblocks = (unsigned)((nb + per_wg - 1) / per_wg);
        hipLaunchKernelGGL(carve_reject_kernel, dim3(rblocks), dim3(kBlock), 0, s, cams, rej->any,
                           g, occ, boxes, per_wg, divu32_magic((uint32_t)cams.n), rej->list,
                           rej->count);
        // four workgroups per CU: every wave of the second pass resident at once
        const unsigned kblocks = (unsigned)rej->n_cus * 4;
        uint64_t* const any_bits = const_cast<uint64_t*>(rej->any.bits);
        const int64_t any_words = (int64_t)cams.n * rej->any.tph * rej->any.bw;
        if (rows)
            hipLaunchKernelGGL(carve_kept_kernel<true>, dim3(kblocks), dim3(kBlock), 0, s, cams,
                               sils, g, occ, rb, rej->list, rej->count, boxes, any_bits,
                               any_words);
        else
            hipLaunchKernelGGL(carve_kept_kernel<false>, dim3(kblocks), dim3(kBlock), 0, s, cams,
                               sils, g, occ, rb, rej->list, rej->count, boxes, any_bits,
                               any_words);
        return hipGetLastError();
    }
#define X(TXV, TZV)                                                                           \
    if (t.tx == TXV && t.tz == TZV) {                                                         \
        if (rows)                                                                             \
            hipLaunchKernelGGL((carve_kernel<TXV, TZV, true>), dim3((unsigned)tiles),         \
                               dim3(kBlock), 0, s, cams, sils, g, occ, rb);                   \
        else                                                                                  \
            hipLaunchKernelGGL((carve_kernel<TXV, TZV, false>), dim3((unsigned)tiles),        \
                               dim3(kBlock), 0, s, cams, sils, g, occ, rb);                   \
        return hipGetLastError();                                                             \
    }
    FVV_TILE_CASES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_carve_batched(fvv_ctx* ctx, const fvv_job* jobs, uint32_t n_jobs,
                                const fvv_camera* cams, const uint32_t* sils, uint8_t* out,
                                uint64_t* finebits, TileShape t, int blocks, bool jobs_prepared,
                                hipStream_t s) {
    // a fresh job table carved without fine bitmaps, 4 samples deep: culled
    if (!jobs_prepared && !finebits && t.tz == 4) {
        // workgroups for the marked units: 32 per CU (8, 16, 32 and 64 take
        // 840, 812, 803 and 825 us on 64 frames x 12 ROIs), fewer for a small
        // table (1000 workgroups take 1 us to start)
        const uint64_t most = (uint64_t)ctx->n_cus * 32;
        uint64_t want = (uint64_t)n_jobs * 32;
        want = want < most / 4 ? most / 4 : want > most ? most : want;
        blocks = (int)((want + kXcds - 1) / kXcds * kXcds);
        const uint64_t pairs = (uint64_t)n_jobs * FVV_MAX_CAMS;
        // the first two passes' waves stay resident: eight workgroups per CU
        const unsigned rblocks = (unsigned)((ctx->n_cus * 8 + kXcds - 1) / kXcds * kXcds);
        const unsigned table = 1u + (unsigned)((pairs + kBlock - 1) / kBlock);
        // zeroing: a workgroup per CU for the long jobs' rest (four times fewer for a
        // large table, whose sum takes each of them a while: one writes 57 GB/s), and
        // for the jobs' parts 64 per job, at least 1 and at most about 16 per CU
        const unsigned cus = (unsigned)ctx->n_cus;
        const unsigned shared = n_jobs <= (uint32_t)kBatchedJobLds ? cus : (cus + 3) / 4;
        const unsigned most_zero = cus * 16, few = n_jobs < most_zero / 64 ? n_jobs * 64 : most_zero;
        const unsigned parts = ((few < cus ? cus : few) + n_jobs - 1) / n_jobs;
        const uint64_t zeroing = (uint64_t)n_jobs * parts;
        hipLaunchKernelGGL(batched_zero_kernel,
                           dim3(table + shared + (unsigned)(zeroing < kMostZero ? zeroing : kMostZero)),
                           dim3(kBlock), 0, s, jobs, n_jobs, cams, ctx->d_job_pad, ctx->d_prefix,
                           ctx->d_counter, ctx->d_status, table, shared, parts, out);
        if (n_jobs <= (uint32_t)kBatchedJobLds) {
            hipLaunchKernelGGL((batched_mark_kernel<true>), dim3(rblocks), dim3(kBlock), 0, s,
                               jobs, ctx->d_prefix, ctx->d_counter, cams, ctx->d_job_pad, sils,
                               out);
            hipLaunchKernelGGL((carve_batched_culled_kernel<true>), dim3(blocks), dim3(kBlock), 0,
                               s, jobs, ctx->d_prefix, ctx->d_counter, cams, ctx->d_job_pad, sils,
                               out);
        } else {
            hipLaunchKernelGGL((batched_mark_kernel<false>), dim3(rblocks), dim3(kBlock), 0, s,
                               jobs, ctx->d_prefix, ctx->d_counter, cams, ctx->d_job_pad, sils,
                               out);
            hipLaunchKernelGGL((carve_batched_culled_kernel<false>), dim3(blocks), dim3(kBlock),
                               0, s, jobs, ctx->d_prefix, ctx->d_counter, cams, ctx->d_job_pad,
                               sils, out);
        }
        return hipGetLastError();
    }
#define X(TXV, TZV)                                                                             \
    if (t.tx == TXV && t.tz == TZV) {                                                           \
        if (!jobs_prepared)                                                                     \
            hipLaunchKernelGGL((batched_prepare_kernel<TXV, TZV>), dim3(1), dim3(kBlock), 0, s,  \
                               jobs, n_jobs, ctx->d_prefix, ctx->d_counter, ctx->d_status,       \
                               (uint32_t)blocks);                                               \
        if (finebits)                                                                           \
            hipLaunchKernelGGL((carve_persistent_kernel<TXV, TZV, true>), dim3(blocks),          \
                               dim3(kBlock), 0, s, jobs, ctx->d_prefix, ctx->d_counter, cams,    \
                               sils, out, finebits);                                            \
        else                                                                                    \
            hipLaunchKernelGGL((carve_persistent_kernel<TXV, TZV, false>), dim3(blocks),         \
                               dim3(kBlock), 0, s, jobs, ctx->d_prefix, ctx->d_counter, cams,    \
                               sils, out, finebits);                                            \
        return hipGetLastError();                                                               \
    }
    FVV_TILE_CASES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace fvv

#ifdef FVV_CARVE_PROBE
// Measurement builds only: the fine carve's probe tables to host memory
// (blocks: kProbeWaves * kProbeIters * 3 words, waves: kProbeWaves * 3), and
// their clearing before a run.
extern "C" int32_t fvv_carve_probe_read(uint64_t* blocks, uint64_t* waves) {
    if (!blocks || !waves)
        return FVV_EINVAL;
    hipError_t e = hipMemcpyFromSymbol(blocks, HIP_SYMBOL(fvv::carve_probe_blocks),
                                       sizeof(fvv::carve_probe_blocks));
    if (e == hipSuccess)
        e = hipMemcpyFromSymbol(waves, HIP_SYMBOL(fvv::carve_probe_waves),
                                sizeof(fvv::carve_probe_waves));
    return e == hipSuccess ? FVV_OK : FVV_EDEVICE;
}

extern "C" int32_t fvv_carve_probe_clear() {
    void* b = nullptr;
    void* w = nullptr;
    hipError_t e = hipGetSymbolAddress(&b, HIP_SYMBOL(fvv::carve_probe_blocks));
    if (e == hipSuccess)
        e = hipGetSymbolAddress(&w, HIP_SYMBOL(fvv::carve_probe_waves));
    if (e == hipSuccess)
        e = hipMemset(b, 0, sizeof(fvv::carve_probe_blocks));
    if (e == hipSuccess)
        e = hipMemset(w, 0, sizeof(fvv::carve_probe_waves));
    if (e == hipSuccess)
        e = hipDeviceSynchronize();
    return e == hipSuccess ? FVV_OK : FVV_EDEVICE;
}
#endif
