// 3x3x3 volumetric convolution + folded batch norm + activation
// (Section 4.1 "Feature Aggregation"; fixed-offset kernel of Section 3, Eq. 1).
//
// bf16 path: implicit GEMM on the MFMA units. M = output voxels, N = output
// channels, K = 27 taps x input channels.
//
//  * One workgroup per CU owns an 8x8x8 brick of output voxels and 32*NB
//    output channels. Its waves form 4 voxel groups x WCH channel groups:
//    each wave computes two u-slices of the brick (128 voxels) against
//    32*NB/WCH channels with v_mfma_f32_32x32x16_bf16: A = weights (rows =
//    output channels), B = voxels (columns), 4 x NB/WCH accumulator blocks,
//    so every voxel fragment feeds NB/WCH MFMAs and every weight fragment
//    four. WCH = 1: four waves, one per SIMD; WCH = 2 (eight waves, two per
//    SIMD, so that one wave's waits overlap the other's MFMAs) for
//    64-channel tiles of narrow inputs on small grids. Inputs of up to 128 channels on grids with enough tiles
//    take 64-channel tiles with compact halos (SB): 72 KB of LDS and at
//    most 128 accumulator registers per wave, so two workgroups share a CU
//    and one's prologue and epilogue overlap the other's MFMAs.
//  * The input is consumed in chunks of 16 channels (one MFMA k step). A
//    chunk's 10x10x10 halo (zero outside the grid) sits in LDS at 48 bytes per
//    voxel (32 bytes of data) and 640 bytes per 10-voxel row: with that
//    padding the 16-byte fragment reads of every tap hit distinct banks (SB:
//    32 bytes per voxel, the two halves swapped where bit 2 of w is set, the
//    same effect). The next chunk's halo is fetched into the other of two
//    buffers during the first taps of the current chunk.
//  * The 27 taps of a chunk are unrolled, so every LDS fragment address is a
//    per-lane base plus an immediate. Weights come pre-packed in fragment
//    order (pv_pack_conv_weights_kernel): each fragment load is one coalesced
//    1 KB buffer load, issued two taps ahead into registers. The only barrier
//    is one per chunk.
//  * The epilogue folds bias + batch norm into one scale/shift per channel
//    (a table in LDS), applies the activation and stages the tile through
//    LDS so that every store instruction writes whole contiguous rows.
//
// fp32 path: four lanes per (voxel, output channel), plain FMA loops.
#include <algorithm>

#include "pv_common.h"
#include "pv_trilinear.h"

namespace {

constexpr int kBrick = 8;                          // output brick edge (u, v, w)
constexpr int kHalo = kBrick + 2;                  // halo edge
constexpr int kHaloVox = kHalo * kHalo * kHalo;    // 1000
constexpr int kKC = 16;                            // input channels per chunk
constexpr int kVoxPitch = 48;                      // LDS bytes per halo voxel
constexpr int kRowPitch = 640;                     // LDS bytes per 10-voxel row
constexpr int kHaloBytes = kHalo * kHalo * kRowPitch;  // 64000 per buffer
constexpr int kPieces = kHaloVox * 2;              // 16-byte pieces per chunk halo
constexpr int kTaps = 27;
constexpr int kOOB = 0x40000000;                   // byte offset always out of range
// Epilogue staging: the output tile goes through LDS as [512 voxels][PW
// channels] rows of up to 256 bytes, padded by 16 bytes, then out with
// coalesced 16-byte stores.
constexpr int kStageRow = 256 + 16;
constexpr int kStageBytes = kBrick * kBrick * kBrick * kStageRow;  // 139264
constexpr int kLdsBytes = kStageBytes > 2 * kHaloBytes ? kStageBytes : 2 * kHaloBytes;
// Two-workgroups-per-CU variant (SB): the epilogue stages the 64-channel
// tile through LDS in one pass (bf16: whole 128-byte halves of the output
// rows) or two (fp32). Its two halo buffers are compact: 32 bytes per
// voxel, 384 per 10-voxel row (64 bytes of padding: consecutive rows start
// half a 256-byte bank window apart), and the two 16-byte halves of a voxel
// swap places where bit 2 of its w is set, so that the 16 lanes of a
// fragment read that are served together (8 consecutive voxels of two
// consecutive rows) hit distinct banks.
constexpr int kStageRowSB = 128 + 16;
constexpr int kVoxPitchSB = 32;
constexpr int kRowPitchSB = kHalo * kVoxPitchSB + 64;            // 384
constexpr int kHaloBytesSB = kHalo * kHalo * kRowPitchSB;        // 38400 per buffer
constexpr int kLdsBytesSB =
    512 * kStageRowSB > 2 * kHaloBytesSB ? 512 * kStageRowSB : 2 * kHaloBytesSB;

__device__ __forceinline__ uint4 pack8(const uint16_t* e) {
    return make_uint4((uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16),
                      (uint32_t)e[4] | ((uint32_t)e[5] << 16), (uint32_t)e[6] | ((uint32_t)e[7] << 16));
}

__device__ __forceinline__ pv_bf16x8 as_frag(uint4 v) {
    pv_bf16x8 r;
    __builtin_memcpy(&r, &v, 16);
    return r;
}

// Raw buffer loads: an offset at or past the resource's size reads as zero,
// which provides the conv's zero padding (and zero channels past C_in)
// without branches or selects on the loaded value.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                             0x00020000);
}

__device__ __forceinline__ uint4 bload16(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    uint4 u;
    __builtin_memcpy(&u, &v, 16);
    return u;
}

// 8 bf16 channels one by one: channel i at voff + 2i if i < valid, else zero.
__device__ __forceinline__ uint4 bload8_elems(__amdgpu_buffer_rsrc_t r, int voff, int soff,
                                              int valid) {
    uint16_t e[8];
#pragma unroll
    for (int i = 0; i < 8; i++)
        e[i] = __builtin_amdgcn_raw_buffer_load_b16(r, i < valid ? voff + 2 * i : kOOB, soff, 0);
    return pack8(e);
}

// WCH channel groups of waves: 1 (four waves, 256 threads) or 2 (eight
// waves, two per SIMD). SB: compact halo buffers and at most 128
// accumulator registers, so that two workgroups share a CU and one's
// prologue and epilogue overlap the other's MFMAs.
// SP (with occ, the forward's first convolution on its sparse grid): an
// MFMA whose 32 input voxels are all empty adds only zeros to accumulators
// that started at +0, so it is skipped (same bits). A bitmap of the halo's
// occupied voxels (one word per halo row) gives each wave, once per brick,
// which of its blocks have an occupied input voxel at each tap.
// Split-K (ksplit > 1): the input channels' chunks are divided among ksplit
// groups of workgroups (cps chunks each); split s reads channels from
// s*cps*16 (rows of x_ld elements), and writes its fp32 partial sums, without
// batch norm or activation, to y + s*B*R^3*Cout (the caller passes an
// identity fold and no activation); pv_conv_split_reduce_kernel adds them.
template <int NB, int WCH, bool VEC, bool SB = false, bool SP = false>
__global__ __launch_bounds__(256 * WCH, SB ? 2 : 1) void pv_conv3d_bf16_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ wpk, PvBnFold bn, int act,
    float slope, void* __restrict__ y, int out_bf16, int vec_out, int R, int Cin, int Cout,
    int nbr, int nblocks, int x_ld, int ksplit, int cps, int B, const int32_t* __restrict__ occ) {
    __shared__ __attribute__((aligned(16))) char lds[SB ? kLdsBytesSB : kLdsBytes];
    __shared__ float bn_tab[2][NB * 32];  // folded scale and shift per output channel
    // SP: occupied w of each halo row
    __shared__ uint32_t occ_row[SP ? kHalo * kHalo : 1];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Blocks are dispatched round-robin over the 8 XCDs; give each XCD a
    // contiguous range of bricks so that neighbouring halos share its L2.
    // With SP a brick's work depends on its cloud's occupancy: there
    // each XCD takes an eighth of every cloud (whole clouds per XCD left the
    // XCDs that drew the denser clouds running long after the others).
    int bid = blockIdx.x;
    const int per = nblocks / max(B, 1);  // workgroups per cloud
    if (SP && (per & 7) == 0 && per * B == nblocks) {
        // every XCD takes one contiguous eighth of every cloud, rotated by
        // the cloud, so that clouds of different occupancy share the XCDs
        const int x = bid & 7, k = bid >> 3, c = k / (per >> 3), j = k % (per >> 3);
        bid = c * per + ((x + c) & 7) * (per >> 3) + j;
    } else if ((nblocks & 7) == 0) {
        bid = (bid & 7) * (nblocks >> 3) + (bid >> 3);
    }
    if (ksplit > 1) {  // this workgroup's share of the input channels
        const int split = bid % ksplit;
        bid /= ksplit;
        const int c_lo = split * cps * kKC;
        x += c_lo;
        wpk += (size_t)split * cps * kTaps * ((Cout + 31) / 32) * 512;
        Cin = min(Cin - c_lo, cps * kKC);
        y = (float*)y + (size_t)split * B * R * R * R * Cout;
    }
    constexpr int NT = NB * 32;
    // Waves = 4 voxel groups x WCH channel groups: each wave owns two u-slices
    // of the brick (4 blocks of 32 voxels) and NBW blocks of 32 channels.
    static_assert(NB % WCH == 0, "channel groups split the tile evenly");
    constexpr int NTH = 256 * WCH, NBW = NB / WCH;
    constexpr int kSets = (kPieces + NTH - 1) / NTH;  // halo pieces per thread
    const int wv = wave / WCH, wc = wave % WCH;
    const int ntiles = (Cout + NT - 1) / NT;  // the last tile may be partly past Cout
    const int nt = bid % ntiles;
    bid /= ntiles;
    const int bw = bid % nbr;
    bid /= nbr;
    const int bv = bid % nbr;
    bid /= nbr;
    const int bu = bid % nbr;
    const int b = bid / nbr;
    const int u0 = bu * kBrick, v0 = bv * kBrick, w0 = bw * kBrick, n0 = nt * NT;
    const size_t cloud = (size_t)b * R * R * R;
    const int nch = (Cin + kKC - 1) / kKC;

    const int r32 = lane & 31, khalf = lane >> 5;
    // LDS byte address of this lane's B fragment (voxel column r32 of block
    // mb, channels khalf*8 .. +7) at tap offset (0,0,0) in buffer 0: block mb
    // covers u = 2*wave + mb/2 and v rows (mb&1)*4 .. +3, eight w each.
    // SB: one base per w shift of the taps (the half swap depends on w).
    constexpr int RP = SB ? kRowPitchSB : kRowPitch, HB = SB ? kHaloBytesSB : kHaloBytes;
    auto half_off = [](int hw, int h) { return SB ? (h ^ ((hw >> 2) & 1)) * 16 : h * 16; };
    // Block mb of the wave: u-slice blk_u(mb), v rows blk_v(mb)*4 .. +3.
    auto blk_u = [&](int mb) -> int { return 2 * wv + (mb >> 1); };
    auto blk_v = [&](int mb) -> int { return mb & 1; };
    int bbase[4], bsw[4][3];
    auto place = [&](int mb, int ul, int vh) {
        const int vl = vh * 4 + (r32 >> 3), wl = r32 & 7;
        bbase[mb] = (ul * kHalo + vl) * kRowPitch + wl * kVoxPitch + khalf * 16;
#pragma unroll
        for (int tw = 0; tw < 3; tw++)
            bsw[mb][tw] = (ul * kHalo + vl) * kRowPitchSB + (wl + tw) * kVoxPitchSB +
                          half_off(wl + tw, khalf);
    };
#pragma unroll
    for (int mb = 0; mb < 4; mb++) place(mb, blk_u(mb), blk_v(mb));
    // LDS byte address (in buffer 0) of block mb's B fragment at tap tn
    auto frag_addr = [&](int mb, int tn) {
        const int tu = tn / 9, tv = (tn / 3) % 3, tw = tn % 3;
        if constexpr (SB) return bsw[mb][tw] + (tu * kHalo + tv) * RP;
        return bbase[mb] + (tu * kHalo + tv) * kRowPitch + tw * kVoxPitch;
    };

    // Halo pieces of this thread: piece p = set*NTH + tid is voxel p/2 (as
    // (hu,hv,hw) of the 10x10x10 halo), channels (p%2)*8 .. +7 of the chunk.
    // Threads past the last piece repeat voxel 999 (same value, same slot).
    // goff: byte offset into the input resource (kOOB outside the grid);
    // loff: LDS byte offset in buffer 0.
    const int ulo = max(u0 - 1, 0), uhi = min(u0 + kBrick + 1, R);
    // rows of x_ld elements, of which the first Cin are this conv's (or this
    // split's) channels; the range ends with the last row's channels
    const size_t slab = (size_t)R * R * x_ld;  // elements per u-slab
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(
        x + cloud * x_ld + ulo * slab, (uint32_t)(((uhi - ulo) * slab - (x_ld - Cin)) * 2));
    const int pq = tid & 1;
    int goff[kSets], loff[kSets];
    if constexpr (SP) {
        if (tid < kHalo * kHalo) occ_row[tid] = 0u;
        __syncthreads();
    }
#pragma unroll
    for (int set = 0; set < kSets; set++) {
        const int h = min(set * (NTH / 2) + (tid >> 1), kHaloVox - 1);
        const int hu = h / (kHalo * kHalo), hv = (h / kHalo) % kHalo, hw = h % kHalo;
        const int gu = u0 + hu - 1, gv = v0 + hv - 1, gw = w0 + hw - 1;
        bool in = gu >= 0 && gu < R && gv >= 0 && gv < R && gw >= 0 && gw < R;
        // a sparse input grid: empty voxels read as zero (their rows were
        // never written), through the out-of-range offset
        if (occ && in) in = occ[cloud + ((size_t)gu * R + gv) * R + gw] > 0;
        if constexpr (SP)
            if (in && pq == 0) atomicOr(&occ_row[hu * kHalo + hv], 1u << hw);
        goff[set] = in ? ((((gu - ulo) * R + gv) * R + gw) * x_ld + pq * 8) * 2 : kOOB;
        loff[set] = SB ? (hu * kHalo + hv) * kRowPitchSB + hw * kVoxPitchSB + half_off(hw, pq)
                       : (hu * kHalo + hv) * kRowPitch + hw * kVoxPitch + pq * 16;
    }
    // Piece of set `set` for the chunk starting at channel cc: pieces whose
    // channels lie past Cin read as zero.
    auto halo_load = [&](int set, int cc) -> uint4 {
        if (VEC) return bload16(xr, cc + pq * 8 < Cin ? goff[set] : kOOB, cc * 2);
        return bload8_elems(xr, goff[set], cc * 2, Cin - cc - pq * 8);
    };

    // Packed weights: for chunk c, tap t and 32-channel output group g the 64
    // lanes' fragments are 1 KB at ((c*27 + t)*G + g)*1024 (output channels
    // past Cout packed as zeros).
    const int G = (Cout + 31) / 32;
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(wpk, (uint32_t)((size_t)nch * kTaps * G * 1024));
    const int wlane = lane * 16;
    auto load_w = [&](int c, int tap, pv_bf16x8 (&wf)[NBW]) {
        const int cc = c < nch ? c : nch - 1;  // past the end: reload, never used
#pragma unroll
        for (int nb = 0; nb < NBW; nb++)
            wf[nb] = as_frag(bload16(wr, wlane,
                                     ((cc * kTaps + tap) * G + nt * NB + wc * NBW + nb) * 1024));
    };

    pv_f32x16 acc[4][NBW];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < NBW; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

    if (tid < NT) {  // channels past Cout take the last one's (never stored)
        float sc, sh;
        pv_bn_coeffs(bn, min(n0 + tid, Cout - 1), sc, sh);
        bn_tab[0][tid] = sc;
        bn_tab[1][tid] = sh;
    }
    // A sparse input (occ) whose halo holds no occupied voxel: every product
    // is zero, so the accumulators stay zero and the epilogue writes
    // act(BN(0)), the same bits as the full loop would. The reduction is also
    // the barrier before the epilogue reads bn_tab.
    bool live = true;
    if (occ) {
        bool any = false;
#pragma unroll
        for (int set = 0; set < kSets; set++) any |= goff[set] != kOOB;
        live = __syncthreads_or(any);
    }
    // SP: bit 10*tv + w of msk[mb][tu] is set when block mb's input row
    // (tu, tv) holds an occupied voxel at halo w; the block's fragment at tap
    // (tu, tv, tw) covers w = tw .. tw + 7 of four such rows.
    uint32_t msk[4][3];
    if constexpr (SP) {
#pragma unroll
        for (int mb = 0; mb < 4; mb++)
#pragma unroll
            for (int tu = 0; tu < 3; tu++) {
                uint32_t m = 0u;
#pragma unroll
                for (int tv = 0; tv < 3; tv++) {
                    uint32_t r = 0u;
#pragma unroll
                    for (int k = 0; k < 4; k++)
                        r |= occ_row[(blk_u(mb) + tu) * kHalo + blk_v(mb) * 4 + tv + k];
                    m |= r << (10 * tv);
                }
                msk[mb][tu] = __builtin_amdgcn_readfirstlane(m);
            }
    }
    if (live) {
        // Chunk 0's halo, the weights of the first kWD taps.
#pragma unroll
        for (int set = 0; set < kSets; set++) *(uint4*)(lds + loff[set]) = halo_load(set, 0);
        // Weights load kWD taps ahead through a ring of kWD + 1 sets (a
        // divisor of 27, so the ring realigns at every chunk). The 32-channel
        // tiles (one wave per SIMD, four MFMAs per tap) look further ahead,
        // and store each halo piece eight taps after its load (1.5-2 % on
        // the small grids' convolutions).
        constexpr int kWD = (!SB && NB == 1) ? 8 : 2, kWR = kWD + 1;
        static_assert(kTaps % kWR == 0, "the weight ring realigns at every chunk");
        pv_bf16x8 wf[kWR][NBW];
#pragma unroll
        for (int k = 0; k < kWD; k++) load_w(0, k, wf[k]);
        __syncthreads();

        // Chunk c sits in LDS buffer c%2: 27 taps, unrolled. Tap t computes with
        // weight set t%kWR while tap t+kWD's weights load, and with B fragments
        // bf[t%2] while tap t+1's are read from LDS into the other set. Piece
        // set s of the next chunk's halo is loaded at tap s into
        // hr[s%kHaloLag] and stored to the other LDS buffer at tap
        // s+kHaloLag. One loop body for every chunk keeps the accumulators in
        // the same registers throughout.
        constexpr int kHaloLag = (!SB && NB == 1) ? 8 : 4;
        for (int c = 0; c < nch; c++) {
            const int cur_off = (c & 1) * HB, nxt_off = HB - cur_off;
            // Next chunk's halo. Past the last chunk the double-buffered
            // variant reloads the last chunk into the idle buffer, and SB
            // loads out of range (zeros, no memory access) into it: with
            // unconditional loads the compiler's wait counts stay exact (with
            // a branch around them it must assume they were skipped, and each
            // tap's weight wait then also waits for the next tap's weights).
            // Element-wise loads (!VEC) keep the branch: unconditional, they
            // spill registers.
            const bool fetch = VEC || !SB || c + 1 < nch;
            const int cn = c + 1 < nch ? (c + 1) * kKC : (SB ? Cin : c * kKC);
            pv_bf16x8 bf[2][4];
            uint4 hr[kHaloLag];
#pragma unroll
            for (int mb = 0; mb < 4; mb++)
                bf[0][mb] = *(const pv_bf16x8*)(lds + frag_addr(mb, 0) + cur_off);
#pragma unroll
            for (int t = 0; t < kTaps; t++) {
                const int cur = t & 1, nxt = cur ^ 1;
                if (t + kWD < kTaps)
                    load_w(c, t + kWD, wf[(t + kWD) % kWR]);
                else
                    load_w(c + 1, t + kWD - kTaps, wf[(t + kWD) % kWR]);
                if (fetch && t >= kHaloLag && t < kSets + kHaloLag)
                    *(uint4*)(lds + loff[t - kHaloLag] + nxt_off) = hr[(t - kHaloLag) % kHaloLag];
                if (fetch && t < kSets) hr[t % kHaloLag] = halo_load(t, cn);
                if (t + 1 < kTaps) {
#pragma unroll
                    for (int mb = 0; mb < 4; mb++)
                        bf[nxt][mb] = *(const pv_bf16x8*)(lds + frag_addr(mb, t + 1) + cur_off);
                }
#pragma unroll
                for (int mb = 0; mb < 4; mb++) {
                    if constexpr (SP) {
                        // opaque here, so that the test stays a scalar shift,
                        // mask and branch inside the loop (hoisted, the 108
                        // tests of a chunk would not fit in scalar registers)
                        uint32_t mm = msk[mb][t / 9];
                        asm volatile("" : "+s"(mm));
                        if (((mm >> (10 * ((t / 3) % 3) + t % 3)) & 0xffu) == 0u) continue;
                    }
#pragma unroll
                    for (int nb = 0; nb < NBW; nb++)
                        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            wf[t % kWR][nb], bf[cur][mb], acc[mb][nb], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // chunk done: the next halo is complete and this buffer is free
            if constexpr (SB)
                pv_lds_barrier();  // LDS only: the weight prefetch stays in flight
            else
                __syncthreads();
        }
    }

    // Epilogue. Block (mb, nb) holds D[n][voxel]: lane has voxel column r32
    // of the block and output channels 8*j + 4*khalf + i (e = 4*j + i). The
    // tile is staged in LDS in passes of PW channels (256 bytes per voxel),
    // then each thread copies 16-byte pieces out, so every store instruction
    // writes whole contiguous rows.
    // The output type is a compile-time branch of the epilogue (one straight
    // copy per type), so that the per-element code carries no type tests.
    const float neg = act == PVCONV_ACT_LEAKY ? slope : (act == PVCONV_ACT_RELU ? 0.f : 1.f);
    auto epilogue = [&](auto out_type) {
        constexpr bool OBF = decltype(out_type)::value;
        constexpr int esz = OBF ? 2 : 4;
        constexpr int PW = SB ? (OBF ? (NT < 64 ? NT : 64) : (NT < 32 ? NT : 32))
                              : (OBF ? (NT < 128 ? NT : 128) : (NT < 64 ? NT : 64));
        constexpr int kRow = SB ? kStageRowSB : kStageRow;  // LDS bytes per staged voxel
        constexpr int pieces = PW * esz / 16;  // 16-byte pieces per voxel row
        const size_t yrow = (size_t)Cout * esz;
#pragma unroll
        for (int pass = 0; pass * PW < NT; pass++) {
#pragma unroll
            for (int nb = 0; nb < NBW; nb++) {
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const int nl = (wc * NBW + nb) * 32 + 8 * j + 4 * khalf;  // channel in the tile
                    if (nl < pass * PW || nl >= (pass + 1) * PW) continue;
                    const float4 sc = *(const float4*)&bn_tab[0][nl];
                    const float4 sh = *(const float4*)&bn_tab[1][nl];
                    const int cb = (nl - pass * PW) * esz;  // byte offset in the row
#pragma unroll
                    for (int mb = 0; mb < 4; mb++) {
                        const int vox = blk_u(mb) * 64 + (blk_v(mb) * 4 + (r32 >> 3)) * 8 +
                                        (r32 & 7);
                        float r[4] = {acc[mb][nb][4 * j + 0] * sc.x + sh.x,
                                      acc[mb][nb][4 * j + 1] * sc.y + sh.y,
                                      acc[mb][nb][4 * j + 2] * sc.z + sh.z,
                                      acc[mb][nb][4 * j + 3] * sc.w + sh.w};
#pragma unroll
                        for (int e = 0; e < 4; e++) r[e] = r[e] >= 0.f ? r[e] : r[e] * neg;
                        char* d = lds + vox * kRow + cb;
                        if constexpr (OBF)
                            *(uint2*)d = make_uint2(pv_pack_bf16x2(r[0], r[1]),
                                                    pv_pack_bf16x2(r[2], r[3]));
                        else
                            *(float4*)d = make_float4(r[0], r[1], r[2], r[3]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            pv_lds_barrier();
            // copy out: piece k of voxel vox (k < pieces); a pass partly past
            // Cout copies its first ncols channels (whole pieces, then the
            // elements of a last partial one)
            const size_t col = ((size_t)n0 + pass * PW) * esz;
            const int ncols = min(PW, Cout - n0 - pass * PW);
            if (ncols <= 0) continue;  // uniform: the whole pass lies past Cout
            const int vbytes = ncols * esz;
            if (ncols == PW && vec_out && u0 + kBrick <= R && v0 + kBrick <= R &&
                w0 + kBrick <= R) {
                // the whole brick inside the grid: batches of UC pieces per
                // thread, every LDS read of a batch issued before its stores
                constexpr int kIt = 512 * pieces / NTH, UC = kIt < 4 ? kIt : 4;
                static_assert(kIt % UC == 0, "copy-out batches divide the pieces");
#pragma unroll 1
                for (int i0 = 0; i0 < kIt; i0 += UC) {
                    uint4 val[UC];
#pragma unroll
                    for (int q = 0; q < UC; q++) {
                        const int i = tid + (i0 + q) * NTH, vox = i / pieces, k = i % pieces;
                        val[q] = *(const uint4*)(lds + vox * kRow + k * 16);
                    }
#pragma unroll
                    for (int q = 0; q < UC; q++) {
                        const int i = tid + (i0 + q) * NTH, vox = i / pieces, k = i % pieces;
                        const int u = u0 + (vox >> 6), v = v0 + ((vox >> 3) & 7),
                                  ww = w0 + (vox & 7);
                        *(uint4*)((char*)y + (cloud + ((size_t)u * R + v) * R + ww) * yrow + col +
                                  k * 16) = val[q];
                    }
                }
                pv_lds_barrier();
                continue;
            }
            for (int i = tid; i < 512 * pieces; i += NTH) {
                const int vox = i / pieces, k = i % pieces;
                const int u = u0 + (vox >> 6), v = v0 + ((vox >> 3) & 7), ww = w0 + (vox & 7);
                if (u >= R || v >= R || ww >= R || k * 16 >= vbytes) continue;
                const uint4 val = *(const uint4*)(lds + vox * kRow + k * 16);
                char* dst = (char*)y + (cloud + ((size_t)u * R + v) * R + ww) * yrow + col + k * 16;
                const int nel = min(16, vbytes - k * 16) / esz;  // elements of this piece
                if (vec_out && nel * esz == 16) {
                    *(uint4*)dst = val;
                } else {
                    const uint32_t q[4] = {val.x, val.y, val.z, val.w};
                    for (int e = 0; e < nel; e++) {
                        if constexpr (OBF)
                            ((uint16_t*)dst)[e] = (uint16_t)(q[e >> 1] >> ((e & 1) * 16));
                        else
                            ((uint32_t*)dst)[e] = q[e];
                    }
                }
            }
            pv_lds_barrier();
        }
    };
    if (out_bf16)
        epilogue(std::integral_constant<bool, true>{});
    else
        epilogue(std::integral_constant<bool, false>{});
}

// ---------------------------------------------------------------------------
// The convolutions inside a layer's forward compute only the rows (voxels)
// that matter. Their grids are internal: the first one's input is zero but for
// the occupied voxels, and the last one's output is read by the devoxelisation
// alone, at its points' corner cells, all within one voxel of an occupied
// voxel. So the last convolution computes the voxels read, and a first one
// before it D1, the voxels within one voxel of an occupied one: everywhere
// else its output is the constant act(BN(0)) that an empty neighbourhood
// gives. (Part-segmentation clouds at R = 32: 12 % and 18 % of the grid, at
// R = 16 24 % and 38 %.)
//
// pv_conv_plan_kernel, one workgroup per 8x8x8 brick, makes the bit maps of
// occupied and D1 voxels (one byte per eight w) and lists each brick's voxels
// for either convolution; pv_conv3d_rows_kernel multiplies blocks of 32 of
// them: a fragment read names a voxel per lane, so any 32 voxels of the brick
// make a block.
//
// The halo is compact: 32 bytes a voxel, 336 a row of ten, so that voxel
// (u, v, w) starts in 16-byte bank 2w + 2u + 5v (mod 16) plus a constant, under
// every tap. Sixteen lanes are served together: a list deals the voxels so
// that position p holds a voxel of bank class p mod 16 as far as the classes
// reach, and the reads do not conflict.
// ---------------------------------------------------------------------------
constexpr int kRowsRow = kHalo * 32 + 16;              // 336
constexpr int kRowsHalo = kHalo * kHalo * kRowsRow;    // 33600 per buffer
constexpr int kRowsMaxCin = 256;                       // the constant's table
constexpr int kListLen = 512;                          // entries per brick
constexpr uint16_t kNoVoxel = 0xffff;

// The D1 bits of row (ru, rv) of a brick from its halo's occupied bits.
__device__ __forceinline__ uint32_t d1_row(const uint32_t* s_occ, int ru, int rv) {
    uint32_t m = 0u;
#pragma unroll
    for (int du = 0; du < 3; du++)
#pragma unroll
        for (int dv = 0; dv < 3; dv++) m |= s_occ[(ru + du) * kHalo + rv + dv];
    return m | (m >> 1) | (m >> 2);
}

// Deals the voxels marked in `need` (row tid / 4 of the brick, of which this
// thread takes two) into s_row. deal_rank counts the bank classes into s_cls
// (zero on entry); after a barrier deal_place stores the voxels (s_row all
// kNoVoxel on entry) and returns the number of blocks of 32. A voxel's order
// within its class is that of the atomics and does not matter: each output's
// arithmetic is its own.
struct DealRank {
    int rank[2], cls[2];
};
__device__ __forceinline__ DealRank deal_rank(uint32_t need, int tid, int* s_cls) {
    const int ru = tid >> 5, rv = (tid >> 2) & 7, rw = (tid & 3) * 2;
    DealRank d;
#pragma unroll
    for (int i = 0; i < 2; i++) {
        d.cls[i] = (2 * (rw + i) + 2 * ru + 5 * rv) & 15;
        d.rank[i] = (need >> (rw + i)) & 1u ? atomicAdd(&s_cls[d.cls[i]], 1) : -1;
    }
    return d;
}
__device__ __forceinline__ int deal_place(const DealRank& d, int tid, const int* s_cls,
                                          uint16_t* s_row) {
    int total = 0;
#pragma unroll
    for (int c = 0; c < 16; c++) total += s_cls[c];
    const int P = (total + 15) >> 4;  // groups of sixteen
#pragma unroll
    for (int i = 0; i < 2; i++) {
        if (d.rank[i] < 0) continue;
        int pos = d.rank[i] * 16 + d.cls[i];
        if (d.rank[i] >= P) {
            // past the class's share: the places other classes leave
            int e = d.rank[i] - P;
            for (int c = 0; c < d.cls[i]; c++) e += max(s_cls[c] - P, 0);
            int c = 0;
            while (c < 15 && e >= max(P - s_cls[c], 0)) e -= max(P - s_cls[c++], 0);
            pos = (s_cls[c] + e) * 16 + c;
        }
        s_row[pos] = (uint16_t)((tid >> 2) * 8 + (tid & 3) * 2 + i);
    }
    return __builtin_amdgcn_readfirstlane((P + 1) >> 1);
}

// The occupied bits of a brick's halo rows, from the counts. Ends before the
// barrier that completes them; s_occ is zeroed here, behind a barrier.
__device__ __forceinline__ void halo_occupied(const int32_t* __restrict__ counts, size_t cloud,
                                              int R, int u0, int v0, int w0, int tid,
                                              uint32_t* s_occ) {
    int n[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int h = tid + i * 256;
        const int gu = u0 + h / (kHalo * kHalo) - 1, gv = v0 + (h / kHalo) % kHalo - 1,
                  gw = w0 + h % kHalo - 1;
        n[i] = 0;
        if (h < kHaloVox && gu >= 0 && gu < R && gv >= 0 && gv < R && gw >= 0 && gw < R)
            n[i] = counts[cloud + ((size_t)gu * R + gv) * R + gw];
    }
    if (tid < kHalo * kHalo) s_occ[tid] = 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int h = tid + i * 256;
        if (n[i] > 0) atomicOr(&s_occ[h / kHalo], 1u << (h % kHalo));
    }
}

// list[0]: D1; list[1]: the voxels read, which are those holding points
// (nearest), or the corner cells of the points at pn, or without pn D1. A list
// without a place is not made, nor are D1's bits.
__global__ __launch_bounds__(256) void pv_conv_plan_kernel(
    const int32_t* __restrict__ counts, const float* __restrict__ pn, int N, int nearest, int R,
    int nbr, PvConvPlan plan) {
    __shared__ uint32_t s_occ[kHalo * kHalo];  // halo rows
    __shared__ uint32_t s_read[kBrick * kBrick];
    constexpr int kPlanNear = 1024;
    __shared__ float s_near_p[kPlanNear][3];
    __shared__ int s_near;
    __shared__ __attribute__((aligned(16))) int s_cls[2][16];
    __shared__ uint16_t s_row[2][kListLen];
    const int tid = threadIdx.x;
    const int brick = blockIdx.x;
    int r = brick;
    const int bw = r % nbr;
    r /= nbr;
    const int bv = r % nbr;
    r /= nbr;
    const int bu = r % nbr;
    const int b = r / nbr;
    const int u0 = bu * kBrick, v0 = bv * kBrick, w0 = bw * kBrick;
    const size_t cloud = (size_t)b * R * R * R;
    if (tid < kBrick * kBrick) s_read[tid] = 0u;
    if (tid == 0) s_near = 0;
    if (tid < 32) s_cls[tid >> 4][tid & 15] = 0;
    ((uint32_t*)s_row)[tid] = 0xffffffffu;
    ((uint32_t*)s_row)[tid + 256] = 0xffffffffu;
    // The few points near the brick (most waves hold one) are gathered first,
    // so that the fp64 cells are formed once per 64 of them.
    const float* p = pn + (size_t)b * N * 3;
    const int lane = tid & 63;
    auto mark = [&](float x, float y, float z) {
        const PvAxis ax = pv_trilinear_axis(x, R), ay = pv_trilinear_axis(y, R),
                     az = pv_trilinear_axis(z, R);
        const int a0 = az.i0 - w0, a1 = az.i1 - w0;
        const uint32_t wbits = (a0 >= 0 && a0 < kBrick ? 1u << a0 : 0u) |
                               (a1 >= 0 && a1 < kBrick ? 1u << a1 : 0u);
        if (wbits == 0u) return;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const int u = (c & 2 ? ax.i1 : ax.i0) - u0, v = (c & 1 ? ay.i1 : ay.i0) - v0;
            if (u >= 0 && u < kBrick && v >= 0 && v < kBrick)
                atomicOr(&s_read[u * kBrick + v], wbits);
        }
    };
    // A thread has U points in flight: two runs of four (three 16-byte loads
    // each, where the cloud's rows allow), 1024 points apart.
    constexpr int U = 8;
    float q[U][3];
    const bool whole = ((uintptr_t)p & 15u) == 0 && (N & 3) == 0;
    auto point = [&](int j0, int i) { return j0 + (i >> 2) * 1024 + tid * 4 + (i & 3); };
    auto load_points = [&](int j0) {
#pragma unroll
        for (int h = 0; h < U / 4; h++) {
            const int j = point(j0, 4 * h);
            if (whole) {
                const float4* s = (const float4*)(p + (size_t)min(j, N - 4) * 3);
                const float4 a = s[0], c = s[1], e = s[2];
                const float v[12] = {a.x, a.y, a.z, a.w, c.x, c.y, c.z, c.w, e.x, e.y, e.z, e.w};
#pragma unroll
                for (int i = 0; i < 12; i++) q[4 * h + i / 3][i % 3] = v[i];
            } else {
#pragma unroll
                for (int i = 0; i < 12; i++)
                    q[4 * h + i / 3][i % 3] = p[(size_t)min(j + i / 3, N - 1) * 3 + i % 3];
            }
        }
    };
    auto gather_near = [&](int j0) {
        const float fR = (float)R;
        uint64_t close[U];
        int n = 0;
#pragma unroll
        for (int i = 0; i < U; i++) {
            // the exact cells lie within 1.5 of R x - 1/2, of R x within the
            // grid: the border cells take what lies beyond (0: NaN)
            auto inside = [&](float v) { return fminf(fmaxf(v * fR, 0.f), fR); };
            const float x = inside(q[i][0]), y = inside(q[i][1]), z = inside(q[i][2]);
            const bool far = x < u0 - 2 || x > u0 + kBrick + 2 || y < v0 - 2 ||
                             y > v0 + kBrick + 2 || z < w0 - 2 || z > w0 + kBrick + 2;
            close[i] = __ballot(!far && point(j0, i) < N);
            n += __popcll(close[i]);
        }
        if (n == 0) return;
        int at = 0;
        if (lane == 0) at = atomicAdd(&s_near, n);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int i = 0; i < U; i++) {
            if ((close[i] >> lane) & 1ull) {
                const int k = at + __popcll(close[i] & ((1ull << lane) - 1ull));
                if (k < kPlanNear) {
                    s_near_p[k][0] = q[i][0];
                    s_near_p[k][1] = q[i][1];
                    s_near_p[k][2] = q[i][2];
                } else {
                    mark(q[i][0], q[i][1], q[i][2]);  // no room
                }
            }
            at += __popcll(close[i]);
        }
    };
    if (pn) load_points(0);  // in flight beside the counts
    halo_occupied(counts, cloud, R, u0, v0, w0, tid, s_occ);
    __syncthreads();
    const int ru = tid >> 5, rv = (tid >> 2) & 7;
    const bool in_row = u0 + ru < R && v0 + rv < R;
    const uint32_t in_w = in_row ? (w0 + kBrick <= R ? 0xffu : (1u << (R - w0)) - 1u) : 0u;
    const uint32_t occ = (s_occ[(ru + 1) * kHalo + rv + 1] >> 1) & in_w;
    const uint32_t near = d1_row(s_occ, ru, rv) & in_w;
    if (in_row && (tid & 3) == 0) {
        const size_t at = (((size_t)b * R + u0 + ru) * R + v0 + rv) * nbr + bw;
        plan.occ[at] = (uint8_t)occ;
        if (plan.d1) plan.d1[at] = (uint8_t)near;
    }
    // no occupied voxel in or beside the brick: no point reads it
    if (!__syncthreads_or((int)near)) return;
    if (pn)
        for (int j0 = 0;;) {
            gather_near(j0);
            j0 += 256 * U;
            if (j0 >= N) break;
            load_points(j0);
        }
    if (pn) {
        __syncthreads();  // s_near's points
        for (int k = tid; k < min(s_near, kPlanNear); k += 256)
            mark(s_near_p[k][0], s_near_p[k][1], s_near_p[k][2]);
        __syncthreads();
    }
    const uint32_t need[2] = {near, nearest ? occ
                                            : (pn ? s_read[ru * kBrick + rv] & in_w : near)};
    DealRank d[2];
#pragma unroll
    for (int q = 0; q < 2; q++)
        if (plan.list[q]) d[q] = deal_rank(need[q], tid, s_cls[q]);
    __syncthreads();
    int blocks[2] = {0, 0};
#pragma unroll
    for (int q = 0; q < 2; q++)
        if (plan.list[q]) blocks[q] = deal_place(d[q], tid, s_cls[q], s_row[q]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; q++) {
        if (tid < blocks[q] * 16)  // 32 entries a block, two a thread
            ((uint32_t*)(plan.list[q] + (size_t)brick * kListLen))[tid] = ((uint32_t*)s_row[q])[tid];
        if (tid == q && blocks[q] > 0) {
            const int at = blocks[q] * kPvPlanSub + brick % kPvPlanSub;
            const int k = atomicAdd(&plan.count[q][at], 1);
            plan.order[q][(size_t)at * ((gridDim.x + kPvPlanSub - 1) / kPvPlanSub) + k] = brick;
        }
    }
}

// One convolution over the listed voxels; rows that are not listed are not
// written. A workgroup owns a brick and 32*NB channels. What bounded aligned
// blocks with every wave on all 64 channels was not the MFMAs but what a wave
// loads per tap: its weights, 1 KB per 32 channels, whatever the number of its
// voxels (55 k cycles of the vector cache, 64 B a cycle, against 27 k of MFMAs
// per live brick); and a wave of 32 channels reads a voxel fragment from LDS,
// 1 KB, for every MFMA, as much as LDS gives at the MFMAs' rate. So the waves
// are, by what the brick holds:
//  * NB = 4, four to eight blocks: two by two, 64 channels and half of the
//    blocks each; more than eight are two items;
//  * NB = 4, up to kAbreast blocks: four abreast, 32 channels and every block
//    each: half the weight loads;
//  * NB = 2: two by two, 32 channels and half of the blocks each;
//  * NB = 1 (small grids): four voxel groups.
// Workgroups take the bricks by falling number of blocks, from the plan's
// buckets: with bricks of 1 to 16 blocks in grid order, a tenth of the work ran
// on alone for a third of the time.
// SELF (counts given): the workgroup makes its brick's D1 list itself, and
// the first tile's stores it and D1's bits in `made` for the next convolution.
// For the grids and widths of rows_small, where the order is of little use and
// the plan's launch (5 to 6 us) costs more than it saves.
// Input modes: bits says which rows exist; the others are zero, or with KONST
// (the output of such a convolution, bits D1) the constant of its batch norm
// bn_in, or with dense exist too.
constexpr int kAbreast = 3;
// The order in which a NB = 4 convolution takes the bricks: by the blocks of
// their items. Entry i (4 bits): the brick's blocks - 1.
constexpr uint64_t kOrderHalved = 0x01234895ab6cd7efull;
constexpr uint64_t kOrderWhole = 0x0123456789abcdefull;

template <int NB, bool VEC, bool KONST, bool SELF>
__global__ __launch_bounds__(256, 2) void pv_conv3d_rows_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ wpk, PvBnFold bn,
    PvBnFold bn_in, float neg, uint16_t* __restrict__ y, int R, int Cin, int Cout, int nbr,
    int nblocks, int B, const uint8_t* __restrict__ bits, int dense,
    const uint16_t* __restrict__ list, const uint8_t* __restrict__ nlist,
    const int32_t* __restrict__ order, const int32_t* __restrict__ bucket,
    const int32_t* __restrict__ counts, PvConvPlan made) {
    static_assert(!SELF || (!KONST && NB == 1), "the first convolution of a small grid");
    constexpr int NT = NB * 32;
    __shared__ __attribute__((aligned(16))) char lds[2 * kRowsHalo];
    __shared__ __attribute__((aligned(16))) uint16_t s_const[KONST ? kRowsMaxCin : 8];
    __shared__ __attribute__((aligned(16))) float bn_tab[2][NT];
    __shared__ uint32_t s_bits[kHalo * kHalo];
    __shared__ __attribute__((aligned(16))) int s_cls[SELF ? 16 : 4];
    __shared__ uint16_t s_row[SELF ? kListLen : 2];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // --- this workgroup's brick and tile
    const int ntiles = (Cout + NT - 1) / NT;
    const int bricks = B * nbr * nbr * nbr;
    int brick, nt, blocks = 0, first = 0;  // `blocks` of the list from `first`
    if (SELF || !order) {
        // each XCD takes one contiguous eighth of every cloud
        int bid = blockIdx.x;
        const int per = nblocks / B;
        if ((per & 7) == 0) {
            const int xcd = bid & 7, k = bid >> 3, c = k / (per >> 3), j = k % (per >> 3);
            bid = c * per + ((xcd + c) & 7) * (per >> 3) + j;
        }
        nt = bid % ntiles;
        brick = bid / ntiles;
        if constexpr (!SELF) blocks = nlist[brick];
    } else {
        // lane l holds two buckets of one size: their bricks, items (a brick's
        // tiles, and its halves past eight blocks) and the items before them
        static_assert(kPvPlanSub == 8, "two of a size's eight buckets a lane");
        constexpr uint64_t sizes = NB == 4 ? kOrderHalved : kOrderWhole;
        const int size = (int)(sizes >> (4 * (lane >> 2)) & 15ull) + 1;
        const int2 c2 = *(const int2*)(bucket + size * kPvPlanSub + (lane & 3) * 2);
        const int each = NB == 4 && size > 8 ? 2 * ntiles : ntiles;
        const int items = (c2.x + c2.y) * each;
        int before = items;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(before, off, 64);
            if (lane >= off) before += o;
        }
        const uint64_t past = __ballot((int)blockIdx.x < before);
        if (past == 0ull) return;  // more workgroups than items
        const int l = __builtin_ctzll(past);
        const int T = __builtin_amdgcn_readlane(each, l);
        const int c0 = __builtin_amdgcn_readlane(c2.x, l);
        const int C = c0 + __builtin_amdgcn_readlane(c2.y, l);
        const int i = blockIdx.x - __builtin_amdgcn_readlane(before - items, l);
        // items of a brick 8 apart (on the same XCD) as far as groups of eight
        // bricks go
        int k, t;
        if (i < C / 8 * 8 * T) {
            k = i / (8 * T) * 8 + (i & 7);
            t = i % (8 * T) >> 3;
        } else {
            const int rest = C & 7, i1 = i - C / 8 * 8 * T;
            k = C / 8 * 8 + i1 % rest;
            t = i1 / rest;
        }
        blocks = __builtin_amdgcn_readlane(size, l);
        const int from = blocks * kPvPlanSub + (l & 3) * 2 + (k >= c0 ? 1 : 0);
        brick = order[(size_t)from * ((bricks + kPvPlanSub - 1) / kPvPlanSub) + k -
                      (k >= c0 ? c0 : 0)];
        nt = t % ntiles;
        if (NB == 4 && blocks > 8) {  // the first or the second half of the list
            const int half = (blocks + 1) / 2;
            first = t / ntiles * half;
            blocks = first ? blocks - half : half;
        }
    }
    int r = brick;
    const int bw = r % nbr;
    r /= nbr;
    const int bv = r % nbr;
    r /= nbr;
    const int bu = r % nbr;
    const int b = r / nbr;
    const int u0 = bu * kBrick, v0 = bv * kBrick, w0 = bw * kBrick, n0 = nt * NT;
    const size_t cloud = (size_t)b * R * R * R;
    const int nch = (Cin + kKC - 1) / kKC;

    // --- the halo's bits
    if constexpr (SELF) {
        if (tid < 16) s_cls[tid] = 0;
        ((uint32_t*)s_row)[tid] = 0xffffffffu;
        halo_occupied(counts, cloud, R, u0, v0, w0, tid, s_bits);
    } else if (tid < kHalo * kHalo) {
        const int gu = u0 + tid / kHalo - 1, gv = v0 + tid % kHalo - 1;
        uint32_t m = 0u;
        if (gu >= 0 && gu < R && gv >= 0 && gv < R) {
            const uint8_t* p = bits + (((size_t)b * R + gu) * R + gv) * nbr + bw;
            m = (uint32_t)p[0] << 1;
            if (bw > 0) m |= p[-1] >> 7;
            if (bw + 1 < nbr) m |= (uint32_t)(p[1] & 1u) << 9;
        }
        s_bits[tid] = m;
    }
    if constexpr (KONST)
        for (int c = tid; c < Cin; c += 256) {
            float sc, sh;
            pv_bn_coeffs(bn_in, c, sc, sh);
            const float k = 0.f * sc + sh;
            s_const[c] = pv_f32_to_bf16(k >= 0.f ? k : k * neg);
        }
    if (tid < NT) {  // channels past Cout take the last one's (never stored)
        float sc, sh;
        pv_bn_coeffs(bn, min(n0 + tid, Cout - 1), sc, sh);
        bn_tab[0][tid] = sc;
        bn_tab[1][tid] = sh;
    }
    __syncthreads();
    if constexpr (SELF) {
        const int ru = tid >> 5, rv = (tid >> 2) & 7;
        const bool in_row = u0 + ru < R && v0 + rv < R;
        const uint32_t in_w = in_row ? (w0 + kBrick <= R ? 0xffu : (1u << (R - w0)) - 1u) : 0u;
        const uint32_t near = d1_row(s_bits, ru, rv) & in_w;
        const bool store = made.d1 && nt == 0;
        if (store && in_row && (tid & 3) == 0)
            made.d1[(((size_t)b * R + u0 + ru) * R + v0 + rv) * nbr + bw] = (uint8_t)near;
        const DealRank d = deal_rank(near, tid, s_cls);
        __syncthreads();
        blocks = deal_place(d, tid, s_cls, s_row);
        __syncthreads();
        if (store) {
            if (tid == 0) made.n[brick] = (uint8_t)blocks;
            if (tid < blocks * 16)
                ((uint32_t*)(made.list[0] + (size_t)brick * kListLen))[tid] =
                    ((uint32_t*)s_row)[tid];
        }
    }
    blocks = __builtin_amdgcn_readfirstlane(blocks);  // uniform over the workgroup
    if (blocks == 0) return;

    // --- halo pieces of this thread: piece p = set*256 + tid is voxel p/2,
    // channels (p%2)*8 .. +7 of the chunk
    constexpr int kSets = (kPieces + 255) / 256;
    const int ulo = max(u0 - 1, 0), uhi = min(u0 + kBrick + 1, R);
    const size_t slab = (size_t)R * R * Cin;
    const __amdgpu_buffer_rsrc_t xr =
        make_rsrc(x + cloud * Cin + ulo * slab, (uint32_t)((uhi - ulo) * slab * 2));
    const int pq = tid & 1;
    auto piece_off = [&](int h, bool& konst) -> int {  // halo voxel h
        const int hr = h / kHalo, hw = h % kHalo;
        const int gu = u0 + hr / kHalo - 1, gv = v0 + hr % kHalo - 1, gw = w0 + hw - 1;
        const bool grid = gu >= 0 && gu < R && gv >= 0 && gv < R && gw >= 0 && gw < R;
        const bool bit = (s_bits[hr] >> hw) & 1u;
        konst = KONST && grid && !bit;
        return grid && (bit || (!KONST && dense))
                   ? ((((gu - ulo) * R + gv) * R + gw) * Cin + pq * 8) * 2 : kOOB;
    };
    int goff[kSets], loff[kSets];
    uint32_t konst = 0u;  // the sets that take the constant
#pragma unroll
    for (int set = 0; set < kSets; set++) {
        const int h = min(set * 128 + (tid >> 1), kHaloVox - 1);
        bool k;
        goff[set] = piece_off(h, k);
        konst |= (k ? 1u : 0u) << set;
        loff[set] = h / kHalo * kRowsRow + h % kHalo * 32 + pq * 16;
    }
    auto halo_load = [&](int off, int cc) -> uint4 {
        if (VEC) return bload16(xr, cc + pq * 8 < Cin ? off : kOOB, cc * 2);
        return bload8_elems(xr, off, cc * 2, Cin - cc - pq * 8);
    };
    auto halo_store = [&](int set, int buf, uint4 v, uint4 kv) {
        if constexpr (KONST) {
            const bool k = (konst >> set) & 1u;
            v.x = k ? kv.x : v.x;
            v.y = k ? kv.y : v.y;
            v.z = k ? kv.z : v.z;
            v.w = k ? kv.w : v.w;
        }
        *(uint4*)(lds + buf + loff[set]) = v;
    };
    auto const_of = [&](int cc) -> uint4 {
        if constexpr (KONST)
            if (cc + pq * 8 < Cin) return *(const uint4*)&s_const[cc + pq * 8];
        return make_uint4(0u, 0u, 0u, 0u);
    };
    {
        const uint4 kv = const_of(0);
#pragma unroll
        for (int set = 0; set < kSets; set++) halo_store(set, 0, halo_load(goff[set], 0), kv);
    }

    // --- this wave's channels and its share of the blocks: block k*vg + wg in
    // slot k
    const bool abreast = NB == 4 && blocks <= kAbreast;
    const int wc = abreast ? 4 : (NB > 1 ? 2 : 1);  // waves side by side
    const int vg = 4 / wc, wg = wave / wc;
    const int cl = wave % wc * (NT / wc);  // the first channel in the tile
    const int G = (Cout + 31) / 32;
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(wpk, (uint32_t)((size_t)nch * kTaps * G * 1024));
    const int wlane = lane * 16, wgrp = (n0 + cl) / 32;
    const int r32 = lane & 31, khalf = lane >> 5;
    const uint16_t* mylist =
        (SELF ? s_row : list + (size_t)brick * kListLen) + (first + wg) * 32 + r32;
    auto run = [&](auto count, auto width) {
        constexpr int n = decltype(count)::value, W = decltype(width)::value;
        // Fragments are read two taps ahead where few MFMAs pass in a tap
        // (an LDS read takes about as long as four of them).
        constexpr int kWD = n * W > 4 ? 2 : 8, kWR = kWD + 1, kHaloLag = 4,
                      kBD = n * W > 4 ? 1 : 2, kBR = kBD + 1;
        static_assert(kTaps % kWR == 0, "the weight ring realigns at every chunk");
        constexpr int nr = n > 0 ? n : 1;
        int vox[nr], base[nr];
#pragma unroll
        for (int k = 0; k < n; k++) vox[k] = k * vg + wg < blocks ? mylist[k * vg * 32] : kNoVoxel;
        pv_bf16x8 wf[kWR][W];
        auto load_w = [&](int c, int tap, pv_bf16x8 (&f)[W]) {
            const int cc = c < nch ? c : nch - 1;  // past the end: reload, never used
#pragma unroll
            for (int j = 0; j < W; j++)
                f[j] = as_frag(bload16(wr, wlane, ((cc * kTaps + tap) * G + wgrp + j) * 1024));
        };
        if (n > 0) {
#pragma unroll
            for (int k = 0; k < kWD; k++) load_w(0, k, wf[k]);
        }
#pragma unroll
        for (int k = 0; k < n; k++) {
            const int v = vox[k] & 511;  // none: any voxel
            base[k] = ((v >> 6) * kHalo + ((v >> 3) & 7)) * kRowsRow + (v & 7) * 32 + khalf * 16;
        }
        pv_f32x16 acc[nr][W];
#pragma unroll
        for (int i = 0; i < n; i++)
#pragma unroll
            for (int j = 0; j < W; j++)
#pragma unroll
                for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
        __syncthreads();  // chunk 0's halo is stored
        for (int c = 0; c < nch; c++) {
            const int cur_off = (c & 1) * kRowsHalo, nxt_off = kRowsHalo - cur_off;
            // past the last chunk the next halo loads out of range (zeros):
            // unconditional loads keep the wait counts exact. Element-wise
            // loads (!VEC: few input channels) follow the taps instead, for
            // their registers.
            const int cn = c + 1 < nch ? (c + 1) * kKC : Cin;
            const uint4 kv = const_of(cn);
            pv_bf16x8 bf[kBR][nr];
            uint4 hr[kHaloLag];
            auto read_b = [&](int tn) {
                const int off = ((tn / 9) * kHalo + (tn / 3) % 3) * kRowsRow + (tn % 3) * 32;
#pragma unroll
                for (int k = 0; k < n; k++)
                    bf[tn % kBR][k] = *(const pv_bf16x8*)(lds + base[k] + off + cur_off);
            };
#pragma unroll
            for (int t = 0; t < kBD; t++) read_b(t);
#pragma unroll
            for (int t = 0; t < kTaps; t++) {
                if (n > 0) {
                    if (t + kWD < kTaps) load_w(c, t + kWD, wf[(t + kWD) % kWR]);
                    else load_w(c + 1, t + kWD - kTaps, wf[(t + kWD) % kWR]);
                }
                if (VEC && t >= kHaloLag && t < kSets + kHaloLag)
                    halo_store(t - kHaloLag, nxt_off, hr[(t - kHaloLag) % kHaloLag], kv);
                if (VEC && t < kSets) hr[t % kHaloLag] = halo_load(goff[t], cn);
                if (t + kBD < kTaps) read_b(t + kBD);
#pragma unroll
                for (int k = 0; k < n; k++)
#pragma unroll
                    for (int j = 0; j < W; j++)
                        acc[k][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            wf[t % kWR][j], bf[t % kBR][k], acc[k][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!VEC && c + 1 < nch) {
#pragma unroll 1
                for (int p = tid; p < kPieces; p += 256) {
                    bool k;
                    const int h = p >> 1, off = piece_off(h, k);
                    *(uint4*)(lds + nxt_off + h / kHalo * kRowsRow + h % kHalo * 32 + pq * 16) =
                        halo_load(off, cn);
                }
            }
            pv_lds_barrier();  // LDS only: the weight prefetch stays in flight
        }
        // lane l holds voxel l % 32 of a block and channels 8j + 4 (l / 32) + i
#pragma unroll
        for (int k = 0; k < n; k++) {
            const int v = vox[k];
            if (v >= kListLen) continue;
            uint16_t* row = y + (cloud + ((size_t)(u0 + (v >> 6)) * R + v0 + ((v >> 3) & 7)) * R +
                                 w0 + (v & 7)) * Cout;
#pragma unroll
            for (int w = 0; w < W; w++)
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const int nl = cl + 32 * w + 8 * j + 4 * khalf;
                    if (n0 + nl >= Cout) continue;
                    const float4 sc = *(const float4*)&bn_tab[0][nl];
                    const float4 sh = *(const float4*)&bn_tab[1][nl];
                    float q[4] = {acc[k][w][4 * j + 0] * sc.x + sh.x,
                                  acc[k][w][4 * j + 1] * sc.y + sh.y,
                                  acc[k][w][4 * j + 2] * sc.z + sh.z,
                                  acc[k][w][4 * j + 3] * sc.w + sh.w};
#pragma unroll
                    for (int e = 0; e < 4; e++) q[e] = q[e] >= 0.f ? q[e] : q[e] * neg;
                    *(uint2*)(row + n0 + nl) =
                        make_uint2(pv_pack_bf16x2(q[0], q[1]), pv_pack_bf16x2(q[2], q[3]));
                }
        }
    };
    // one straight loop for each number of blocks
#define PV_RUN(N_, W_) run(std::integral_constant<int, N_>{}, std::integral_constant<int, W_>{})
    const int mine = (blocks - wg + vg - 1) / vg;
    if constexpr (NB == 4) {
        if (abreast) {
            if (mine == 1) PV_RUN(1, 1);
            else if (mine == 2) PV_RUN(2, 1);
            else PV_RUN(3, 1);
        } else {
            if (mine <= 2) PV_RUN(2, 2);
            else if (mine == 3) PV_RUN(3, 2);
            else PV_RUN(4, 2);
        }
    } else {
        switch (mine) {
            case 0: PV_RUN(0, 1); break;
            case 1: PV_RUN(1, 1); break;
            case 2: PV_RUN(2, 1); break;
            case 3: PV_RUN(3, 1); break;
            case 4: PV_RUN(4, 1); break;
            case 5:
            case 6: if constexpr (NB == 2) PV_RUN(6, 1); break;
            default: if constexpr (NB == 2) PV_RUN(8, 1);
        }
    }
#undef PV_RUN
}

// Repack bf16 weights [Cout][27][Cin] into the fragment order the MFMA conv
// reads: 16-byte element ((c*27 + t)*G + g)*64 + lane holds the 8 channels
// k = c*16 + (lane/32)*8 .. +7 of output channel g*32 + lane%32 at tap t
// (zero past Cin and past Cout), G = ceil(Cout/32). One thread per element;
// one launch packs the
// weights of all the convolutions of a layer (the blocks of job q follow those of
// jobs 0 .. q-1).
static_assert(kKC == kPvPackKC && kTaps == kPvPackTaps, "the packing matches the kernel");

__global__ __launch_bounds__(256) void pv_pack_conv_weights_kernel(PvPackJobs jobs) {
    pv_pack_role(jobs, blockIdx.x);
}

// fp32 path: four consecutive lanes per output (voxel, channel), each
// summing the taps tap = part, part + 4, ... over all input channels (16
// bytes at a time when the rows allow), then a 4-lane sum.
template <bool V4>
__global__ __launch_bounds__(256) void pv_conv3d_f32_kernel(const float* __restrict__ x,
                                                            const float* __restrict__ w,
                                                            PvBnFold bn, int act, float slope,
                                                            void* __restrict__ y, int out_bf16,
                                                            int B, int R, int Cin, int Cout) {
    const size_t V = (size_t)R * R * R;
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t i = t >> 2;  // output element
    const int part = (int)(t & 3);
    const bool live = i < (size_t)B * V * Cout;
    const size_t ic = live ? i : 0;  // dead lanes still join the 4-lane sum
    const int o = (int)(ic % Cout);
    const size_t vox = ic / Cout;
    const size_t b = vox / V;
    const int r = (int)(vox % V);
    const int u = r / (R * R), v = (r / R) % R, ww = r % R;
    float s = 0.f;
    if (live) {
        for (int tap = part; tap < 27; tap += 4) {
            const int nu = u + tap / 9 - 1, nv = v + (tap / 3) % 3 - 1, nw = ww + tap % 3 - 1;
            if (nu < 0 || nu >= R || nv < 0 || nv >= R || nw < 0 || nw >= R) continue;
            const float* xi = x + (b * V + ((size_t)nu * R + nv) * R + nw) * Cin;
            const float* wk = w + ((size_t)o * 27 + tap) * Cin;
            if (V4) {
                for (int c = 0; c < Cin; c += 4) {
                    const float4 a = *(const float4*)(xi + c), q = *(const float4*)(wk + c);
                    s += q.x * a.x;
                    s += q.y * a.y;
                    s += q.z * a.z;
                    s += q.w * a.w;
                }
            } else {
                for (int c = 0; c < Cin; c++) s += wk[c] * xi[c];
            }
        }
    }
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    if (!live || part != 0) return;
    float scale, shift;
    pv_bn_coeffs(bn, o, scale, shift);
    const float val = pv_activate(s * scale + shift, act, slope);
    if (out_bf16)
        ((uint16_t*)y)[i] = pv_f32_to_bf16(val);
    else
        ((float*)y)[i] = val;
}

// y = act(BN(sum of the ksplit partial sums)), the partials added in split
// order. Four channels per thread (C_out % 4 == 0 and 16-byte aligned rows),
// else one.
template <bool V4>
__global__ __launch_bounds__(256) void pv_conv_split_reduce_kernel(
    const float* __restrict__ part, int ksplit, size_t n, int Cout, PvBnFold bn, int act,
    float slope, void* __restrict__ y, int out_bf16) {
    const size_t i0 = ((size_t)blockIdx.x * 256 + threadIdx.x) * (V4 ? 4 : 1);
    if (i0 >= n) return;
    const int c0 = (int)(i0 % Cout);
    float v[V4 ? 4 : 1];
    if constexpr (V4) {
        float4 a = *(const float4*)(part + i0);
        for (int s = 1; s < ksplit; s++) {
            const float4 b = *(const float4*)(part + (size_t)s * n + i0);
            a.x += b.x;
            a.y += b.y;
            a.z += b.z;
            a.w += b.w;
        }
        v[0] = a.x;
        v[1] = a.y;
        v[2] = a.z;
        v[3] = a.w;
    } else {
        float a = part[i0];
        for (int s = 1; s < ksplit; s++) a += part[(size_t)s * n + i0];
        v[0] = a;
    }
#pragma unroll
    for (int e = 0; e < (V4 ? 4 : 1); e++) {
        float sc, sh;
        pv_bn_coeffs(bn, c0 + e, sc, sh);
        v[e] = pv_activate(v[e] * sc + sh, act, slope);
    }
    if (out_bf16) {
        uint16_t* o = (uint16_t*)y + i0;
        if constexpr (V4)
            *(uint2*)o = make_uint2(pv_pack_bf16x2(v[0], v[1]), pv_pack_bf16x2(v[2], v[3]));
        else
            o[0] = pv_f32_to_bf16(v[0]);
    } else {
        float* o = (float*)y + i0;
        if constexpr (V4)
            *(float4*)o = make_float4(v[0], v[1], v[2], v[3]);
        else
            o[0] = v[0];
    }
}

template <int NB, int WCH, bool SB = false>
void launch_bf16(const void* x, int B, int R, int Cin, int Cout, const void* w,
                 const PvBnFold& bn, int act, float slope, void* y, bool out_bf16, bool vec,
                 hipStream_t s, int ksplit = 1, int cps = 0, const int32_t* occ = nullptr) {
    const int nbr = (R + kBrick - 1) / kBrick;
    const size_t blocks =
        (size_t)B * nbr * nbr * nbr * ((Cout + NB * 32 - 1) / (NB * 32)) * ksplit;
    // 16-byte stores: aligned output with rows of whole 16-byte pieces
    const bool vec_out = pv_aligned16(y) && ((size_t)Cout * (out_bf16 ? 2 : 4)) % 16 == 0;
#define PV_CONV(V, SPX)                                                                     \
    hipLaunchKernelGGL((pv_conv3d_bf16_kernel<NB, WCH, V, SB, SPX>), dim3((unsigned)blocks),   \
                       dim3(256 * WCH), 0, s, (const uint16_t*)x, (const uint16_t*)w, bn, act, \
                       slope, y, (int)out_bf16, (int)vec_out, R, Cin, Cout, nbr, (int)blocks, \
                       Cin, ksplit, cps, B, occ)
    // a sparse input on the two-per-CU form skips its empty fragments' MFMAs
    if (vec && SB && occ)
        PV_CONV(true, SB);
    else if (vec)
        PV_CONV(true, false);
    else
        PV_CONV(false, false);
#undef PV_CONV
}

template <int NB>
void launch_rows(const PvConvRows& c, const PvBnFold& bn, float neg, bool vec, hipStream_t s) {
    constexpr bool SMALL = NB == 1;
    const int nbr = (c.R + kBrick - 1) / kBrick;
    int blocks = c.B * nbr * nbr * nbr * ((c.Cout + NB * 32 - 1) / (NB * 32));
    if (NB == 4) blocks *= 2;  // halves of bricks with more than eight blocks
#define PV_ROWS_CONV(V, K, SELFX)                                                             \
    hipLaunchKernelGGL((pv_conv3d_rows_kernel<NB, V, K, SELFX>), dim3(blocks), dim3(256), 0, s,  \
                       (const uint16_t*)c.x, (const uint16_t*)c.packed, bn, c.bn_in, neg,        \
                       (uint16_t*)c.y, c.R, c.Cin, c.Cout, nbr, blocks, c.B,                     \
                       c.input == PvConvRows::kRowsOfFirst ? c.plan.d1 : c.plan.occ,             \
                       (int)(c.input == PvConvRows::kWhole), c.plan.list[c.which],               \
                       c.plan.n, SMALL ? nullptr : c.plan.order[c.which],                        \
                       c.plan.count[c.which], c.counts, made)
    PvConvPlan made{};
    if (c.input == PvConvRows::kRowsOfFirst) {
        PV_ROWS_CONV(true, true, false);
    } else if constexpr (SMALL) {
        if (c.which == 0) made = c.plan;
        if (vec)
            PV_ROWS_CONV(true, false, true);
        else
            PV_ROWS_CONV(false, false, true);
    } else if (vec) {
        PV_ROWS_CONV(true, false, false);
    } else {
        PV_ROWS_CONV(false, false, false);
    }
#undef PV_ROWS_CONV
}

// No plan, 32-channel tiles:
//  * grids of fewer than 512 tiles of 64 channels (two a CU), whose workgroups
//    are about all resident at once;
//  * widths that are no multiple of 64, on grids of any size. Their workgroups
//    are not all resident on large grids, every tile lists its brick again,
//    and the last convolution computes D1; but a plan with 32-channel tiles
//    gains only from three tiles a brick on (us a layer of two convolutions,
//    this form, the plan's and the complete grid, 16 clouds of 2048 points at
//    R = 32: 16 -> 16 66, 73, 99; 24 -> 24 77, 80, 117; 32 -> 32 80, 82, 115; 24
//    -> 40 107, 104, 211; 48 -> 48 119, 115, 234; 96 -> 96 225, 197, 491; 64
//    clouds: 32 -> 32 233, 230, 393; 32 -> 96 628, 544, 1564). With 96 channels
//    and more on large grids this form gives away an eighth.
bool rows_small(int B, int R, int Cout) {
    const int nbr = (R + kBrick - 1) / kBrick;
    return Cout % 64 != 0 || (long)B * nbr * nbr * nbr * (Cout / 64) < 512;
}

}  // namespace

size_t pv_conv3d_ws_bytes(int Cin, int Cout, bool bf16) {
    if (!bf16) return 0;
    const size_t nch = (size_t)(Cin + kKC - 1) / kKC;
    return nch * kKC * kTaps * (size_t)((Cout + 31) / 32 * 32) * 2;  // Cout padded to 32
}

void pv_pack_job(PvPackJobs& jobs, const void* w, int Cin, int Cout, void* packed) {
    PvPackJob& J = jobs.job[jobs.n++];
    J.w = (const uint16_t*)w;
    J.packed = (uint4*)packed;
    J.Cin = Cin;
    J.Cout = Cout;
    J.total = (int)(pv_conv3d_ws_bytes(Cin, Cout, true) / 16);
    J.vec = (int)(Cin % 8 == 0 && pv_aligned16(w));
    J.blocks = (J.total + 255) / 256;
}

void pv_launch_pack_conv_weights(const PvPackJobs& jobs, hipStream_t s) {
    const int blocks = pv_pack_blocks(jobs);
    if (blocks > 0)
        hipLaunchKernelGGL(pv_pack_conv_weights_kernel, dim3(blocks), dim3(256), 0, s, jobs);
}

int pv_conv3d_splits(int B, int R, int Cin, int Cout) {
    // Grids so small that the unsplit launch (32-channel tiles) leaves most
    // CUs idle, fewer than 64 workgroups (PVCNN++'s R = 8 level: 16), divide
    // the input channels among more workgroups of the two-per-CU variant.
    // At 64 and more (the R = 16 blocks) the split's extra prologues, fp32
    // partials and reduction cost more than the occupancy gains (measured).
    const int nbr = (R + kBrick - 1) / kBrick;
    const long bricks = (long)B * nbr * nbr * nbr;
    const long tiles = bricks * (Cout / 64);
    const int nch = (Cin + kKC - 1) / kKC;
    if (Cout % 64 != 0 || Cin % kKC != 0 || bricks * ((Cout + 31) / 32) >= 64 || nch < 2 ||
        tiles == 0)
        return 1;
    const int want = (int)((512 + tiles - 1) / tiles);
    const int cps = (nch + std::min(want, nch) - 1) / std::min(want, nch);
    return (nch + cps - 1) / cps;
}

size_t pv_conv3d_split_ws_bytes(int B, int R, int Cin, int Cout) {
    const int S = pv_conv3d_splits(B, R, Cin, Cout);
    return S > 1 ? (size_t)S * B * R * R * R * Cout * 4 : 0;
}

pvconv_status pv_launch_conv3d(const void* x, int B, int R, int Cin, int Cout, const void* w,
                               const PvBnFold& bn, int act, float slope, bool bf16, void* y,
                               bool out_bf16, void* ws, hipStream_t s, bool packed,
                               float* split_ws, const int32_t* occ) {
    if (B == 0) return PVCONV_OK;
    if (bf16) {
        if (!packed) {
            PvPackJobs jobs{};
            pv_pack_job(jobs, w, Cin, Cout, ws);
            pv_launch_pack_conv_weights(jobs, s);
        }
        w = ws;
        const bool vec = (Cin % 8 == 0) && pv_aligned16(x);
        const int S = split_ws ? pv_conv3d_splits(B, R, Cin, Cout) : 1;
        if (S > 1) {
            // fp32 partial sums per split (identity fold, no activation),
            // then their fixed-order sum with the batch norm and activation
            const int nch = (Cin + kKC - 1) / kKC, cps = (nch + S - 1) / S;
            launch_bf16<2, 1, true>(x, B, R, Cin, Cout, w, PvBnFold{}, PVCONV_ACT_NONE, 0.f,
                                    split_ws, false, vec, s, S, cps, occ);
            const size_t n = (size_t)B * R * R * R * Cout;
            const bool v4 = Cout % 4 == 0 && pv_aligned16(y) && pv_aligned16(split_ws);
            const size_t threads = v4 ? n / 4 : n;
            const unsigned blocks = (unsigned)((threads + 255) / 256);
            if (v4)
                hipLaunchKernelGGL(pv_conv_split_reduce_kernel<true>, dim3(blocks), dim3(256), 0,
                                   s, split_ws, S, n, Cout, bn, act, slope, y, (int)out_bf16);
            else
                hipLaunchKernelGGL(pv_conv_split_reduce_kernel<false>, dim3(blocks), dim3(256),
                                   0, s, split_ws, S, n, Cout, bn, act, slope, y, (int)out_bf16);
            return pv_launch_status();
        }
        // Channel tile: the widest (most reuse of each halo) that still gives
        // about one workgroup per CU; small grids (R = 16) take narrow tiles.
        const int nbr = (R + kBrick - 1) / kBrick;
        const long bricks = (long)B * nbr * nbr * nbr;
        // Inputs of up to 128 channels with enough tiles for two workgroups
        // per CU: 64-channel tiles with compact halos, two per CU (one's
        // prologue and epilogue overlap the other's MFMAs: 11 % faster at
        // 64->128 and 64->64, 2.5 % at 128->128, than one 128-channel
        // workgroup per CU). Otherwise 64-channel tiles, one workgroup per
        // CU: eight waves (two channel groups) for narrow inputs, four for
        // wide ones (a 128-channel tile of four waves would hold all 256
        // accumulator registers and spill in its epilogue).
        const bool two = Cin <= 64;
        if (Cin <= 128 && Cout % 64 == 0 && bricks * (Cout / 64) >= 512) {
            launch_bf16<2, 1, true>(x, B, R, Cin, Cout, w, bn, act, slope, y, out_bf16, vec, s, 1, 0, occ);
        } else if (Cout % 64 == 0 && bricks * (Cout / 64) >= 256) {
            if (two)
                launch_bf16<2, 2>(x, B, R, Cin, Cout, w, bn, act, slope, y, out_bf16, vec, s, 1, 0, occ);
            else
                launch_bf16<2, 1>(x, B, R, Cin, Cout, w, bn, act, slope, y, out_bf16, vec, s, 1, 0, occ);
        } else {
            launch_bf16<1, 1>(x, B, R, Cin, Cout, w, bn, act, slope, y, out_bf16, vec, s, 1, 0, occ);
        }
    } else {
        const size_t total = (size_t)B * R * R * R * Cout;
        const unsigned blocks = (unsigned)((4 * total + 255) / 256);
        if (Cin % 4 == 0 && pv_aligned16(x) && pv_aligned16(w))
            hipLaunchKernelGGL(pv_conv3d_f32_kernel<true>, dim3(blocks), dim3(256), 0, s,
                               (const float*)x, (const float*)w, bn, act, slope, y, (int)out_bf16,
                               B, R, Cin, Cout);
        else
            hipLaunchKernelGGL(pv_conv3d_f32_kernel<false>, dim3(blocks), dim3(256), 0, s,
                               (const float*)x, (const float*)w, bn, act, slope, y, (int)out_bf16,
                               B, R, Cin, Cout);
    }
    return pv_launch_status();
}

bool pv_conv3d_rows_ok(int B, int N, int R, int Cin, int Cout, int n_convs) {
    // Grids so small that the dense convolution splits its input channels
    // keep that form, and with three or more convolutions, where only the last
    // one is listed, so do all that rows_small names (B = 1, R = 37, 32
    // channels: 99 us dense, 102 listed; the list costs more than it saves. Not
    // so on large grids of widths that are no multiple of 64, whose form
    // without a plan is then not used either: 16 clouds of 2048 points at R =
    // 32, 32 -> 32 156 us dense, 150 with a plan, 32 -> 96 629, 489).
    if (n_convs > 2 && rows_small(B, R, Cout)) return false;
    // Clouds of one whole brick with a CU for every workgroup keep the complete
    // form: most voxels of eight a side are near a point, the workgroups take
    // as long as the fullest brick, and listing adds to that (us a layer,
    // complete and listed: 40 clouds of 256 points, 64 -> 128 twice, 61.6 and
    // 65.7; 64 of 64, 64 -> 64 twice, 49.8 and 53.4; but 80 of 256, 64 -> 128
    // twice, 320 workgroups, 107 and 97; 40 of 256 at R = 7 62.2 and 59.6, at R
    // = 8 16 -> 16 41.2 and 40.1).
    if (R == kBrick && Cout > 16 && (long)B * ((Cout + 31) / 32) <= 256) return false;
    // More channels than the table of constants holds, which only a second
    // convolution reads: a single one of 512 tiles and more, from clouds whose
    // grids stay sparse (us a layer, complete and listed: 16 clouds of 2048
    // points, R = 32, 64 -> 512 481 and 214; 128 of 4096, R = 8, 64 -> 320 614
    // and 608; but one of 65536, R = 32, 64 -> 512 178 and 276).
    if (Cout > kRowsMaxCin &&
        (n_convs > 1 || rows_small(B, R, Cout) || !pv_voxelize_sparse_ok(N)))
        return false;
    return Cout % 8 == 0 && pv_conv3d_splits(B, R, Cin, Cout) == 1 &&
           (n_convs < 2 || pv_conv3d_splits(B, R, Cout, Cout) == 1);
}

PvConvPlan pv_conv_plan_carve(void* base, int B, int R, int n_convs, size_t* bytes) {
    const int nbr = (R + kBrick - 1) / kBrick;
    const size_t bricks = (size_t)B * nbr * nbr * nbr;
    size_t off = 0;
    auto take = [&](size_t n) {
        char* q = (char*)base + off;
        off += pv_align256(n);
        return q;
    };
    PvConvPlan plan{};
    plan.count[0] = (int32_t*)take(kPvPlanCounts * sizeof(int32_t));
    plan.count[1] = plan.count[0] + kPvPlanCounts / 2;
    plan.occ = (uint8_t*)take((size_t)B * R * R * nbr);
    if (n_convs == 2) {
        plan.d1 = (uint8_t*)take((size_t)B * R * R * nbr);
        plan.n = (uint8_t*)take(bricks);
    }
    for (int q = n_convs == 2 ? 0 : 1; q < 2; q++) {
        plan.list[q] = (uint16_t*)take(bricks * kListLen * sizeof(uint16_t));
        plan.order[q] = (int32_t*)take(17 * kPvPlanSub *
                                       ((bricks + kPvPlanSub - 1) / kPvPlanSub) * sizeof(int32_t));
    }
    *bytes = off;
    return plan;
}

pvconv_status pv_launch_conv_plan(PvConvPlan& plan, const int32_t* counts, const float* pn,
                                  bool nearest, int B, int N, int R, int Cin, int Cout,
                                  hipStream_t s) {
    const int nbr = (R + kBrick - 1) / kBrick;
    const int nb3 = nbr * nbr * nbr;
    // Every brick's workgroup reads its cloud's points, 2048 a turn of 2.5 us:
    // 2.1 M of them (16 clouds of 2048 points, 64 bricks each) cost 9 of the
    // plan's 14.5 us and save a third of the last convolution's MFMAs. Past
    // four times that, on small grids, and where the convolution has few
    // channels for the points (Cin x Cout below 2 N), the last convolution
    // computes D1 (us a layer, the voxels read and D1, Cin x Cout / N in
    // brackets: 8 clouds of 16384 points, 64 -> 64 twice, R = 32 [0.25] 187 and
    // 156; 4 of 16384, 64 -> 128 once [0.5] 141 and 115; 8 of 8192, 64 -> 128
    // once [1] 133 and 125; 16 of 5000, 64 -> 128 once [1.6] 161 and 158; 64 of
    // 2048, 64 -> 64 twice [2] 332 and 348; 16 of 2048, 64 -> 128 twice [8] 181
    // and 196, 64 -> 256 twice [32] 411 and 504).
    const bool small = rows_small(B, R, Cout);
    if (nearest || (long long)B * nb3 * N > (8ll << 20) || (long long)Cin * Cout < 2ll * N)
        pn = nullptr;
    const bool one = plan.list[0] && (small || (!nearest && !pn));  // the same list for both
    if (one) plan.list[1] = nullptr;
    if (!small)
        hipLaunchKernelGGL(pv_conv_plan_kernel, dim3(B * nb3), dim3(256), 0, s, counts, pn, N,
                           (int)nearest, R, nbr, plan);
    if (one) {
        plan.list[1] = plan.list[0];
        plan.order[1] = plan.order[0];
        plan.count[1] = plan.count[0];
    }
    return pv_launch_status();
}

pvconv_status pv_launch_conv3d_rows(const PvConvRows& c, const PvBnFold& bn, int act, float slope,
                                    hipStream_t s) {
    const float neg = act == PVCONV_ACT_LEAKY ? slope : (act == PVCONV_ACT_RELU ? 0.f : 1.f);
    const bool vec = c.Cin % 8 == 0 && pv_aligned16(c.x);
    const int nbr = (c.R + kBrick - 1) / kBrick;
    const long bricks = (long)c.B * nbr * nbr * nbr;
    if (rows_small(c.B, c.R, c.Cout))
        launch_rows<1>(c, bn, neg, vec, s);
    else if (c.Cout % 128 == 0 && bricks >= 512)
        // about half of the bricks are live: 128 channels an item need twice
        // the CUs in bricks
        launch_rows<4>(c, bn, neg, vec, s);
    else
        launch_rows<2>(c, bn, neg, vec, s);
    return pv_launch_status();
}
