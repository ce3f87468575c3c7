// GEMM kernels: C[i][j] = sum_k A[i][k] * B[j][k] with A and B both stored
// row-major with K contiguous ("A times B transposed"), optionally batched.
//
// The result never goes to memory as a plain matrix: an epilogue functor
// receives each lane's output as four consecutive i for one j,
//     p = epi.pre(i0, j, z); epi(i0, j, z, v0, v1, v2, v3, p)
// (rows i0..i0+3 of batch z, column j; pre() issues the loads first),
// and stores it in whatever layout the consumer wants (bias, GELU, residual
// add, per-head or transposed cache layouts). Call sites pick which operand
// is A so that the four consecutive i are the contiguous output dimension.
//
// gemm_bf16: bf16 inputs, v_mfma_f32_16x16x32_bf16 with fp32 accumulation,
//   K tiles streamed into LDS with direct global->LDS loads (no staging
//   registers), 16-byte chunks XOR-swizzled against bank conflicts. Tiles of
//   256x256 (8 waves of 128x64 in two alternating groups, one workgroup per
//   CU), 256x128 (8 waves of 64x64, a 3-stage ring, two per CU),
//   128x128 and 64x64, chosen by the number of workgroups they give; a
//   result's sum is the same in all of them. Tiles are mapped to the XCDs so
//   that workgroups sharing an L2 share operand tiles.
//   Requires K % 64 == 0, MA % 4 == 0, 16-byte aligned rows (lda, ldb % 8 == 0).
// gemm_f32: fp32 inputs on v_mfma_f32_16x16x4_f32 for the fp32 model, 64x64 or
//   128x128 tiles. Requires K % 32 == 0 and 16-byte aligned rows.
#pragma once

#include <atomic>

#include "common.h"

namespace wmi {

typedef __bf16 mfma_bf16x8 __attribute__((ext_vector_type(8)));
typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ bf16 MFMA

namespace gb {
constexpr int BM = 256;       // A rows per workgroup
constexpr int BN = 256;       // B rows per workgroup
constexpr int BK = 64;        // K per LDS buffer
constexpr int THREADS = 512;  // 8 waves
constexpr int OP_BYTES = 256 * BK * 2;         // one operand tile of a buffer (32 KiB)
constexpr int STAGE_BYTES = 2 * OP_BYTES;      // A and B tiles (64 KiB)
constexpr int LDS_BYTES = 2 * STAGE_BYTES;     // two buffers (128 KiB)
}  // namespace gb

// Byte offset of 16-byte chunk c (0..3) of row r in a [rows][32] bf16 LDS tile:
// position c ^ ((r >> 1) & 3), so the 8 rows read together by a ds_read_b128
// group hit distinct banks.
__device__ inline int swz32(int r, int c) { return r * 64 + ((c ^ ((r >> 1) & 3)) << 4); }

// s_waitcnt immediate that waits until at most n vector-memory ops are outstanding.
#define WMI_VMCNT(n) ((((n) & 0xF)) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))
// The same, and for every LDS read of this wave. A barrier does not wait for
// them, and after it other waves' direct loads refill the buffer read last.
#define WMI_VMCNT_LDS(n) (WMI_VMCNT(n) & ~(0xF << 8))

// Byte offset of 16-byte chunk c (0..7) of row r inside a [rows][64] bf16 LDS tile.
__device__ inline int swz(int r, int c) { return r * 128 + ((c ^ (r & 7)) << 4); }

// Tile of workgroup `bid` among tilesA x tilesB tiles, arranged for the L2
// of each XCD: workgroups are handed to the 8 XCDs in turn (bid mod 8), so
// XCD x gets a contiguous run of tiles, and runs are ordered in groups of
// GA A-tiles (A-tile fastest): the ~32 workgroups an XCD holds at a time
// then cover about 4 A-tiles x 8 B-tiles, and each tile's K-slices are
// fetched into that XCD's L2 once for several workgroups.
__device__ inline void xcd_tile(int bid, int tilesA, int tilesB, int& ta, int& tb) {
    constexpr int GA = 4;
    const int T = tilesA * tilesB, per = T >> 3, rem = T & 7;
    const int x = bid & 7, j = bid >> 3;
    const int v = x * per + min(x, rem) + j;
    const int g = v / (GA * tilesB), ga = min(GA, tilesA - g * GA);
    const int w = v - g * GA * tilesB;
    tb = w / ga;
    ta = g * GA + (w - tb * ga);
}

// Epilogue of a wave's NI x NJ blocks of 16 x 16 results: lane (fr, fc) of
// block (i, j) holds rows ia + 16 i + 4 fc .. + 3 of column jb + 16 j + fr.
// For each column block, all of its loads (pre) are issued before its
// stores. A tile wholly inside the output (full, the common case) skips the
// per-element bounds tests, each a branch and an exec-mask update.
template <int NI, int NJ, class Epi>
__device__ __forceinline__ void tile_epilogue(const Epi& epi, const mfma_f32x4 (&acc)[NI][NJ], int ia, int jb, int fr,
                                              int fc, int z, int MA, int MB, bool full) {
    if (full) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int jj = jb + j * 16 + fr;
            EpiPre pre[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) pre[i] = epi.pre(ia + i * 16 + fc * 4, jj, z);
#pragma unroll
            for (int i = 0; i < NI; ++i)
                epi(ia + i * 16 + fc * 4, jj, z, acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3], pre[i]);
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int jj = jb + j * 16 + fr;
        const bool jok = jj < MB;
        EpiPre pre[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int ii = ia + i * 16 + fc * 4;
            if (jok && ii < MA) pre[i] = epi.pre(ii, jj, z);
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int ii = ia + i * 16 + fc * 4;
            if (jok && ii < MA) epi(ii, jj, z, acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3], pre[i]);
        }
    }
}

// C = A B^T for A [MA][K], B [MB][K] (bf16, row-major, batched over z):
// a 256 x 256 workgroup tile, 8 waves of 128 x 64 on 16x16x32 MFMAs, K tiles
// of 64 in two LDS buffers (128-byte rows, 16-byte chunk c of row r at
// c ^ ((r >> 1) & 7)), filled by direct global->LDS loads.
//
// A CU reads LDS at 128 bytes per clock, and these wave tiles need as many
// clocks of fragment reads as of MFMAs, so the two have to run side by side
// all the time. The waves therefore work in two groups of four, one wave of
// each per SIMD, half a phase apart: while one group runs the 16 MFMAs of a
// phase, the other reads its next fragments and issues loads, and a barrier
// swaps them. Raised priority keeps a group's MFMAs ahead of the other
// group's reads. A K tile takes four phases, over the wave's quadrants
//   (a0, b0) (a0, b1) (a1, b1) (a1, b0),
// a0 / a1 being its 64-row halves and b0 / b1 its 32-row halves, so a phase
// reads 12, 4, 8 and 0 fragments. The loads of tile t + 2 go into tile t's
// buffer by halves (A rows with bit 6 = h, B rows with bit 5 = h), each two
// phases after its half of tile t was read (the groups being one barrier
// apart, every wave's reads have then completed) and 12 barriers before its
// own first read; the vmcnt waits count exactly the later loads in flight.
// In a result's sum k runs in order, as in every tile size.
//
// 48000 x 5120 x 1280 without an epilogue 446 us (1412 TFLOP/s) against
// 528 us (1191) of a four-stage ring with one barrier per 32-wide K tile, in
// which all waves read at once and then multiplied at once; with GELU 597
// against 677 us; 48000 x 1280 x 5120 with the residual update 563 against
// 662 us. What is left is mostly the epilogue, which nothing overlaps.
template <class Epi>
__global__ __launch_bounds__(512, 2) void gemm_bf16_kernel(
    const bf16* __restrict__ A, int lda, long long sA, const bf16* __restrict__ B, int ldb,
    long long sB, int MA, int MB, int K, int tilesA, Epi epi) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int z = blockIdx.z;
    int ta, tb;
    xcd_tile(blockIdx.x, tilesA, (int)(gridDim.x / tilesA), ta, tb);
    const int a0 = ta * gb::BM, b0 = tb * gb::BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wa = (wave & 1) * 128, wb = (wave >> 1) * 64;
    const int fr = lane & 15, fc = lane >> 4;
    const unsigned char* pA = reinterpret_cast<const unsigned char*>(A + (long long)z * sA + (long long)a0 * lda);
    const unsigned char* pB = reinterpret_cast<const unsigned char*>(B + (long long)z * sB + (long long)b0 * ldb);

    // Direct loads: of each half tile (128 rows) wave w fills the 8-row groups
    // 2 w and 2 w + 1, one instruction each; lane i loads the logical chunk
    // stored at position i % 8 of row i / 8. Offsets are from the tile's first
    // row; rows past the matrix re-read its last one.
    unsigned oa[2][2], ob[2][2];
    int la[2][2], lb[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int g = wave * 2 + s;
            const int ra = (g >> 3) * 128 + (g & 7) * 8 + 64 * h, rb = (g >> 2) * 64 + (g & 3) * 8 + 32 * h;
            const int r = ra + (lane >> 3), q = rb + (lane >> 3);
            oa[h][s] = (unsigned)(min(a0 + r, MA - 1) - a0) * (unsigned)(lda * 2) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
            ob[h][s] = (unsigned)(min(b0 + q, MB - 1) - b0) * (unsigned)(ldb * 2) + (((lane & 7) ^ ((q >> 1) & 7)) << 4);
            la[h][s] = ra * 128;
            lb[h][s] = gb::OP_BYTES + rb * 128;
        }
#define WMI_LOAD_A(H, T)                                                                       \
    do {                                                                                       \
        const int b_ = ((T) & 1) * gb::STAGE_BYTES;                                            \
        const unsigned char* p_ = pA + (T) * 128;                                              \
        __builtin_amdgcn_global_load_lds(p_ + oa[H][0], lds + b_ + la[H][0], 16, 0, 0);        \
        __builtin_amdgcn_global_load_lds(p_ + oa[H][1], lds + b_ + la[H][1], 16, 0, 0);        \
    } while (0)
#define WMI_LOAD_B(H, T)                                                                       \
    do {                                                                                       \
        const int b_ = ((T) & 1) * gb::STAGE_BYTES;                                            \
        const unsigned char* p_ = pB + (T) * 128;                                              \
        __builtin_amdgcn_global_load_lds(p_ + ob[H][0], lds + b_ + lb[H][0], 16, 0, 0);        \
        __builtin_amdgcn_global_load_lds(p_ + ob[H][1], lds + b_ + lb[H][1], 16, 0, 0);        \
    } while (0)
#define WMI_SWAP()                             \
    do {                                       \
        __builtin_amdgcn_sched_barrier(0);     \
        __builtin_amdgcn_s_barrier();          \
        __builtin_amdgcn_sched_barrier(0);     \
    } while (0)

    mfma_f32x4 acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
    int ra[2], rb[2];  // this lane's fragment bytes of the first row block, k-steps 0 and 1
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        ra[s] = (wa + fr) * 128 + (((4 * s + fc) ^ (fr >> 1)) << 4);
        rb[s] = gb::OP_BYTES + (wb + fr) * 128 + (((4 * s + fc) ^ (fr >> 1)) << 4);
    }
    mfma_bf16x8 fa[4][2], fb0[2][2], fb1[2][2];
#define WMI_READ_A(H)                                                                                          \
    _Pragma("unroll") for (int i = 0; i < 4; ++i) _Pragma("unroll") for (int s = 0; s < 2; ++s) fa[i][s] =     \
        *reinterpret_cast<const mfma_bf16x8*>(stage + ra[s] + ((H) * 4 + i) * 2048)
#define WMI_READ_B(F, H)                                                                                       \
    _Pragma("unroll") for (int j = 0; j < 2; ++j) _Pragma("unroll") for (int s = 0; s < 2; ++s) F[j][s] =      \
        *reinterpret_cast<const mfma_bf16x8*>(stage + rb[s] + ((H) * 2 + j) * 2048)
#define WMI_MMA(F, AH, BH)                                                                                     \
    do {                                                                                                       \
        __builtin_amdgcn_sched_barrier(0);                                                                     \
        __builtin_amdgcn_s_setprio(1);                                                                         \
        _Pragma("unroll") for (int s = 0; s < 2; ++s) _Pragma("unroll") for (int j = 0; j < 2; ++j)           \
            _Pragma("unroll") for (int i = 0; i < 4; ++i) acc[(AH) * 4 + i][(BH) * 2 + j] =                    \
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i][s], F[j][s], acc[(AH) * 4 + i][(BH) * 2 + j], 0, 0, 0); \
        __builtin_amdgcn_s_setprio(0);                                                                         \
        __builtin_amdgcn_sched_barrier(0);                                                                     \
    } while (0)
    constexpr int LGKM0 = 0xC07F;  // wait for every LDS read, for no vector-memory operation

    const int nk = K / gb::BK;  // at least 2
    WMI_LOAD_A(0, 0);
    WMI_LOAD_B(0, 0);
    WMI_LOAD_B(1, 0);
    WMI_LOAD_A(1, 0);
    WMI_LOAD_A(0, 1);
    WMI_LOAD_B(0, 1);
    WMI_LOAD_B(1, 1);
    __builtin_amdgcn_s_waitcnt(WMI_VMCNT(10));  // a0 and b0 of tile 0
    WMI_SWAP();
    if (wave >= 4) WMI_SWAP();  // the second group starts half a phase later
    for (int t = 0; t < nk; ++t) {
        const unsigned char* stage = lds + (t & 1) * gb::STAGE_BYTES;
        const bool last = t == nk - 1, last2 = t == nk - 2;
        WMI_READ_B(fb0, 0);
        WMI_READ_A(0);
        if (!last) {
            WMI_LOAD_A(1, t + 1);
            __builtin_amdgcn_s_waitcnt(WMI_VMCNT(10));  // b1 of tile t
        } else {
            __builtin_amdgcn_s_waitcnt(WMI_VMCNT(2));
        }
        WMI_SWAP();
        __builtin_amdgcn_s_waitcnt(LGKM0);
        WMI_MMA(fb0, 0, 0);
        WMI_SWAP();
        WMI_READ_B(fb1, 1);
        if (!last) __builtin_amdgcn_s_waitcnt(WMI_VMCNT(8));  // a1 of tile t
        else __builtin_amdgcn_s_waitcnt(WMI_VMCNT(0));
        WMI_SWAP();
        __builtin_amdgcn_s_waitcnt(LGKM0);
        WMI_MMA(fb1, 0, 1);
        WMI_SWAP();
        WMI_READ_A(1);
        if (!last && !last2) {
            WMI_LOAD_A(0, t + 2);
            WMI_LOAD_B(0, t + 2);
        }
        WMI_SWAP();
        __builtin_amdgcn_s_waitcnt(LGKM0);
        WMI_MMA(fb1, 1, 1);
        WMI_SWAP();
        if (!last && !last2) {
            WMI_LOAD_B(1, t + 2);
            __builtin_amdgcn_s_waitcnt(WMI_VMCNT(10));  // a0 and b0 of tile t + 1
        } else if (last2) {
            __builtin_amdgcn_s_waitcnt(WMI_VMCNT(4));
        }
        WMI_SWAP();
        WMI_MMA(fb0, 1, 0);
        WMI_SWAP();
    }
    if (wave < 4) WMI_SWAP();  // as many barriers as the second group
#undef WMI_LOAD_A
#undef WMI_LOAD_B
#undef WMI_SWAP
#undef WMI_READ_A
#undef WMI_READ_B
#undef WMI_MMA
    tile_epilogue(epi, acc, a0 + wa, b0 + wb, fr, fc, z, MA, MB, a0 + gb::BM <= MA && b0 + gb::BN <= MB);
}

// Two-workgroups-per-CU variant: a 256 x 128 tile, 8 waves of 64 x 64
// (64 accumulator registers), a 3-stage ring of 24 KiB stages (72 KiB), so
// two workgroups share a CU and one's prologue and epilogue overlap the
// other's main loop.
namespace gh {
constexpr int BM = 256, BN = 128, BK = 32, NS = 3, THREADS = 512;
constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;  // 16 KiB, 8 KiB
constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
constexpr int LDS_BYTES = NS * STAGE_BYTES;  // 72 KiB
}  // namespace gh

template <class Epi>
__global__ __launch_bounds__(512, 2) void gemm_bf16_h_kernel(
    const bf16* __restrict__ A, int lda, long long sA, const bf16* __restrict__ B, int ldb,
    long long sB, int MA, int MB, int K, int tilesA, Epi epi) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int z = blockIdx.z;
    A += (long long)z * sA;
    B += (long long)z * sB;
    int ta, tb;
    xcd_tile(blockIdx.x, tilesA, (int)(gridDim.x / tilesA), ta, tb);
    const int a0 = ta * gh::BM, b0 = tb * gh::BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wa = (wave & 3) * 64, wb = (wave >> 2) * 64;
    const int fr = lane & 15, fc = lane >> 4;

    // Direct loads: wave w fills A rows 32 w .. 32 w + 31 (2 instructions of
    // 16 rows x 64 B) and B rows 16 w .. 16 w + 15 (1 instruction).
    const int dr = lane >> 2;
    const int dc = (lane & 3) ^ ((dr >> 1) & 3);
    const bf16* ga[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) ga[s] = A + (long long)min(a0 + wave * 32 + s * 16 + dr, MA - 1) * lda + dc * 8;
    const bf16* gp = B + (long long)min(b0 + wave * 16 + dr, MB - 1) * ldb + dc * 8;

    mfma_f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};

#define WMI_ISSUE3(KT)                                                                                  \
    do {                                                                                                \
        const int st_ = ((KT) % gh::NS) * gh::STAGE_BYTES;                                              \
        const int k_ = (KT) * gh::BK;                                                                   \
        _Pragma("unroll") for (int s = 0; s < 2; ++s)                                                  \
            __builtin_amdgcn_global_load_lds(ga[s] + k_, lds + st_ + wave * 2048 + s * 1024, 16, 0, 0); \
        __builtin_amdgcn_global_load_lds(gp + k_, lds + st_ + gh::A_BYTES + wave * 1024, 16, 0, 0);     \
    } while (0)

    const int nk = K / gh::BK;
    WMI_ISSUE3(0);
    if (nk > 1) WMI_ISSUE3(1);
    for (int kt = 0; kt < nk; ++kt) {
        // tile kt has landed once only the 3-load group of the next tile is pending
        if (kt + 1 < nk) __builtin_amdgcn_s_waitcnt(WMI_VMCNT_LDS(3));
        else __builtin_amdgcn_s_waitcnt(WMI_VMCNT_LDS(0));
        __builtin_amdgcn_s_barrier();
        if (kt + gh::NS - 1 < nk) WMI_ISSUE3(kt + gh::NS - 1);
        const unsigned char* stage = lds + (kt % gh::NS) * gh::STAGE_BYTES;
        mfma_bf16x8 fa[4], fb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) fa[i] = *reinterpret_cast<const mfma_bf16x8*>(stage + swz32(wa + i * 16 + fr, fc));
#pragma unroll
        for (int j = 0; j < 4; ++j)
            fb[j] = *reinterpret_cast<const mfma_bf16x8*>(stage + gh::A_BYTES + swz32(wb + j * 16 + fr, fc));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
#undef WMI_ISSUE3
    tile_epilogue(epi, acc, a0 + wa, b0 + wb, fr, fc, z, MA, MB, a0 + gh::BM <= MA && b0 + gh::BN <= MB);
}

// Raises kernel f's dynamic LDS limit to `bytes` on the current device, once
// per device (the attribute is per device; `done` holds one bit per device).
inline void lds_limit(const void* f, int bytes, std::atomic<uint64_t>& done) {
    int dev = 0;
    WMI_HIP(hipGetDevice(&dev));
    const uint64_t bit = 1ull << (dev & 63);
    if (done.load() & bit) return;
    WMI_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    done.fetch_or(bit);
}

// ----------------------------------------------------------------- 64 x 64 and 128 x 128 tiles
//
// C = A B^T with a workgroup tile of 32 WT x 32 WT, 4 waves of 16 WT x 16 WT,
// for the fp32 model (fp32 products and sums on v_mfma_f32_16x16x4_f32) and
// for the bf16 launches whose larger tiles would leave CUs without work. K
// tiles are 128 bytes of a row (32 fp32 or 64 bf16 columns), streamed into an
// LDS ring of NS stages with direct global->LDS loads; 16-byte chunk c of row
// r sits at c ^ ((r >> 1) & 7), so the 16 rows of one read pass fill the 64
// banks once. A lane reads 16 bytes of a row per fragment: eight k of one
// bf16 MFMA, or four k that feed four fp32 MFMAs, step r reducing over
// k = 4 (lane / 16) + r of a 16-wide slice in both operands. In bf16 a
// result's sum is taken in the order of the larger tiles' kernels, so it is
// the same bit for bit with every tile.
// fp32 is bound by the matrix rate (a 16x16x4 takes 32 cycles of a SIMD):
// 13500 x 1536 x 384 with GELU: 153 us (104 TFLOP/s; with vector FMAs 10500
// rows took 374 us, 33 TFLOP/s); 1500 x 1536 x 384: 29 us (74 us).
template <class T> struct Frag;  // 16 bytes of an operand per lane
template <> struct Frag<bf16> {
    typedef mfma_bf16x8 type;
    static constexpr int STEPS = 1;  // MFMAs of a fragment pair
    static __device__ __forceinline__ mfma_f32x4 step(type a, type b, mfma_f32x4 c, int) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct Frag<float> {
    typedef mfma_f32x4 type;
    static constexpr int STEPS = 4;
    static __device__ __forceinline__ mfma_f32x4 step(type a, type b, mfma_f32x4 c, int r) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], b[r], c, 0, 0, 0);
    }
};

template <class T, int WT, int NS, class Epi>
__global__ __launch_bounds__(256, 2) void gemm_tile_kernel(const T* __restrict__ A, int lda, long long sA,
                                                           const T* __restrict__ B, int ldb, long long sB, int MA,
                                                           int MB, int K, int tilesA, Epi epi) {
    typedef typename Frag<T>::type frag;
    constexpr int TB = 32 * WT, OP_BYTES = TB * 128, STAGE = 2 * OP_BYTES;
    constexpr int BK = 128 / sizeof(T), EL = 16 / sizeof(T);
    extern __shared__ __align__(16) unsigned char lds[];
    const int z = blockIdx.z;
    A += (long long)z * sA;
    B += (long long)z * sB;
    int ta, tb;
    xcd_tile(blockIdx.x, tilesA, (int)(gridDim.x / tilesA), ta, tb);
    const int a0 = ta * TB, b0 = tb * TB;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wa = (wave & 1) * 16 * WT, wb = (wave >> 1) * 16 * WT;
    const int fr = lane & 15, fc = lane >> 4;

    // Direct loads: wave w fills rows 8 WT w .. 8 WT (w + 1) - 1 of both tiles
    // with WT + WT instructions of 8 rows; lane i loads the logical chunk
    // stored at position i % 8 of row i / 8.
    const unsigned char* ga[4];  // WT of them
    const unsigned char* gp[4];
#pragma unroll
    for (int s = 0; s < WT; ++s) {
        const int r = wave * 8 * WT + s * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        ga[s] = reinterpret_cast<const unsigned char*>(A + (long long)min(a0 + r, MA - 1) * lda + c * EL);
        gp[s] = reinterpret_cast<const unsigned char*>(B + (long long)min(b0 + r, MB - 1) * ldb + c * EL);
    }
#define WMI_ISSUET(KT)                                                                                    \
    do {                                                                                                  \
        int sa_ = ((KT) % NS) * STAGE + wave * 8 * WT * 128, sb_ = sa_ + OP_BYTES;                        \
        const int k_ = (KT) * 128;                                                                        \
        _Pragma("unroll") for (int s = 0; s < WT; ++s) {                                                 \
            __builtin_amdgcn_global_load_lds(ga[s] + k_, lds + sa_ + s * 1024, 16, 0, 0);                 \
            __builtin_amdgcn_global_load_lds(gp[s] + k_, lds + sb_ + s * 1024, 16, 0, 0);                 \
        }                                                                                                 \
    } while (0)
    mfma_f32x4 acc[WT][WT];
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[i][j] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};

    const int nk = K / BK;
#pragma unroll
    for (int q = 0; q < NS - 1; ++q)
        if (q < nk) WMI_ISSUET(q);
    for (int kt = 0; kt < nk; ++kt) {
        // tile kt has landed once only the later tiles' 2 WT loads are pending
        const int later = min(nk - 1 - kt, NS - 2);
        static_assert((WT == 2 && NS <= 4) || NS == 2, "the waits below are literals");
        if (later >= 2) __builtin_amdgcn_s_waitcnt(WMI_VMCNT_LDS(8));
        else if (later == 1) __builtin_amdgcn_s_waitcnt(WMI_VMCNT_LDS(4));
        else __builtin_amdgcn_s_waitcnt(WMI_VMCNT_LDS(0));
        __builtin_amdgcn_s_barrier();
        if (kt + NS - 1 < nk) WMI_ISSUET(kt + NS - 1);
        const unsigned char* stage = lds + (kt % NS) * STAGE;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            frag fa[WT], fb[WT];
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                const int ra = wa + i * 16 + fr, rb = wb + i * 16 + fr, c = 4 * h + fc;
                fa[i] = *reinterpret_cast<const frag*>(stage + ra * 128 + ((c ^ ((ra >> 1) & 7)) << 4));
                fb[i] = *reinterpret_cast<const frag*>(stage + OP_BYTES + rb * 128 + ((c ^ ((rb >> 1) & 7)) << 4));
            }
#pragma unroll
            for (int r = 0; r < Frag<T>::STEPS; ++r)
#pragma unroll
                for (int j = 0; j < WT; ++j)
#pragma unroll
                    for (int i = 0; i < WT; ++i) acc[i][j] = Frag<T>::step(fa[i], fb[j], acc[i][j], r);
        }
    }
#undef WMI_ISSUET
    tile_epilogue(epi, acc, a0 + wa, b0 + wb, fr, fc, z, MA, MB, a0 + TB <= MA && b0 + TB <= MB);
}

template <class T, int WT, int NS, class Epi>
inline void gemm_tile(const T* A, int lda, long long sA, const T* B, int ldb, long long sB, int MA, int MB, int K,
                      int batch, const Epi& epi, hipStream_t st) {
    const int ta = (MA + 32 * WT - 1) / (32 * WT), tb = (MB + 32 * WT - 1) / (32 * WT);
    hipLaunchKernelGGL((gemm_tile_kernel<T, WT, NS, Epi>), dim3(ta * tb, 1, batch), dim3(256), NS * 2 * 32 * WT * 128, st,
                       A, lda, sA, B, ldb, sB, MA, MB, K, ta, epi);
}

// 128 x 128 tiles once they fill the chip's 512 workgroup slots (two per
// CU); below that the 64 x 64 tiles' four times as many workgroups.
inline int gemm_f32_tile(int MA, int MB, int batch) {
    return (long long)((MA + 127) / 128) * ((MB + 127) / 128) * batch >= 512 ? 128 : 64;
}

template <class Epi>
inline void gemm_f32(const float* A, int lda, long long sA, const float* B, int ldb, long long sB, int MA, int MB,
                     int K, int batch, const Epi& epi, hipStream_t st) {
    // rows i0..i0+3 past MA reach the epilogue when MA % 4 != 0: it must drop them
    if (MA <= 0 || MB <= 0 || K <= 0 || K % 32 || lda % 4 || ldb % 4 || sA % 4 || sB % 4 || batch <= 0)
        throw ArgError(-1, "gemm_f32: unsupported shape");
    if (gemm_f32_tile(MA, MB, batch) == 128)
        gemm_tile<float, 4, 2>(A, lda, sA, B, ldb, sB, MA, MB, K, batch, epi, st);
    else
        gemm_tile<float, 2, 4>(A, lda, sA, B, ldb, sB, MA, MB, K, batch, epi, st);
}

// The tile by the number of workgroups it gives 256 CUs. Measured on whole
// passes of 1 to 32 segments at widths 512 to 2048 as they run, the two halves
// of a pass side by side, so that one half's workgroups fill the CUs that the
// other's last round leaves idle (pass times in us):
//  - 64 x 64 while 128 x 128 tiles are fewer than 144 (100: d = 1280, 1
//    segment 16 % slower; 200: d = 2048, 2 segments 9 % slower);
//  - 256 x 256, one per CU, from 144 tiles on (128 the same, 176 and 112 up to
//    4 % slower), unless K < 2048 and the rounds of more than one are less
//    than 60 % full (d = 768, 8 segments 4 % slower without this; a line at
//    75 %, right for a launch alone, lost 7 % at d = 1536, 20 segments, and d =
//    2048, 14 segments), and K >= 128, the two K tiles its loop needs;
//  - for K <= 640 (line at 75 %) with at least 750 of them, 256 x 128, two per
//    CU (alone, d = 512, 16 segments, QK: 38.5 against 41.7 us with 128; whole
//    passes at d = 384 and 512 measure the same with either, within 2 %);
//  - 128 x 128, two per CU, otherwise.
// Returns 64, 128, 256 or 384 (256 x 128).
inline int gemm_bf16_tile(int MA, int MB, int K, int batch) {
    const int tilesA = (MA + gb::BM - 1) / gb::BM, tilesB = (MB + gb::BN - 1) / gb::BN;
    const long long t128 = (long long)((MA + 127) / 128) * ((MB + 127) / 128) * batch;
    const long long t384 = (long long)tilesA * ((MB + gh::BN - 1) / gh::BN) * batch;
    const long long t256 = (long long)tilesA * tilesB * batch;
    const bool big = t256 >= 144 && (t256 <= 256 || K >= 2048 ||
                                     t256 * 100 >= (t256 + 255) / 256 * 256 * (K <= 640 ? 75 : 60));
    return t128 < 144 ? 64 : big && K >= 128 ? 256 : K <= 640 && t384 >= 750 ? 384 : 128;
}

template <class Epi>
inline void gemm_bf16(const bf16* A, int lda, long long sA, const bf16* B, int ldb, long long sB,
                      int MA, int MB, int K, int batch, const Epi& epi, hipStream_t st) {
    if (K <= 0 || K % 64 || MA % 4 || lda % 8 || ldb % 8 || MA <= 0 || MB <= 0 || batch <= 0)
        throw ArgError(-1, "gemm_bf16: unsupported shape");
    // WHISPER_GEMM_TILE = 64, 128, 256 or 384 forces one tile; the older
    // WHISPER_GEMM_H = 1 or 0 stands for 384 or 256.
    static const int force = [] {
        if (const char* g = getenv("WHISPER_GEMM_TILE")) {
            const int t = atoi(g);
            if (t != 64 && t != 128 && t != 256 && t != 384)
                throw ArgError(-1, "WHISPER_GEMM_TILE must be 64, 128, 256 or 384");
            return t;
        }
        if (const char* g = getenv("WHISPER_GEMM_H")) return g[0] == '1' ? 384 : 256;
        return 0;
    }();
    const int tile = force && (force != 256 || K >= 128) ? force : gemm_bf16_tile(MA, MB, K, batch);
    const int tilesA = (MA + gb::BM - 1) / gb::BM, tilesB = (MB + gb::BN - 1) / gb::BN;
    if (tile == 64) return gemm_tile<bf16, 2, 4>(A, lda, sA, B, ldb, sB, MA, MB, K, batch, epi, st);
    if (tile == 128) return gemm_tile<bf16, 4, 2>(A, lda, sA, B, ldb, sB, MA, MB, K, batch, epi, st);
    if (tile == 384) {
        static std::atomic<uint64_t> done_h{0};  // one per epilogue instantiation
        lds_limit(reinterpret_cast<const void*>(&gemm_bf16_h_kernel<Epi>), gh::LDS_BYTES, done_h);
        const int tb2 = (MB + gh::BN - 1) / gh::BN;
        dim3 grid(tilesA * tb2, 1, batch);
        hipLaunchKernelGGL((gemm_bf16_h_kernel<Epi>), grid, dim3(gh::THREADS), gh::LDS_BYTES, st, A, lda, sA, B,
                           ldb, sB, MA, MB, K, tilesA, epi);
        return;
    }
    static std::atomic<uint64_t> done{0};
    lds_limit(reinterpret_cast<const void*>(&gemm_bf16_kernel<Epi>), gb::LDS_BYTES, done);
    dim3 grid(tilesA * tilesB, 1, batch);
    hipLaunchKernelGGL((gemm_bf16_kernel<Epi>), grid, dim3(gb::THREADS), gb::LDS_BYTES, st, A, lda,
                       sA, B, ldb, sB, MA, MB, K, tilesA, epi);
}

}  // namespace wmi
