// Grouped W4A8 GEMMs on int8 MFMA for expert groups of more than a few token
// rows (paper Sec. 3.2: the token-expert pairs grouped by expert, one launch
// over all groups; Sec. 3.3: 4-bit weight codes times 8-bit activation codes,
// one scaling per 32 elements).
//
// Workgroup tile: up to 64 token rows of one group by one slice of 128 weight
// rows.  Each of the four waves owns 32 weight rows and both 32-row halves of
// the tokens (the second half is compiled out for tiles of at most 32 rows),
// so one weight operand feeds two v_mfma_i32_32x32x32_i8 per Q-block.
//   * Staging: four blocks (K = 128) of every operand at a time, by direct
//     loads into a ring of LDS slots: 80 bytes of each weight row (raw), 128
//     bytes of codes and 16 of scales of each token row.  A wave waits only
//     for its oldest stage (a vmcnt of the younger ones' loads; the two slots of
//     a 64-row tile leave none, so it waits for all) before the
//     stage's one barrier.  The raw weights go through LDS because a lane per
//     row read straight from memory touches a cache line per lane and
//     instruction; and because they then take no registers while under way.
//   * Weights: a lane of the 32x32x32 product supplies 16 of a row's 32 codes,
//     any 16 as long as the tokens' are the same ones: lanes l and l + 32
//     take the first and last 8 payload bytes of the row's block (two 4-bit
//     codes each), turned into the int8 16*(q-8) (the nibble q ^ 8 in the
//     high half of its byte).  The aligned codes of the tokens are stored in
//     that order (aligned_pos).
//   * Activations: the 16-byte pieces of a row XOR-swizzled by the row so the
//     rows a half-wave reads sit in distinct banks.
//   * Products: the weights are the A operand and the token rows the B
//     operand, so element e of an MFMA in lane l is weight row
//     8*(e/4) + 4*(l/32) + e%4 of the wave's 32 and token row l%32 of the
//     half: a lane holds one token's sums for 16 weight rows.  Tiles of at
//     most 16 rows run v_mfma_i32_16x16x32_i8 (half the padding): two per
//     block, weight rows 0..15 and 16..31 of the wave, lane l supplying the 8
//     codes of payload dword l/16 of row l%16.
//   * Scaling: the accumulator input is 0x4B400000, so the int32 result read
//     as a float is exactly 1.5*2^23 + 16 s (|16 s| < 2^22); t = fma(f, dx,
//     -1.5*2^23*dx) = 16 s dx rounded once and acc = fma(t, d_w/16, acc).  The
//     per-lane factor is the activation scale; the per-element factor is
//     the weight-row scale, which both token halves share: each wave puts
//     its rows' scales of the current stage in a small LDS table and reads
//     16 of them per block (broadcast reads, one set for both halves).
// Gate/up waves hold 16 gate rows and the 16 matching up rows, so element e
// and e + 8 of a lane are the gate and up sums of one column and SwiGLU
// needs no lane exchange; Q8_0 of each 32-wide h block goes through LDS.
// Down tiles write w * y per pair, through LDS in whole rows of 512 bytes.
//
// What bounds it.  Large products: VALU issue (16384 x 2048 x 2048: the VALU
// issues in 85% of the cycles, the matrix cores work in 16%; the two fp32
// operations per output and block are 32 of 43 VALU instructions per product).
// Prompt layers and products of few workgroups: latency (947 tokens, gate/up and
// down: VALU 58 and 49%; of the waves' cycles 28 and 41% wait on a counter or the
// barrier, 36 and 26% for issue).  A stage is a short chain (barrier, weight
// scales read, converted, written and read back, operands, products) that three
// workgroups per compute unit do not cover; registers (at most 168) and LDS
// (51 KB) allow no more.  Measured slower: four workgroups of 128 registers, waves
// of 64 weight rows, rings of four slots at two workgroups (also with one
// workgroup per compute unit), every slot filled before the first stage, and
// several slices per workgroup with the ring running on across them.
// Kernel times, trace medians before (weights loaded per lane into registers one
// group of eight blocks ahead, codes of K <= 512 resident over several slices, two
// workgroups per compute unit) and now, top-8 of 256 experts with skewed load, H =
// 2048, I = 512: gate/up of 947 tokens 125.5 -> 111.8 us, of 5120 tokens 404.9 ->
// 363.8; down 69.6 -> 67.4 and 221.0 -> 241.2 (a long prompt's down gives back half
// of what its gate/up gains); 333 tokens of 128 experts, I = 768: 76.7 -> 72.8 and
// 46.6 -> 41.7; 32 rows over 151936 x 2048 62.8 -> 59.6 (2.9 TB/s), 947 over 4096 x
// 2048 34.7 -> 33.7.  The fp32-scale form (one more operation per output and block,
// each stage summed on its own: 220 registers, two workgroups per compute unit)
// takes 132 and 80 us for gate/up and down of 947 tokens.
#include <algorithm>

#include "w4a8_dev.h"
#include "w4a8_host.h"

namespace w4a8 {

namespace {

constexpr int MNT = 256;           // threads: four waves
constexpr int MT = 64;             // token rows per tile
constexpr int WROWS = 128;         // weight rows per slice (32 per wave)
constexpr int Q4SB = W4A8_Q4_SYM_BLOCK_BYTES;
constexpr int BIAS = 0x4B400000;   // float 1.5 * 2^23
constexpr float BIASF = 12582912.0f;

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(4))) const int32_t CInt;

struct MArgs {
  const uint8_t *w, *ws;           // routed experts [E][N][K/32] Q4_0 / shared [N][K/32]
  const uint32_t *act;             // aligned Q8_0 codes [row][K/32][8 dwords]
  const float *actd;               // their scales [row][K/32]
  const int32_t *meta, *perm;
  const int4 *tiles;               // {expert, first sorted position, rows, -}
  const float *topk_w;
  const float *shared_w;           // down: the shared expert's weight per token, or null (1)
  float *h;                        // gate/up: fp32 h [P][I]
  uint8_t *hq;                     // gate/up: Q8_0(h) [P][I/32]
  uint32_t *ha;                    // gate/up: aligned codes of Q8_0(h) [P][I/32][8]
  float *hd;                       // gate/up: their scales [P][I/32]
  float *y;                        // down: w * y [P][H]
  int64_t T, k, E, N, K, I;
  int64_t M;                       // dense product (M > 0): M activation rows in implicit
                                   // tiles of tr rows, one weight matrix (ws), no route
  int tr, run;                     // dense product: rows per tile (16, 32 or 64), slices per run
};

// Weight of pair p in the combine: its routing weight, or for the shared
// pair of token t = p - T*k the shared expert's weight (1 without a gate).
__device__ __forceinline__ float pair_weight(const MArgs &a, int p) {
  const int64_t pr = a.T * a.k;
  return p < pr ? a.topk_w[p] : (a.shared_w ? a.shared_w[p - pr] : 1.0f);
}

// A stage is four blocks (K = 128) of the tile's operands in LDS, moved there
// by direct loads (global_load_lds) into a ring of slots.
constexpr int SB = 4;              // blocks per stage
constexpr int WCH = 5;             // 16-byte pieces of a weight row per stage (80 bytes)
constexpr int WDW = WCH * 4;       // ... in dwords

// Tile kinds by token rows: at most 16 (16x16x32 products), 32, 64.
constexpr int T16 = 0, T32 = 1, T64 = 2;
constexpr int tile_rows(int kind) { return kind == T64 ? 64 : kind == T32 ? 32 : 16; }

// A ring slot: the raw weight rows [wave][32 rows x 80 bytes], then the
// codes [row][piece ^ (row/2)%8] and scales [row] of the stage's four blocks.
constexpr int SLOT_W = 4 * 32 * WCH * 16;
constexpr int slot_bytes(int kind) { return SLOT_W + tile_rows(kind) * (128 + 16); }
// Two slots for 64-row tiles, three for 32, four for 16 (whose stages take
// least time to compute), within a third of a compute unit's LDS.
constexpr int RING_BYTES = 4 * slot_bytes(T16);
constexpr int ring_slots(int kind) { return RING_BYTES / slot_bytes(kind); }
constexpr int HVS = 68;            // row stride of the h tile
constexpr int EPI_BYTES = MT * (WROWS + 4) * 4;

struct MLds {
  // the ring; after it the tile's h (gate/up, float [64][68]) or output (down,
  // float [64][132]), then its pairs and combine weights (int and float [64])
  uint4 ring[RING_BYTES / 16];
  float dw[4][SB][32];             // weight-row scales of the current stage, [wave][block][row]
};

// Direct load of 16 bytes per active lane into LDS at dst + 16 * lane.
// Written as an instruction the compiler does not model: through the builtin
// it cannot tell a copy into one slot from reads of another, and waits for
// every outstanding load before reading LDS.  The copies are ordered by the
// explicit wait and barrier at the top of the stage that reads them.
// M0 is named as clobbered; nothing else in these kernels keeps a value in it.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma16(const uint8_t *src, const void *dst) {
  const uint32_t m0 =
      (uint32_t)(uintptr_t)(const void __attribute__((address_space(3))) *)dst;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(src), "s"(m0)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// All but this wave's youngest N vector memory operations are done, its LDS
// reads too, and so for every other wave of the workgroup.
template <int N>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Dwords of a weight row in a slot: block j's fp16 scale and payload.  A
// stage of Q4_0 is half a 144-byte group: the first half is loaded as bytes
// 0..79 of the group, the second as bytes 64..143, so its blocks start 8
// bytes into the row (o = 2 dwords).
__device__ __forceinline__ v4i codes4(uint32_t sh0, uint32_t nib0, uint32_t sh1, uint32_t nib1) {
  // q ^ 8 read as a signed 4-bit number is q - 8; placed in the high half of
  // a byte it is the int8 16 * (q - 8).  sh: the payload dword shifted up by
  // 4 (what is shifted in lands in the masked low half of a byte)
  return v4i{(int)((sh0 ^ 0x80808080u) & 0xF0F0F0F0u), (int)((nib0 ^ 0x88888888u) & 0xF0F0F0F0u),
             (int)((sh1 ^ 0x80808080u) & 0xF0F0F0F0u), (int)((nib1 ^ 0x88888888u) & 0xF0F0F0F0u)};
}
// Payload dwords c and c + 1 of block j of the row at wl: read, and turned
// into the int8 codes of elements 4c..4c+3, 4c+16..4c+19, 4c+4..4c+7,
// 4c+20..4c+23.
struct Raw {
  uint32_t d0, d1, d2;
};
template <bool SYM>
__device__ __forceinline__ Raw wraw(const uint32_t *wl, int j, int c) {
  if (SYM) return Raw{wl[5 * j + 1 + c], wl[5 * j + 2 + c], 0};
  const uint32_t *p = wl + 9 * (j >> 1) + c;
  return (j & 1) == 0 ? Raw{p[0], p[1], p[2]} : Raw{p[5], p[6], 0};
}
template <bool SYM>
__device__ __forceinline__ v4i wcodes2(const Raw &r, int j) {
  if (!SYM && (j & 1) == 0)
    return codes4(__builtin_amdgcn_alignbit(r.d1, r.d0, 12), align2(r.d1, r.d0),
                  __builtin_amdgcn_alignbit(r.d2, r.d1, 12), align2(r.d2, r.d1));
  return codes4(r.d0 << 4, r.d0, r.d1 << 4, r.d1);
}
// Payload dword c of block j: elements 4c..4c+3, 4c+16..4c+19.
template <bool SYM>
__device__ __forceinline__ long wcodes1(const uint32_t *wl, int j, int c) {
  uint32_t nib, sh;
  if (SYM) {
    nib = wl[5 * j + 1 + c];
    sh = nib << 4;
  } else {
    const uint32_t *p = wl + 9 * (j >> 1) + c;
    if ((j & 1) == 0) {
      const uint32_t d0 = p[0], d1 = p[1];
      nib = align2(d1, d0);
      sh = __builtin_amdgcn_alignbit(d1, d0, 12);
    } else {
      nib = p[5];
      sh = nib << 4;
    }
  }
  return __builtin_bit_cast(long, v2u{(sh ^ 0x80808080u) & 0xF0F0F0F0u,
                                      (nib ^ 0x88888888u) & 0xF0F0F0F0u});
}
// The scale of block j as the scaling step wants it: Q4_0 divided by 16
// (exact), the fp32 format as stored.
template <bool SYM>
__device__ __forceinline__ float wscale(const uint32_t *wl, int j) {
  if (SYM) return __builtin_bit_cast(float, wl[5 * j]);
  const uint32_t sd = wl[9 * (j >> 1) + 4 * (j & 1)];
  return 0.0625f * f16_bits_to_f32((j & 1) ? sd >> 16 : sd);
}

// Integer product with the bias accumulator input, read as floats (the whole
// vector at once: an element-wise bit cast has been folded to element 0).
__device__ __forceinline__ v16f mm(v4i a, v4i b, v16i c) {
  return __builtin_bit_cast(v16f, __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0));
}
typedef float v4f __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4f mm16(long a, long b, v4i c) {
  return __builtin_bit_cast(v4f, __builtin_amdgcn_mfma_i32_16x16x32_i8(a, b, c, 0, 0, 0));
}

// acc += s * dx * dw of one element; f = 1.5*2^23 + 16 s.  fp16 scales: t =
// fma(f, dx, nbx) = 16 s dx rounded once (nbx = -1.5*2^23*dx is exact for an
// 11-bit scale), dw divided by 16.  fp32 scales: that product would round,
// so s alone (exact) times the two scales' product, as the pair-by-pair and
// VALU kernels form it (s dx first could overflow where dw dx does not).
template <bool SYM>
__device__ __forceinline__ float scale1(float acc, float f, float dx, float nbx, float dw) {
  if (SYM) return fmaf(fmaf(f, 0.0625f, -0.0625f * BIASF), dw * dx, acc);
  return fmaf(fmaf(f, dx, nbx), dw, acc);
}
template <bool SYM>
__device__ __forceinline__ void scale4(float *acc, float f0, float f1, float f2, float f3, float dx,
                                       float nbx, float4 dw) {
  acc[0] = scale1<SYM>(acc[0], f0, dx, nbx, dw.x);
  acc[1] = scale1<SYM>(acc[1], f1, dx, nbx, dw.y);
  acc[2] = scale1<SYM>(acc[2], f2, dx, nbx, dw.z);
  acc[3] = scale1<SYM>(acc[3], f3, dx, nbx, dw.w);
}
template <bool SYM>
__device__ __forceinline__ void scale16(float acc[16], const v16f &f, float dx, float nbx,
                                        const float4 dw[4]) {
#pragma unroll
  for (int q = 0; q < 4; q++)
    scale4<SYM>(acc + 4 * q, f[4 * q], f[4 * q + 1], f[4 * q + 2], f[4 * q + 3], dx, nbx, dw[q]);
}

// One block's product operands in LDS as a lane of the 32-row form reads
// them: its weight payload and its token's codes of both halves.
struct BlockIn {
  Raw r;
  v4i u0, u1;
};
template <bool SYM, bool TWO>
__device__ __forceinline__ BlockIn block_in(const uint32_t *wl, const uint4 *a0, const uint4 *a1,
                                            int j, int hh, int sw) {
  BlockIn o;
  o.r = wraw<SYM>(wl, j, 2 * hh);
  o.u0 = __builtin_bit_cast(v4i, a0[(2 * j + hh) ^ sw]);
  o.u1 = TWO ? __builtin_bit_cast(v4i, a1[(2 * j + hh) ^ sw]) : v4i{0, 0, 0, 0};
  return o;
}

// One tile: rows token rows of expert's group from sorted position pos (or of
// the dense rows from pos), against one slice of weight rows.
template <bool GATEUP, int KIND, bool SYM>
__device__ __forceinline__ void mfma_tile(const MArgs &a, MLds &L, int expert, int pos, int rows,
                                          int slice) {
  constexpr int ROWS = tile_rows(KIND), NS = ring_slots(KIND), SLOT = slot_bytes(KIND);
  static_assert(NS >= 2 && EPI_BYTES + MT * 8 <= RING_BYTES, "two stages, and the epilogue, fit the ring");
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int nblk = (int)(a.K / 32), S = nblk / SB;
  uint8_t *const ring = reinterpret_cast<uint8_t *>(L.ring);

  // the pair of tile row m, or -1 (padding)
  auto row_pair = [&](int m) { return m < rows ? (a.M ? pos + m : a.perm[pos + m]) : -1; };
  // its activation row (padding rows read the last row)
  auto row_act = [&](int m) {
    const int p = row_pair(min(m, rows - 1)), pr = (int)(a.T * a.k);
    return GATEUP ? (p < pr ? p / (int)a.k : p - pr) : p;
  };

  // ---- direct loads: this lane's sources
  // weights: the wave's 32 rows as 160 pieces of 16 bytes, piece i of row i / 5
  constexpr int BB = SYM ? Q4SB : Q4B;
  const uint32_t rowbytes = (uint32_t)nblk * BB;
  const uint8_t *const W =
      expert < a.E ? a.w + (int64_t)expert * a.N * (int64_t)rowbytes : a.ws;
  const uint8_t *wsrc[3];
#pragma unroll
  for (int u = 0; u < 3; u++) {
    const int i = min(64 * u + lane, 32 * WCH - 1);
    const int r = i / WCH;
    uint32_t grow;
    if (GATEUP) {
      const uint32_t col = (uint32_t)slice * 64 + 16 * wave + (r & 15);
      grow = r < 16 ? col : (uint32_t)a.I + col;
    } else {
      // a last slice past N (dense products) reads row N - 1 and stores nothing
      grow = min((uint32_t)slice * WROWS + 32 * wave + r, (uint32_t)a.N - 1);
    }
    wsrc[u] = W + (uint64_t)grow * rowbytes + 16 * (i - r * WCH);
  }
  // codes: 8 rows of 128 bytes per instruction, CPW of them per wave (a
  // 16-row tile has two; waves 2 and 3 repeat them); scales: 16 bytes per
  // row, a quarter of the rows per wave
  constexpr int CPW = ROWS == 64 ? 2 : 1;
  constexpr int PER = 3 + CPW + 1;                // direct loads of a wave per stage
  const uint8_t *csrc[CPW];
  int crow[CPW];
#pragma unroll
  for (int u = 0; u < CPW; u++) {
    crow[u] = (8 * (CPW * wave + u)) % ROWS;
    const int r = crow[u] + (lane >> 3);
    csrc[u] = reinterpret_cast<const uint8_t *>(a.act) + (int64_t)row_act(r) * nblk * 32 +
              16 * ((lane & 7) ^ ((r >> 1) & 7));
  }
  constexpr int SPW = ROWS / 4;                   // scale rows per wave
  const uint8_t *ssrc = reinterpret_cast<const uint8_t *>(a.actd) +
                        (int64_t)row_act(SPW * wave + (lane & (SPW - 1))) * nblk * 4;
  auto load_stage = [&](int t) {
    uint8_t *const slot = ring + (t % NS) * SLOT;
    // a stage of Q4_0 is half a 144-byte group: bytes 0..79 or 64..143
    const uint32_t o = SYM ? t * 80u : (t >> 1) * 144u + (t & 1) * 64u;
    uint8_t *const dst = slot + wave * (32 * WCH * 16);
    lds_dma16(wsrc[0] + o, dst);
    lds_dma16(wsrc[1] + o, dst + 1024);
    if (lane < 32 * WCH - 128) lds_dma16(wsrc[2] + o, dst + 2048);
#pragma unroll
    for (int u = 0; u < CPW; u++)
      lds_dma16(csrc[u] + t * 128u, slot + SLOT_W + crow[u] * 128);
    if (lane < SPW) lds_dma16(ssrc + t * 16u, slot + SLOT_W + ROWS * 128 + SPW * wave * 16);
  };
  // the epilogue's pair and combine weight of tile row tid, fetched ahead of the
  // stages rather than behind the last (a dense product has nothing to fetch)
  int ep = -1;
  float epw = 0.0f;
  if (!a.M && tid < ROWS) {
    ep = row_pair(tid);
    if (!GATEUP && ep >= 0) epw = pair_weight(a, ep);
  }
#pragma unroll
  for (int t = 0; t < NS - 1; t++)
    if (t < S) load_stage(t);

  // this lane's roles: 32-row halves: weight row and token l % 32, half hh of
  // the block's elements; 16-row tiles: weight rows l % 16 and 16 + l % 16,
  // token l % 16, quarter c of the elements
  const int r32 = lane & 31, hh = lane >> 5;
  const int t16 = lane & 15, c16 = lane >> 4;
  float(*const Lw)[32] = L.dw[wave];

  float acc0[16], acc1[16];
#pragma unroll
  for (int e = 0; e < 16; e++) { acc0[e] = 0.0f; acc1[e] = 0.0f; }
  v16i c0;
#pragma unroll
  for (int e = 0; e < 16; e++) c0[e] = BIAS;
  const v4i c4 = v4i{BIAS, BIAS, BIAS, BIAS};

  for (int t = 0; t < S; t++) {
    // stage t has landed (of what is younger, up to NS - 2 stages' loads may
    // be under way), and every wave is done with stage t - 1, whose slot the
    // next loads fill
    if (NS > 2 && t + NS - 2 < S)
      wait_barrier<(NS - 2) * PER>();
    else if (NS > 3 && t + 1 < S)
      wait_barrier<(NS > 3 ? PER : 0)>();
    else
      wait_barrier<0>();
    if (t + NS - 1 < S) load_stage(t + NS - 1);
    const uint8_t *slot = ring + (t % NS) * SLOT;
    const uint32_t *wb =
        reinterpret_cast<const uint32_t *>(slot + wave * (32 * WCH * 16)) + (SYM ? 0 : 2 * (t & 1));
    const uint4 *ab = reinterpret_cast<const uint4 *>(slot + SLOT_W);
    const float4 *db = reinterpret_cast<const float4 *>(slot + SLOT_W + ROWS * 128);
    // the stage's weight-row scales to the wave's table: blocks 2hh, 2hh + 1
    // of row r32 (the wave's earlier reads of the table were issued before
    // these writes, and LDS runs one wave's accesses in order)
    {
      const uint32_t *wl = wb + r32 * WDW + (SYM ? 10 : 9) * hh;
      Lw[2 * hh][r32] = wscale<SYM>(wl, 0);
      Lw[2 * hh + 1][r32] = wscale<SYM>(wl, 1);
    }
    __builtin_amdgcn_wave_barrier();
    // fp32 scales: a stage's four blocks summed on their own, so that the long
    // sum's rounding error is no larger than that of the pair-by-pair kernel,
    // whose rows are summed by four lanes
    float p0[16], p1[16];
#pragma unroll
    for (int e = 0; e < 16; e++) { p0[e] = 0.0f; p1[e] = 0.0f; }
    if constexpr (KIND == T16) {
      const uint32_t *wl = wb + t16 * WDW;
      const float4 d = db[t16];
      const float dx[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
      for (int j = 0; j < SB; j++) {
        const long m0 = wcodes1<SYM>(wl, j, c16), m1 = wcodes1<SYM>(wl + 16 * WDW, j, c16);
        const v2u *bp = reinterpret_cast<const v2u *>(
            ab + t16 * 8 + ((2 * j + (c16 >> 1)) ^ ((t16 >> 1) & 7)));
        const long b = __builtin_bit_cast(long, bp[c16 & 1]);
        const v4f f0 = mm16(m0, b, c4), f1 = mm16(m1, b, c4);
        const float4 w0 = *reinterpret_cast<const float4 *>(&Lw[j][4 * c16]);
        const float4 w1 = *reinterpret_cast<const float4 *>(&Lw[j][16 + 4 * c16]);
        const float nb = -BIASF * dx[j];
        float *const sum = SYM ? p0 : acc0;
        scale4<SYM>(sum, f0[0], f0[1], f0[2], f0[3], dx[j], nb, w0);
        scale4<SYM>(sum + 4, f1[0], f1[1], f1[2], f1[3], dx[j], nb, w1);
      }
    } else {
      const uint32_t *wl = wb + r32 * WDW;
      const int sw = (r32 >> 1) & 7;              // rows r32 and r32 + 32 swizzle alike
      const uint4 *a0 = ab + r32 * 8, *a1 = ab + (32 + r32) * 8;
      const float4 d0 = db[r32];
      const float4 d1 = KIND == T64 ? db[32 + r32] : make_float4(0.f, 0.f, 0.f, 0.f);
      const float dx0[4] = {d0.x, d0.y, d0.z, d0.w}, dx1[4] = {d1.x, d1.y, d1.z, d1.w};
      // the scales of block j and the operands of block j + 1 are read behind
      // block j's products; the latter land while block j is scaled
      BlockIn in = block_in<SYM, KIND == T64>(wl, a0, a1, 0, hh, sw);
#pragma unroll
      for (int j = 0; j < SB; j++) {
        const v4i wo = wcodes2<SYM>(in.r, j);
        const v16f f0 = mm(wo, in.u0, c0);
        v16f f1;
        if (KIND == T64) f1 = mm(wo, in.u1, c0);
        float4 dw[4];
#pragma unroll
        for (int q = 0; q < 4; q++)
          dw[q] = *reinterpret_cast<const float4 *>(&Lw[j][8 * q + 4 * hh]);
        if (j + 1 < SB) in = block_in<SYM, KIND == T64>(wl, a0, a1, j + 1, hh, sw);
        __builtin_amdgcn_sched_barrier(0);
        scale16<SYM>(SYM ? p0 : acc0, f0, dx0[j], -BIASF * dx0[j], dw);
        if (KIND == T64) scale16<SYM>(SYM ? p1 : acc1, f1, dx1[j], -BIASF * dx1[j], dw);
      }
    }
    if (SYM) {
#pragma unroll
      for (int e = 0; e < 16; e++) { acc0[e] += p0[e]; acc1[e] += p1[e]; }
    }
  }

  // the ring becomes the h tile and the rows' pairs and combine weights
  wait_barrier<0>();
  float(*const hv)[HVS] = reinterpret_cast<float(*)[HVS]>(ring);
  int *const Lpair = reinterpret_cast<int *>(ring + EPI_BYTES);
  float *const Lpw = reinterpret_cast<float *>(ring + EPI_BYTES + 4 * MT);
  if (tid < ROWS) {
    Lpair[tid] = a.M ? row_pair(tid) : ep;
    if (!GATEUP) Lpw[tid] = a.M ? 1.0f : epw;
  }
  if (GATEUP) {
    // element e < 8 holds the gate sum and e + 8 the up sum of column
    // 16*wave + 8*(e/4) + 4*hh + e%4 for this lane's token (16-row tiles:
    // e < 4 gate and e + 4 up of column 16*wave + 4*(lane/16) + e of
    // token lane%16)
    if constexpr (KIND == T16) {
      const float *acc = acc0;
      *reinterpret_cast<float4 *>(&hv[lane & 15][16 * wave + 4 * (lane >> 4)]) =
          make_float4(silu_f32(acc[0]) * acc[4], silu_f32(acc[1]) * acc[5],
                      silu_f32(acc[2]) * acc[6], silu_f32(acc[3]) * acc[7]);
    } else {
#pragma unroll
      for (int half = 0; half < (KIND == T64 ? 2 : 1); half++) {
        const float *acc = half ? acc1 : acc0;
        float *hrow = &hv[32 * half + r32][16 * wave + 4 * hh];
#pragma unroll
        for (int q = 0; q < 2; q++)
          *reinterpret_cast<float4 *>(hrow + 8 * q) =
              make_float4(silu_f32(acc[4 * q + 0]) * acc[4 * q + 8],
                          silu_f32(acc[4 * q + 1]) * acc[4 * q + 9],
                          silu_f32(acc[4 * q + 2]) * acc[4 * q + 10],
                          silu_f32(acc[4 * q + 3]) * acc[4 * q + 11]);
      }
    }
    __syncthreads();
    // Q8_0 of each row's two 32-wide blocks: 8 lanes per block
    const int nbh = (int)(a.I / 32);
#pragma unroll
    for (int pass = 0; pass < ROWS * 16 / MNT; pass++) {
      const int idx = pass * MNT + tid;
      const int rb = idx >> 3, jq = idx & 7, m = rb >> 1, cb = rb & 1;
      const int p = Lpair[m];
      if (p >= 0) {                             // whole 8-lane groups agree
        const float4 hv4 = *reinterpret_cast<const float4 *>(&hv[m][32 * cb + 4 * jq]);
        const float v[4] = {hv4.x, hv4.y, hv4.z, hv4.w};
        const int bi = 2 * slice + cb;
        const int64_t blk = (int64_t)p * nbh + bi;
        float d;
        const uint32_t packed = quantize_block8<SYM>(v, a.hq, blk, jq, true, d);
        a.ha[blk * 8 + aligned_pos(jq)] = packed;
        if (jq == 0) a.hd[blk] = d;
        *reinterpret_cast<float4 *>(a.h + (int64_t)p * a.I + 32 * bi + 4 * jq) = hv4;
      }
    }
  } else {
    __syncthreads();
    // w * y of the tile through LDS, so that half a wave stores a whole row
    // of 512 bytes instead of 32-byte pieces of 32 rows: element 4q + i is
    // column 32*wave + 8q + 4hh + i of the slice (16-row tiles: of token
    // lane%16, column 32*wave + 16q + 4*(lane/16) + i)
    constexpr int YVS = WROWS + 4;
    float *const yt = reinterpret_cast<float *>(ring);
    static_assert(MT * YVS * 4 <= EPI_BYTES, "the output tile fits the epilogue");
    if constexpr (KIND == T16) {
      const float pw = Lpw[t16];
#pragma unroll
      for (int q = 0; q < 2; q++)
        *reinterpret_cast<float4 *>(yt + t16 * YVS + 32 * wave + 16 * q + 4 * c16) =
            make_float4(pw * acc0[4 * q], pw * acc0[4 * q + 1], pw * acc0[4 * q + 2],
                        pw * acc0[4 * q + 3]);
    } else {
#pragma unroll
      for (int half = 0; half < (KIND == T64 ? 2 : 1); half++) {
        const float *acc = half ? acc1 : acc0;
        const float pw = Lpw[32 * half + r32];
#pragma unroll
        for (int q = 0; q < 4; q++)
          *reinterpret_cast<float4 *>(yt + (32 * half + r32) * YVS + 32 * wave + 8 * q + 4 * hh) =
              make_float4(pw * acc[4 * q], pw * acc[4 * q + 1], pw * acc[4 * q + 2],
                          pw * acc[4 * q + 3]);
      }
    }
    __syncthreads();
    const bool vec = (a.N & 3) == 0;
    const int64_t n = (int64_t)slice * WROWS + 4 * r32;
#pragma unroll
    for (int u = 0; u < ROWS / 8; u++) {
      const int m = 8 * u + 2 * wave + hh, p = Lpair[m];
      if (p < 0 || n >= a.N) continue;
      const float4 v = *reinterpret_cast<const float4 *>(yt + m * YVS + 4 * r32);
      float *yp = a.y + (int64_t)p * a.N + n;
      if (vec) {
        *reinterpret_cast<float4 *>(yp) = v;
      } else {
        yp[0] = v.x;
        if (n + 1 < a.N) yp[1] = v.y;
        if (n + 2 < a.N) yp[2] = v.z;
        if (n + 3 < a.N) yp[3] = v.w;
      }
    }
  }
}

template <bool GATEUP, bool SYM>
__device__ __forceinline__ void mfma_body(const MArgs &a, MLds &L) {
  // Work items are (tile, slice).  Workgroup b runs on XCD b % 8 and is the
  // (b / 8)-th item there.  Each XCD takes an
  // even share of the long tiles (more than 32 rows), then an even share of
  // the short ones, each share a contiguous run of tiles (neighbouring tiles
  // of one expert share its weights in that XCD's L2), and all slices of a
  // tile in a row (they share the tile's codes).
  const int nsl = (int)(GATEUP ? a.I / 64 : (a.N + WROWS - 1) / WROWS);
  const int x = blockIdx.x & 7, q = blockIdx.x >> 3;
  int expert, pos, rows, slice;
  if (a.M) {
    // Dense products: runs of `run` slices of weight rows, within a run the
    // tiles in order, all the run's slices of a tile in a row, XCD x taking the
    // x-th of 8 even contiguous parts: a run's weights and a tile's codes are
    // shared in that XCD's L2, every XCD streams its own part of the weights
    // (so a handful of tiles still spreads over all 8), and an output row is
    // written in pieces of run * 512 bytes (one slice at a time, 512, reached
    // less of the memory's rate; see mfma_dense).
    const int ntl = (int)((a.M + a.tr - 1) / a.tr);
    const int tot = nsl * ntl;
    const int i0 = x * tot / 8, nx = (x + 1) * tot / 8 - i0;
    if (q >= nx) return;
    const int r = (i0 + q) / (ntl * a.run), in = (i0 + q) - r * (ntl * a.run);
    const int w = min(a.run, nsl - r * a.run);
    const int tile = in / w;
    slice = r * a.run + in - tile * w;
    expert = 0;                  // E = 0: the weights are ws
    pos = tile * a.tr;
    rows = (int)min((int64_t)a.tr, a.M - pos);
  } else {
    const int qt = q / nsl;
    slice = q - qt * nsl;
    const int ntiles = ((CInt *)a.meta)[2], nlong = ((CInt *)a.meta)[4];   // META_NTILES, META_NLONG
    const int l0 = x * nlong / 8, nl = (x + 1) * nlong / 8 - l0;
    const int nshort = ntiles - nlong;
    const int s0t = nlong + x * nshort / 8, ns_ = nlong + (x + 1) * nshort / 8 - s0t;
    if (qt >= nl + ns_) return;
    const int tile = qt < nl ? l0 + qt : s0t + (qt - nl);
    CInt *tp = (CInt *)a.tiles + 4 * tile;
    expert = tp[0]; pos = tp[1]; rows = tp[2];
  }
  if (rows > 32)
    mfma_tile<GATEUP, T64, SYM>(a, L, expert, pos, rows, slice);
  else if (rows > 16)
    mfma_tile<GATEUP, T32, SYM>(a, L, expert, pos, rows, slice);
  else
    mfma_tile<GATEUP, T16, SYM>(a, L, expert, pos, rows, slice);
}

template <bool GATEUP, bool SYM>
__global__ __launch_bounds__(MNT) __attribute__((amdgpu_waves_per_eu(SYM ? 2 : 3))) void mfma_kernel(MArgs a) {
  __shared__ MLds L;
  mfma_body<GATEUP, SYM>(a, L);
}

}  // namespace

int mfma_gateup(const uint8_t *w_gu, const uint8_t *ws_gu, const uint32_t *xa, const float *xd,
                const int32_t *meta, const int32_t *perm, const int4 *tiles, float *h,
                uint8_t *hq, uint32_t *ha, float *hd, int64_t maxtiles, int64_t T, int64_t H,
                int64_t I, int64_t E, int64_t k, bool sym, hipStream_t s) {
  MArgs a{};
  a.w = w_gu; a.ws = ws_gu; a.act = xa; a.actd = xd;
  a.meta = meta; a.perm = perm; a.tiles = tiles;
  a.h = h; a.hq = hq; a.ha = ha; a.hd = hd;
  a.T = T; a.k = k; a.E = E; a.N = 2 * I; a.K = H; a.I = I;
  // an XCD takes at most ceil(long/8) + ceil(short/8) <= ceil(maxtiles/8) + 1 tiles
  const dim3 grid((unsigned)(8 * ((maxtiles + 7) / 8 + 1) * (I / 64)));
  if (sym)
    mfma_kernel<true, true><<<grid, dim3(MNT), 0, s>>>(a);
  else
    mfma_kernel<true, false><<<grid, dim3(MNT), 0, s>>>(a);
  return check_launch();
}

int mfma_down(const uint8_t *w_d, const uint8_t *ws_d, const uint32_t *ha, const float *hd,
              const int32_t *meta, const int32_t *perm, const int4 *tiles, const float *topk_w,
              const float *shared_w, float *y, int64_t maxtiles, int64_t T, int64_t H, int64_t I,
              int64_t E, int64_t k, bool sym, hipStream_t s) {
  MArgs a{};
  a.w = w_d; a.ws = ws_d; a.act = ha; a.actd = hd;
  a.meta = meta; a.perm = perm; a.tiles = tiles;
  a.topk_w = topk_w; a.shared_w = shared_w; a.y = y;
  a.T = T; a.k = k; a.E = E; a.N = H; a.K = I; a.I = I;
  const int64_t nsl = H / WROWS;
  const dim3 grid((unsigned)(8 * ((maxtiles + 7) / 8 + 1) * nsl));
  if (sym)
    mfma_kernel<false, true><<<grid, dim3(MNT), 0, s>>>(a);
  else
    mfma_kernel<false, false><<<grid, dim3(MNT), 0, s>>>(a);
  return check_launch();
}

// Dense product y[m][n] = sum_b d_w[n,b] d_x[m,b] s[m,n,b] of M activation
// rows (aligned codes and fp32 scales) with one weight matrix [N][K/32].
int mfma_dense(const uint8_t *w, const uint32_t *act, const float *actd, float *y, int64_t M,
               int64_t N, int64_t K, int cus, hipStream_t s) {
  MArgs a{};
  a.w = nullptr; a.ws = w; a.act = act; a.actd = actd; a.y = y;
  a.T = 0; a.k = 0; a.E = 0; a.N = N; a.K = K; a.I = K; a.M = M;
  const int64_t nsl = (N + WROWS - 1) / WROWS;
  // Smaller tiles while each still has a compute unit to itself: a workgroup
  // alone on its unit overlaps nothing, so its time goes by its tile's rows.  us
  // at 64 / 32 / 16 rows: 129 x 2048 x 2048 (48, 80, 144 workgroups) 22.4 / 18.5 /
  // 14.9, 400 x 2048 x 2048 (112, 208, 400) 23.3 / 19.8 / 19.3, 700 x 2048 x 2048
  // (176, 352, 704) 24.4 / 25.0 / 25.4, 64 x 2048 x 4096 (16, 32, 64) 38.2 / 31.5 /
  // 24.3, 256 x 8192 x 4096 (256, 512, 1024) 40.8 / 42.0 / 56.2.
  a.tr = MT;
  for (int tr = MT / 2; tr >= 16 && nsl * ((M + tr - 1) / tr) <= cus; tr /= 2) a.tr = tr;
  // Runs of 16 slices while their weights fill no more than 2.5 of an L2's 4 MB.
  // us with runs of 1 / 4 / 16: 4096 x 151936 x 256 820 / 743 / 734, 16384 x 2048 x
  // 512 75.3 / 72.9 / 67.6, 4096 x 2048 x 1024 38.2 / 37.9 / 34.5, 947 x 2048 x 2048
  // 25.6 / 25.4 / 24.2; at K = 4096 (8 slices) 4096 x 8192 386 / 389 / 376.
  const int64_t slice_bytes = WROWS * (K / 32) * Q4B;
  a.run = (int)std::max<int64_t>(1, std::min<int64_t>(16, ((int64_t)5 << 19) / slice_bytes));
  const int64_t ntiles = (M + a.tr - 1) / a.tr;
  const int64_t grid = 8 * ((nsl * ntiles + 7) / 8);    // an XCD takes at most ceil(items/8)
  if (grid >= ((int64_t)1 << 31)) return W4A8_ERANGE;
  mfma_kernel<false, false><<<dim3((unsigned)grid), dim3(MNT), 0, s>>>(a);
  return check_launch();
}

}  // namespace w4a8
