// The gated-delta-net (GDN) recurrence of the model's linear-attention layers
// (Sec. 2.2: a state S in R^{dk x dv} per value head, updated token by token;
// the update is the gated delta rule of the work the paper cites)
//   S_t = a_t (I - b_t k_t k_t^T) S_{t-1} + b_t k_t v_t^T,   o_t = S_t^T q_t,
// a_t = exp(g_t), as a chunked scan: the paper names a chunked / parallel scan
// as the lever its token-by-token kernel lacked (Sec. 5.5).
//
// Within a chunk of C = 32 tokens, with L_i the sum of g over the chunk up to
// token i, the delta-rule corrections u_i = b_i (v_i - a_i S_{i-1}^T k_i)
// solve a unit lower-triangular system, and everything else is products:
//   (I + A) U = diag(b) (V - diag(e^L) K S),  A_ij = b_i e^{L_i - L_j} k_i.k_j (j < i)
//   O = diag(e^L) Q S + P U,                  P_ij = e^{L_i - L_j} q_i.k_j  (j <= i)
//   S <- e^{L_C} S + K^T diag(e^{L_C - L}) U.
// Up to 8 tokens (decode) one launch steps through the recurrence as
// written (gdn_step).  Longer sequences take two launches:
//   gdn_prep: per (head, chunk), in parallel: L, the dot products k.k and q.k,
//     A and P, T' = (I + A)^{-1} diag(b) and P T';
//   gdn_scan: per (head, 16 columns of the value dimension) -- the columns of
//     S evolve independently -- the chunks in order, the workgroup's slice of S
//     (DK x 16) in the accumulators of fp32 matrix products.  All column
//     slices of a head run on one XCD, so the head's inputs are fetched into
//     that XCD's L2 once.
// All arithmetic in fp32.
#include "w4a8_dev.h"
#include "w4a8_host.h"

namespace w4a8 {

namespace {

constexpr int GC = 32;      // tokens per chunk
constexpr int GNT = 256;    // threads per workgroup
constexpr int SNT = 512;    // ... of the scan
constexpr int DVS = 16;     // value columns per scan workgroup
constexpr int STC = 8;      // ... per step workgroup (and the granularity of DV)
constexpr int MAT = GC * GC;
constexpr int GDN_STEP_T = 8;   // up to this many tokens: the step kernel, no chunks

inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

struct GdnArgs {
  const float *q, *k, *v, *g, *beta, *s0;
  float *out, *s_out;
  float *tw, *pw, *lw;      // workspace: T' and P T' [NH][nch][C][C], L [NH][nch][C]
  int64_t T, NH, DV;
  int nch;
};

// Rows t0 .. t0 + 31 of head h of a [T][NH][D] tensor into LDS rows of
// stride D + 4 (zero past T).
template <int D>
__device__ __forceinline__ void load_rows(float (*dst)[D + 4], const float *src, int64_t t0,
                                          int64_t T, int64_t NH, int64_t h) {
  constexpr int D4 = D / 4;
  for (int idx = threadIdx.x; idx < GC * D4; idx += GNT) {
    const int i = idx / D4, c4 = idx - i * D4;
    const int64_t t = t0 + i;
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    if (t < T) x = reinterpret_cast<const float4 *>(src)[(t * NH + h) * D4 + c4];
    *reinterpret_cast<float4 *>(&dst[i][4 * c4]) = x;
  }
}

// One chunk's inputs of a scan workgroup, loaded into registers two chunks
// ahead: rows of K and Q (KF pieces of four per thread), one value of the 32 x
// 16 slice of V, two each of T' and P T', and L.
template <int DK>
struct ChunkRegs {
  static constexpr int KF = GC * DK / 4 / SNT;
  v4f k[KF], q[KF];
  v2f tp, pt;
  float v, l;
};

// Four products of 16 x 16 x 4 of a 16-byte piece of either operand, in two
// sums: lane l's pieces are k = 4 (l / 16) .. + 3 of row (A) and column (B) l % 16
// of 16 k in all; element e of a sum is row 4 (l / 16) + e, column l % 16.
__device__ __forceinline__ void mm4(float4 x, float4 y, v4f &c0, v4f &c1) {
  c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.x, c0, 0, 0, 0);
  c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, y.y, c1, 0, 0, 0);
  c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, y.z, c0, 0, 0, 0);
  c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, y.w, c1, 0, 0, 0);
}
__device__ __forceinline__ float4 quad(const float *p) {
  return *reinterpret_cast<const float4 *>(p);
}

// One (head, chunk): L, A, P, T' and P T'.  k.k and q.k on matrix products
// (waves 0, 1 the rows of K, waves 2, 3 those of Q, by 16 tokens, the lower tiles
// only).  (I + A)^{-1} by blocks of 16: the diagonal blocks by forward
// substitution, a column per lane of one wave (each column depends only on
// itself), the block below as -X22 A21 X11, then P T' on the products again.
// A chain of short steps, so as many workgroups per compute unit as fit (the
// matrices take the rows' place in LDS: four): 17 us for 947 tokens of 32 heads
// (22 with three workgroups; 35 with the dot products on the VALU out of LDS,
// a substitution over all 32 rows and P T' by the same 32 lanes).
template <int DK>
__global__ __launch_bounds__(GNT) void gdn_prep_kernel(GdnArgs a) {
  constexpr int MP = GC + 4;
  struct Rows {
    float K[GC][DK + 4], Q[GC][DK + 4];
  };
  struct Mats {
    float A[GC][MP], P[GC][MP];
    float Xt[GC][MP];                              // (I + A)^{-1} by column, then T'
    float Mt[16][20];                              // A21 X11 by column
  };
  static_assert(sizeof(Mats) <= sizeof(Rows), "the matrices take the rows' place");
  __shared__ __align__(16) uint8_t lds[sizeof(Rows)];
  __shared__ float Lc[GC], Bc[GC];
  float(*const Ks)[DK + 4] = reinterpret_cast<Rows *>(lds)->K;
  float(*const Qs)[DK + 4] = reinterpret_cast<Rows *>(lds)->Q;
  float(*const Am)[MP] = reinterpret_cast<Mats *>(lds)->A;
  float(*const Pm)[MP] = reinterpret_cast<Mats *>(lds)->P;
  float(*const Xt)[MP] = reinterpret_cast<Mats *>(lds)->Xt;
  float(*const Mt)[20] = reinterpret_cast<Mats *>(lds)->Mt;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, gq = lane >> 4;
  const int64_t h = blockIdx.x % a.NH;
  const int ch = (int)(blockIdx.x / a.NH);
  const int64_t t0 = (int64_t)ch * GC;
  const int64_t mat = ((int64_t)h * a.nch + ch) * MAT;
  load_rows<DK>(Ks, a.k, t0, a.T, a.NH, h);
  load_rows<DK>(Qs, a.q, t0, a.T, a.NH, h);
  if (tid < 64) {                                  // inclusive sums of g over the chunk
    const int64_t t = t0 + (tid & (GC - 1));
    float g = t < a.T ? a.g[t * a.NH + h] : 0.0f;
#pragma unroll
    for (int o = 1; o < GC; o *= 2) {
      const float p = __shfl_up(g, o, GC);
      if ((tid & (GC - 1)) >= o) g += p;
    }
    if (tid < GC) {
      Lc[tid] = g;
      Bc[tid] = t < a.T ? a.beta[t * a.NH + h] : 0.0f;
      a.lw[((int64_t)h * a.nch + ch) * GC + tid] = g;
    }
  }
  __syncthreads();
  {
    const int it = wave & 1;
    const bool isq = wave >= 2;
    const float(*const R)[DK + 4] = isq ? Qs : Ks;
    float(*const D)[MP] = isq ? Pm : Am;
    v4f c[2];
#pragma unroll
    for (int jt = 0; jt < 2; jt++) {
      v4f c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
      if (jt <= it) {
#pragma unroll 4
        for (int kb = 0; kb < DK; kb += 16)
          mm4(quad(&R[16 * it + n][kb + 4 * gq]), quad(&Ks[16 * jt + n][kb + 4 * gq]), c0, c1);
      }
      c[jt] = c0 + c1;
    }
    __syncthreads();                               // the matrices take the rows' place
#pragma unroll
    for (int jt = 0; jt < 2; jt++) {
      const int j = 16 * jt + n;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int i = 16 * it + 4 * gq + e;
        const float d = j <= i ? expf(Lc[i] - Lc[j]) * c[jt][e] : 0.0f;
        D[i][j] = isq ? d : (j < i ? Bc[i] * d : 0.0f);
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    // column n of diagonal block (lane / 16) % 2: m_r = [r = n] - sum_{l<r} A_rl m_l
    // (rows above n come out zero)
    if (lane < GC) {
      const int b0 = 16 * (lane >> 4);
      float m[16];
#pragma unroll
      for (int r = 0; r < 16; r++) {
        float acc = r == n ? 1.0f : 0.0f;
#pragma unroll
        for (int l = 0; l < r; l += 4) {
          const float4 av = quad(&Am[b0 + r][b0 + l]);
          acc = fmaf(-av.x, m[l], acc);
          if (l + 1 < r) acc = fmaf(-av.y, m[l + 1], acc);
          if (l + 2 < r) acc = fmaf(-av.z, m[l + 2], acc);
          if (l + 3 < r) acc = fmaf(-av.w, m[l + 3], acc);
        }
        m[r] = acc;
      }
#pragma unroll
      for (int r = 0; r < 16; r += 4) {
        *reinterpret_cast<float4 *>(&Xt[lane][b0 + r]) = make_float4(m[r], m[r + 1], m[r + 2], m[r + 3]);
        if (b0) *reinterpret_cast<float4 *>(&Xt[lane][r]) = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    __builtin_amdgcn_wave_barrier();               // LDS runs one wave's accesses in order
    v4f c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
    mm4(quad(&Am[16 + n][4 * gq]), quad(&Xt[n][4 * gq]), c0, c1);
    *reinterpret_cast<v4f *>(&Mt[n][4 * gq]) = c0 + c1;
    __builtin_amdgcn_wave_barrier();
    c0 = c1 = v4f{0.f, 0.f, 0.f, 0.f};
    mm4(make_float4(Xt[16 + 4 * gq][16 + n], Xt[16 + 4 * gq + 1][16 + n], Xt[16 + 4 * gq + 2][16 + n],
                    Xt[16 + 4 * gq + 3][16 + n]),
        quad(&Mt[n][4 * gq]), c0, c1);
    *reinterpret_cast<v4f *>(&Xt[n][16 + 4 * gq]) = -(c0 + c1);
    __builtin_amdgcn_wave_barrier();
    // T' = (I + A)^{-1} diag(b)
    if (lane < GC) {
      const float bj = Bc[lane];
#pragma unroll
      for (int r = 0; r < GC; r += 4)
        *reinterpret_cast<v4f *>(&Xt[lane][r]) = bj * *reinterpret_cast<const v4f *>(&Xt[lane][r]);
    }
  }
  __syncthreads();
  {
    const int r = tid >> 3, c = 4 * (tid & 7);
    *reinterpret_cast<float4 *>(a.tw + mat + 4 * tid) =
        make_float4(Xt[c][r], Xt[c + 1][r], Xt[c + 2][r], Xt[c + 3][r]);
  }
  // P T' (both lower triangular): the scan forms the output's second term P U =
  // (P T') W from W directly
  const int it = wave >> 1, jt = wave & 1;
  v4f c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
#pragma unroll
  for (int kb = 0; kb < GC; kb += 16)
    mm4(quad(&Pm[16 * it + n][kb + 4 * gq]), quad(&Xt[16 * jt + n][kb + 4 * gq]), c0, c1);
  c0 += c1;
#pragma unroll
  for (int e = 0; e < 4; e++) a.pw[mat + (16 * it + 4 * gq + e) * GC + 16 * jt + n] = c0[e];
}

// The chunks in order for 16 value columns of one head, eight waves, three
// phases per chunk on fp32 matrix products of 16 x 16 x 4:
//   1. X = K S: wave w the tokens 16 (w % 2) .. + 15 over a quarter of the DK rows
//      (w / 2), partial sums to LDS by column;
//   2. waves 0, 1: U = T' W with W = V - e^L X formed from the partials as it
//      is read, e^{L_C - L} U to LDS; waves 2, 3: (P T') W; waves 4..7: Y = Q S
//      (half the rows each); the next chunk's K and Q go to LDS;
//   3. S <- e^{L_C} S + K^T (e^{L_C - L} U), wave w the rows 16 w .. + 15, which
//      stay in its accumulators; waves 2, 3 O = e^L Y + (P T') W; S and what
//      phase 2 reads of the next chunk go to LDS.
// What bounds it is the chain of chunk steps, 2.1 us each at 947 tokens and 32
// heads of 128 x 128, of which the products are about 0.7 (two waves per SIMD).
// 16 columns fill the products' 16 and make one workgroup per compute unit.
// The scan of 947 tokens took 118 us with 8 columns (half of every product
// padding), four waves and U on the VALU; 78 with eight waves and 16 columns;
// 64 with Y and the outputs' stores off the chain and one multiply-add per
// load address.  The whole call at 16, 32, 33 and 64 heads (128, 256, 264 and 512
// workgroups, one per compute unit): 99 -> 68 us, 143 -> 73, 215 -> 133, 265 -> 143.
template <int DK>
__global__ __launch_bounds__(SNT) void gdn_scan_kernel(GdnArgs a) {
  constexpr int DKP = DK + 4;            // LDS row stride (rows of 8 threads hit distinct banks)
  constexpr int MP = GC + 4;             // ... of the chunk's 32-wide rows
  constexpr int KQ = DK / 4;             // rows of S per quarter
  constexpr int NT = DK / 16;            // row tiles of S
  static_assert(GC == 32 && DVS == 16 && SNT == 512 && MAT == 2 * SNT && KQ % 16 == 0 && NT <= 8,
                "roles of the scan");
  // K in two buffers: the next chunk's rows are written while the state
  // update still reads this chunk's
  __shared__ __align__(16) float Ks[2][GC][DKP], Qs[2][GC][DKP];
  // the slice of S before the chunk, column-major, in two buffers too
  __shared__ __align__(16) float St[2][DVS][DKP];
  __shared__ __align__(16) float Tp[GC][MP], PT[GC][MP];
  __shared__ __align__(16) float Xp[4][DVS][MP], Yp[2][DVS][MP];   // partial sums, by column
  __shared__ __align__(16) float Vt[DVS][MP], Ut[DVS][MP];
  __shared__ __align__(16) float eLs[GC], dLs[GC];                 // e^L, e^{L_C - L}
  const int tid = threadIdx.x;
  const int nsl = (int)((a.DV + DVS - 1) / DVS);
  // workgroup b runs on XCD b % 8: with NH a multiple of 8, all column
  // slices of head h run on XCD h % 8, so each head's K, Q, T' and P come
  // from HBM once and are shared in that XCD's L2
  int64_t h;
  int sl;
  if (a.NH % 8 == 0) {
    const int x = blockIdx.x % 8, slot = blockIdx.x / 8;
    h = x + 8 * (slot / nsl);
    sl = slot % nsl;
  } else {
    h = blockIdx.x / nsl;
    sl = blockIdx.x % nsl;
  }
  const int cb = sl * DVS;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, gq = lane >> 4;
  const bool col = cb + n < a.DV;        // columns past DV repeat the last one, unstored
  // rows 16 wave + 4 gq + e of column n
  v4f S = {0.f, 0.f, 0.f, 0.f};
  if (wave < NT && a.s0 && col) {
#pragma unroll
    for (int e = 0; e < 4; e++) S[e] = a.s0[(h * DK + 16 * wave + 4 * gq + e) * a.DV + cb + n];
  }

  // A chunk's loads.  None is conditional, and the loop below has no path
  // around them: otherwise the compiler cannot count the loads behind a
  // register's own and waits for all of them, two chunks' worth, at its use.
  // Tokens past T read the last one: their step beta is zero in T' and P T',
  // so they add nothing.
  constexpr int KF = ChunkRegs<DK>::KF, D4 = DK / 4, RPP = SNT / D4;       // rows per piece
  const int kr = tid / D4, kc = tid - kr * D4;       // row and piece of K, Q
  const int vr = tid / DVS, vc = tid % DVS;          // token and column of V
  // bytes per token (NH < 2^16 rows of at most 512 bytes, DV <= 4096)
  const uint32_t krow = (uint32_t)(a.NH * DK * 4), vrow = (uint32_t)(a.NH * a.DV * 4);
  const uint8_t *const kb = reinterpret_cast<const uint8_t *>(a.k + h * DK + 4 * kc);
  const uint8_t *const qb = reinterpret_cast<const uint8_t *>(a.q + h * DK + 4 * kc);
  const uint8_t *const vb =
      reinterpret_cast<const uint8_t *>(a.v + h * a.DV + min(cb + vc, (int)a.DV - 1));
  const int Tm1 = (int)a.T - 1;
  auto load = [&](int ch, ChunkRegs<DK> &r) {
    const int t0 = ch * GC;
#pragma unroll
    for (int u = 0; u < KF; u++) {
      const uint64_t row = (uint64_t)(uint32_t)min(t0 + kr + u * RPP, Tm1) * krow;
      r.k[u] = *reinterpret_cast<const v4f *>(kb + row);
      r.q[u] = *reinterpret_cast<const v4f *>(qb + row);
    }
    const int64_t hc = h * a.nch + ch;
    r.v = *reinterpret_cast<const float *>(vb + (uint64_t)(uint32_t)min(t0 + vr, Tm1) * vrow);
    r.tp = reinterpret_cast<const v2f *>(a.tw + hc * MAT)[tid];
    r.pt = reinterpret_cast<const v2f *>(a.pw + hc * MAT)[tid];
    r.l = a.lw[hc * GC + (lane & (GC - 1))];
  };
  // to LDS: K and Q of chunk ch
  auto stage_kq = [&](int ch, const ChunkRegs<DK> &r) {
    float(*const Kb)[DKP] = Ks[ch & 1];
#pragma unroll
    for (int u = 0; u < KF; u++) {
      *reinterpret_cast<v4f *>(&Kb[kr + u * RPP][4 * kc]) = r.k[u];
      *reinterpret_cast<v4f *>(&Qs[ch & 1][kr + u * RPP][4 * kc]) = r.q[u];
    }
  };
  // ... and what its phase 2 reads, with the state before it
  auto stage_rest = [&](int ch, const ChunkRegs<DK> &r, float el, float dl) {
    *reinterpret_cast<v2f *>(&Tp[tid >> 4][2 * (tid & 15)]) = r.tp;
    *reinterpret_cast<v2f *>(&PT[tid >> 4][2 * (tid & 15)]) = r.pt;
    Vt[vc][vr] = r.v;
    if (wave == 4 && lane < GC) {
      eLs[lane] = el;
      dLs[lane] = dl;
    }
    if (wave < NT) *reinterpret_cast<v4f *>(&St[ch & 1][n][16 * wave + 4 * gq]) = S;
  };
  // e^L and e^{L_C - L} (wave 4; the whole wave: the shuffle's source lane)
  auto decays = [&](const ChunkRegs<DK> &r, float &el, float &dl) {
    el = expf(r.l);
    dl = expf(__shfl(r.l, GC - 1) - r.l);
  };
  // out of this lane's tokens 16 (wave % 2) + 4 gq .. + 3 of the chunk
  float *op = a.out + ((16 * (wave & 1) + 4 * gq) * a.NH + h) * a.DV + cb + n;
  const int64_t orow = a.NH * a.DV;
  // nx holds chunk ch + 1's inputs; once they are in LDS it takes chunk ch + 3
  auto chunk_step = [&](int ch, ChunkRegs<DK> &nx) {
    const float(*const Kb)[DKP] = Ks[ch & 1];
    const float(*const Sb)[DKP] = St[ch & 1];
    const int tt = wave & 1, tk = 16 * tt + 4 * gq;
    __syncthreads();
    {
      const int arow = 16 * tt + n, kq = wave >> 1;
      v4f x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0;
#pragma unroll
      for (int kb = 0; kb < KQ; kb += 16) {
        const int k0 = KQ * kq + kb + 4 * gq;
        mm4(quad(&Kb[arow][k0]), quad(&Sb[n][k0]), x0, x1);
      }
      *reinterpret_cast<v4f *>(&Xp[kq][n][tk]) = x0 + x1;
    }
    __syncthreads();
    float el = 0.0f, dl = 0.0f;
    v4f o = {0.f, 0.f, 0.f, 0.f}, dl4 = o;     // waves 2, 3: (P T') W and e^L
    if (wave < 4) {
      const float(*const A)[MP] = wave < 2 ? Tp : PT;
      v4f c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
#pragma unroll
      for (int kb = 0; kb < GC; kb += 16) {
        const int j = kb + 4 * gq;
        const float4 xa = quad(&Xp[0][n][j]), xb = quad(&Xp[1][n][j]), xc = quad(&Xp[2][n][j]),
                     xd = quad(&Xp[3][n][j]), v = quad(&Vt[n][j]), e4 = quad(&eLs[j]);
        const float4 w = make_float4(v.x - e4.x * ((xa.x + xb.x) + (xc.x + xd.x)),
                                     v.y - e4.y * ((xa.y + xb.y) + (xc.y + xd.y)),
                                     v.z - e4.z * ((xa.z + xb.z) + (xc.z + xd.z)),
                                     v.w - e4.w * ((xa.w + xb.w) + (xc.w + xd.w)));
        mm4(quad(&A[16 * tt + n][j]), w, c0, c1);
      }
      o = c0 + c1;
      if (wave < 2)
        *reinterpret_cast<v4f *>(&Ut[n][tk]) = *reinterpret_cast<const v4f *>(&dLs[tk]) * o;
      else
        dl4 = *reinterpret_cast<const v4f *>(&eLs[tk]);
    } else {
      const int arow = 16 * tt + n, kh = (wave >> 1) & 1;
      v4f y0 = {0.f, 0.f, 0.f, 0.f}, y1 = y0;
#pragma unroll
      for (int kb = 0; kb < DK / 2; kb += 16) {
        const int k0 = DK / 2 * kh + kb + 4 * gq;
        mm4(quad(&Qs[ch & 1][arow][k0]), quad(&Sb[n][k0]), y0, y1);
      }
      *reinterpret_cast<v4f *>(&Yp[kh][n][tk]) = y0 + y1;
      if (wave == 4) decays(nx, el, dl);
    }
    stage_kq(ch + 1, nx);
    const float eC = eLs[GC - 1];
    __syncthreads();
    if (wave < NT) {
      S *= eC;
      v4f S1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < GC; kb += 16) {
        const int j = kb + 4 * gq;
        mm4(make_float4(Kb[j][16 * wave + n], Kb[j + 1][16 * wave + n], Kb[j + 2][16 * wave + n],
                        Kb[j + 3][16 * wave + n]),
            quad(&Ut[n][j]), S, S1);
      }
      S += S1;
    }
    if (wave == 2 || wave == 3) {
      const v4f ya = *reinterpret_cast<const v4f *>(&Yp[0][n][tk]),
                yb = *reinterpret_cast<const v4f *>(&Yp[1][n][tk]);
      o += dl4 * (ya + yb);
      const int left = (int)min((int64_t)4, a.T - (int64_t)ch * GC - tk);
      if (col) {
        if (left > 0) op[0] = o[0];
        if (left > 1) op[orow] = o[1];
        if (left > 2) op[2 * orow] = o[2];
        if (left > 3) op[3 * orow] = o[3];
      }
    }
    op += GC * orow;
    stage_rest(ch + 1, nx, el, dl);
    load(min(ch + 3, a.nch - 1), nx);
  };
  // (past the last chunk the last one is loaded and staged again, unused)
  ChunkRegs<DK> na, nb;
  load(0, nb);
  load(min(1, a.nch - 1), na);
  asm volatile("" : "+v"(S));            // S has landed: no wait for it inside the loop
  {
    float el = 0.0f, dl = 0.0f;
    stage_kq(0, nb);
    if (wave == 4) decays(nb, el, dl);
    stage_rest(0, nb, el, dl);
    load(min(2, a.nch - 1), nb);
  }
  for (int ch = 0;;) {
    chunk_step(ch, na);
    if (++ch >= a.nch) break;
    chunk_step(ch, nb);
    if (++ch >= a.nch) break;
  }
  if (a.s_out && wave < NT && col) {
#pragma unroll
    for (int e = 0; e < 4; e++) a.s_out[(h * DK + 16 * wave + 4 * gq + e) * a.DV + cb + n] = S[e];
  }
}

// A few tokens (decode) step by step, the recurrence as written: per token,
// d = k^T S and o = S^T q reduced over the rows (8 neighbouring lanes by DPP,
// the four waves through LDS), S <- a (S - b k d^T) + b k v^T in between.
// 8 value columns per workgroup, DK/32 rows per thread.
template <int DK>
__global__ __launch_bounds__(GNT) void gdn_step_kernel(GdnArgs a) {
  constexpr int RPT = DK / (GNT / STC);
  __shared__ float red[2][GNT / 64][STC];
  const int tid = threadIdx.x;
  const int nsl = (int)(a.DV / STC);
  const int64_t h = blockIdx.x / nsl;
  const int cb = (int)(blockIdx.x % nsl) * STC;
  const int wave = tid >> 6, part = tid & 7;
  const int c = (tid >> 3) & (STC - 1), r0 = (8 * wave + part) * RPT;
  float S[RPT];
#pragma unroll
  for (int m = 0; m < RPT; m++)
    S[m] = a.s0 ? a.s0[(h * DK + r0 + m) * a.DV + cb + c] : 0.0f;
  for (int64_t t = 0; t < a.T; t++) {
    const int64_t tk = (t * a.NH + h) * DK + r0;
    float kr[RPT], qr[RPT];
#pragma unroll
    for (int m = 0; m < RPT; m += 2) {
      const float2 k2 = *reinterpret_cast<const float2 *>(a.k + tk + m);
      const float2 q2 = *reinterpret_cast<const float2 *>(a.q + tk + m);
      kr[m] = k2.x; kr[m + 1] = k2.y;
      qr[m] = q2.x; qr[m + 1] = q2.y;
    }
    const float vc = a.v[(t * a.NH + h) * a.DV + cb + c];
    const float al = expf(a.g[t * a.NH + h]), be = a.beta[t * a.NH + h];
    float dp = 0.0f;
#pragma unroll
    for (int m = 0; m < RPT; m++) dp = fmaf(kr[m], S[m], dp);
    dp = sum8(dp);
    if (part == 0) red[0][wave][c] = dp;
    __syncthreads();
    float d = 0.0f;
#pragma unroll
    for (int w = 0; w < GNT / 64; w++) d += red[0][w][c];
    float op = 0.0f;
#pragma unroll
    for (int m = 0; m < RPT; m++) {
      S[m] = al * (S[m] - be * kr[m] * d) + be * kr[m] * vc;
      op = fmaf(qr[m], S[m], op);
    }
    op = sum8(op);
    if (part == 0) red[1][wave][c] = op;
    __syncthreads();
    if (tid < STC) {
      float o = 0.0f;
#pragma unroll
      for (int w = 0; w < GNT / 64; w++) o += red[1][w][tid];
      a.out[(t * a.NH + h) * a.DV + cb + tid] = o;
    }
    __syncthreads();                       // red is rewritten for the next token
  }
  if (a.s_out) {
#pragma unroll
    for (int m = 0; m < RPT; m++) a.s_out[(h * DK + r0 + m) * a.DV + cb + c] = S[m];
  }
}

int gdn_validate(int64_t T, int64_t NH, int64_t DK, int64_t DV) {
  if (T < 0 || NH <= 0 || DV <= 0 || DV % STC != 0 || (DK != 64 && DK != 128)) return W4A8_ESHAPE;
  if (T >= ((int64_t)1 << 31) || NH >= (1 << 16) || DV > 4096) return W4A8_ERANGE;
  const int64_t nch = (T + GC - 1) / GC;
  if (nch * NH >= ((int64_t)1 << 31) || T * NH * (DK > DV ? DK : DV) >= ((int64_t)1 << 40))
    return W4A8_ERANGE;
  return W4A8_OK;
}

}  // namespace

}  // namespace w4a8

using namespace w4a8;

extern "C" size_t gdn_workspace_size(int64_t T, int64_t NH, int64_t DK, int64_t DV) {
  if (gdn_validate(T, NH, DK, DV) != W4A8_OK) return 0;
  const int64_t nch = (T + GC - 1) / GC;
  return 2 * up256(sizeof(float) * (size_t)(NH * nch) * MAT) +
         up256(sizeof(float) * (size_t)(NH * nch) * GC) + 256;
}

extern "C" int gdn_chunked_scan(const float *q, const float *k, const float *v, const float *g,
                                const float *beta, const float *s0, float *out, float *s_out,
                                int64_t T, int64_t NH, int64_t DK, int64_t DV, void *workspace,
                                size_t ws_bytes, void *stream) {
  int rc = gdn_validate(T, NH, DK, DV);
  if (rc != W4A8_OK) return rc;
  if (T == 0 && !s_out) return W4A8_OK;
  if (!q || !k || !v || !g || !beta || !out || !workspace) return W4A8_ENULL;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(s0) ||
      !aligned16(s_out) || !aligned16(workspace) || (reinterpret_cast<uintptr_t>(g) & 3) ||
      (reinterpret_cast<uintptr_t>(beta) & 3))
    return W4A8_EALIGN;
  if (ws_bytes < gdn_workspace_size(T, NH, DK, DV)) return W4A8_EWORKSPACE;
  if ((rc = check_device()) != W4A8_OK) return rc;
  hipStream_t s = as_stream(stream);
  const int64_t nch = (T + GC - 1) / GC;
  uint8_t *ws = reinterpret_cast<uint8_t *>(workspace);
  GdnArgs a{};
  a.q = q; a.k = k; a.v = v; a.g = g; a.beta = beta; a.s0 = s0;
  a.out = out; a.s_out = s_out;
  a.tw = reinterpret_cast<float *>(ws);
  a.pw = reinterpret_cast<float *>(ws + up256(sizeof(float) * (size_t)(NH * nch) * MAT));
  a.lw = reinterpret_cast<float *>(ws + 2 * up256(sizeof(float) * (size_t)(NH * nch) * MAT));
  a.T = T; a.NH = NH; a.DV = DV; a.nch = (int)nch;
  if (T <= GDN_STEP_T) {                      // a few tokens: the recurrence step by step
    const unsigned nwg = (unsigned)(NH * (DV / STC));
    if (DK == 128)
      gdn_step_kernel<128><<<dim3(nwg), dim3(GNT), 0, s>>>(a);
    else
      gdn_step_kernel<64><<<dim3(nwg), dim3(GNT), 0, s>>>(a);
    return check_launch();
  }
  if (nch > 0) {
    if (DK == 128)
      gdn_prep_kernel<128><<<dim3((unsigned)(NH * nch)), dim3(GNT), 0, s>>>(a);
    else
      gdn_prep_kernel<64><<<dim3((unsigned)(NH * nch)), dim3(GNT), 0, s>>>(a);
    if ((rc = check_launch()) != W4A8_OK) return rc;
  }
  const unsigned nwg = (unsigned)(NH * ((DV + DVS - 1) / DVS));   // T > GDN_STEP_T: nch >= 1
  if (DK == 128)
    gdn_scan_kernel<128><<<dim3(nwg), dim3(SNT), 0, s>>>(a);
  else
    gdn_scan_kernel<64><<<dim3(nwg), dim3(SNT), 0, s>>>(a);
  return check_launch();
}
