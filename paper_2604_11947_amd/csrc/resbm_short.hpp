// Kernels of the one-linear ops for calls whose T x n streams are short (bf16
// build): one pass of a block over its tile, no software pipeline.
//
// The streaming kernels hold one block per compute unit and start their loops
// two or three empty steps early, which a long token range hides.  With few
// tokens they leave most units idle (encode_fwd: one 64-token block walks all
// of n) or run more empty steps than full ones (decode_bwd, encode_bwd).  The
// kernels here cut both dimensions into tiles instead, several blocks per unit,
// and rely on the other blocks of the unit to cover a block's loads.
#pragma once

namespace resbm {

#if !RESBM_IO_F32_BUILD

// 8 elements of a stream.  Default cache policy: a short stream is still in the
// last-level cache when its producer wrote it just before (T = 8192, n = 2048:
// 13.6 -> 11.0 us for encode_fwd, 22.6 -> 19.5 for encode_bwd against the
// non-temporal loads of the long streams; stores measured alike either way).
__device__ __forceinline__ XFrag bld_s8(rsrc_t r, uint32_t off) {
  return XFrag{__builtin_bit_cast(bf16x8, bld16(r, off))};
}

// ------------------------------------------------------------ encode forward
// Partial a = z W_e of 16 MT tokens (blockIdx.x), the 64-column units of slice
// blockIdx.y of n, and j-tiles [JT blockIdx.z, ...) of r.  The 8 waves take the
// slice's units in turn; a wave splits its unit's 64 rows of W_e into hi / lo
// planes of its own LDS region and reads them back transposed (no barrier, and
// no prologue kernel: a block splits only its slice).  Their sums meet in LDS
// in wave order.  One slice: the epilogue is applied here; several: the partials
// go to part[slice][T][RP] and k_enc_fwd_fin adds them in slice order.
template <int JT, int MT>
__global__ __launch_bounds__(512) void k_enc_fwd_short(int64_t T, int n, int r, int RP, int act,
                                                       const io_t* __restrict__ x_attn, int64_t ld_x,
                                                       const io_t* __restrict__ z, int64_t ld_z,
                                                       const float* __restrict__ W_e, io_t* __restrict__ b,
                                                       float* __restrict__ a_save, float* __restrict__ part) {
  constexpr int KW = 8, RPT = 16 * JT, TOK = 16 * MT;
  constexpr int WLL = RPT / 4, WRPI = 64 / WLL, WQ = 64 / WRPI;  // W_e: lanes per row, rows per load, loads per unit
  constexpr int WPL = 64 * RPT;                                  // elements of one plane
  constexpr int RPITCH = RPT + 4;
  constexpr int WBYTES = KW * 2 * WPL * 2, RED = KW * TOK * RPITCH * 4;
  __shared__ __attribute__((aligned(16))) char smem[WBYTES > RED ? WBYTES : RED];
  const int l = lane_id(), row16 = l & 15, grp = l >> 4, wave = wave_id();
  const int64_t tok0 = (int64_t)blockIdx.x * TOK;
  const int jb = blockIdx.z * RPT;
  const int nu = n / 64;
  const int u0 = (int)((int64_t)blockIdx.y * nu / gridDim.y), u1 = (int)((int64_t)(blockIdx.y + 1) * nu / gridDim.y);
  const rsrc_t zr = make_rsrc(z + tok0 * ld_z, rows_bytes(min((int64_t)TOK, T - tok0), n, ld_z, kEs));
  const rsrc_t we = make_rsrc(W_e, (int64_t)n * r * 4);
  __bf16* const ph = reinterpret_cast<__bf16*>(smem) + wave * 2 * WPL;
  __bf16* const pl = ph + WPL;
  const int wcol = 4 * (l % WLL), wrow = l / WLL;
  const bool won = jb + wcol < r;

  f32x4 acc[MT][JT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) acc[mt][jt] = f32x4{0.f, 0.f, 0.f, 0.f};

  XFrag zf[MT][2];
  uint4 wq[WQ];
  auto load = [&](int u) {
    const bool on = u < u1;
#pragma unroll
    for (int q = 0; q < WQ; ++q)
      wq[q] = bld16(we, on && won ? (uint32_t)(((64 * u + q * WRPI + wrow) * r + jb + wcol) * 4) : kOOB);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        zf[mt][ks] = bld_s8(zr, on ? (uint32_t)(((16 * mt + row16) * ld_z + 64 * u + 32 * ks + 8 * grp) * kEs) : kOOB);
  };
  load(u0 + wave);
  for (int u = u0 + wave; u < u1; u += KW) {
#pragma unroll
    for (int q = 0; q < WQ; ++q) {
      const int row = q * WRPI + wrow;
      const float f4[4] = {__builtin_bit_cast(float, wq[q].x), __builtin_bit_cast(float, wq[q].y),
                           __builtin_bit_cast(float, wq[q].z), __builtin_bit_cast(float, wq[q].w)};
      bf16x4 h, lo;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        __bf16 a, c;
        split_hi_lo(f4[e], a, c);
        h[e] = a;
        lo[e] = c;
      }
      const int pos = row * RPT + tile_col<RPT>(row, wcol);
      *reinterpret_cast<uint2*>(ph + pos) = __builtin_bit_cast(uint2, h);
      *reinterpret_cast<uint2*>(pl + pos) = __builtin_bit_cast(uint2, lo);
    }
    XFrag zc[MT][2];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) zc[mt][ks] = zf[mt][ks];
    load(u + KW);
    wave_lds_fence();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        SFrag w;
        w.hi = tr_plane<RPT>(ph, 32 * ks, 16 * jt, row16, grp);
        w.lo = tr_plane<RPT>(pl, 32 * ks, 16 * jt, row16, grp);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt][jt] = mma_sx(w, zc[mt][ks], acc[mt][jt]);
      }
    wave_lds_fence();  // the planes are read before the next unit overwrites them
  }
  __syncthreads();  // the reduction area overlaps the planes
  float (*s_red)[TOK][RPITCH] = reinterpret_cast<float (*)[TOK][RPITCH]>(smem);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
      *reinterpret_cast<float4*>(&s_red[wave][16 * mt + row16][16 * jt + 4 * grp]) =
          make_float4(acc[mt][jt][0], acc[mt][jt][1], acc[mt][jt][2], acc[mt][jt][3]);
  __syncthreads();
  constexpr int Q = RPT / 4;
  for (int idx = threadIdx.x; idx < TOK * Q; idx += KW * 64) {
    const int tt = idx / Q, jj = (idx % Q) * 4, j0 = jb + jj;
    const int64_t t = tok0 + tt;
    if (t >= T || j0 >= r) continue;
    float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < KW; ++w) {
      const float4 p = *reinterpret_cast<const float4*>(&s_red[w][tt][jj]);
      a[0] += p.x; a[1] += p.y; a[2] += p.z; a[3] += p.w;
    }
    if (gridDim.y > 1) {
      *reinterpret_cast<float4*>(part + ((int64_t)blockIdx.y * T + t) * RP + j0) = make_float4(a[0], a[1], a[2], a[3]);
      continue;
    }
    if (a_save) *reinterpret_cast<float4*>(a_save + t * r + j0) = make_float4(a[0], a[1], a[2], a[3]);
    float x[4], o[4];
    load_x4(x_attn + t * ld_x + j0, x);
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = x[v] + act_phi(a[v], act);
    store_x4(b + t * r + j0, o);
  }
}

// a = the slices' partials in order; a_save = a, b = x_attn[:, :r] + phi(a).
__global__ __launch_bounds__(64) void k_enc_fwd_fin(int64_t T, int r, int RP, int act, int nsl,
                                                    const float* __restrict__ part, const io_t* __restrict__ x_attn,
                                                    int64_t ld_x, io_t* __restrict__ b, float* __restrict__ a_save) {
  const int nq = r / 4;
  const int64_t gid = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (gid >= T * nq) return;
  const int64_t t = gid / nq;
  const int j0 = (int)(gid % nq) * 4;
  float x[4], o[4];
  load_x4(x_attn + t * ld_x + j0, x);
  const float4 p = sum_ordered4(part + t * RP + j0, T * RP, nsl);
  const float a[4] = {p.x, p.y, p.z, p.w};
  if (a_save) *reinterpret_cast<float4*>(a_save + t * r + j0) = p;
#pragma unroll
  for (int v = 0; v < 4; ++v) o[v] = x[v] + act_phi(a[v], act);
  store_x4(b + t * r + j0, o);
}

// ------------------------------------------------------------ backward tiles
// 64 tokens x 256 columns per step of a block of 8 waves, nstep steps of
// consecutive tokens per block.
constexpr int kOnceTS = 64, kOnceBC = 256;

// The tile of TS rows x BC columns at token t0 that a block of 8 waves loads
// (this lane's 16-byte pieces): piece q is row (512 q + threadIdx) / (BC / 8),
// columns 8 (threadIdx % (BC / 8)) .. + 7; zeros outside.
template <int TS, int BC>
__device__ __forceinline__ void once_load(XFrag (&v)[TS * BC / 4096], const io_t* x, int64_t ld, int64_t t0, int64_t T,
                                          int bc0, int bcv) {
  constexpr int LPR = BC / 8;
  const rsrc_t xr = make_rsrc(x + t0 * ld + bc0, rows_bytes(min((int64_t)TS, T - t0), bcv, ld, kEs));
  const int row = threadIdx.x / LPR, c = 8 * (threadIdx.x % LPR);
#pragma unroll
  for (int q = 0; q < TS * BC / 4096; ++q)
    v[q] = bld_s8(xr, c < bcv ? (uint32_t)(((row + q * (512 / LPR)) * ld + c) * kEs) : kOOB);
}
template <int TS, int BC>
__device__ __forceinline__ void once_put(io_t* tile, const XFrag (&v)[TS * BC / 4096]) {
  constexpr int LPR = BC / 8;
#pragma unroll
  for (int q = 0; q < TS * BC / 4096; ++q) {
    const int row = threadIdx.x / LPR + q * (512 / LPR);
    *reinterpret_cast<uint4*>(tile + row * BC + wide_col(row, 8 * (threadIdx.x % LPR))) =
        __builtin_bit_cast(uint4, v[q].v);
  }
}

// What bounds them: at 1024 x 4096 a block has one step, so its time is a chain
// of launch, load, split, two barriers and stores (about 7 us of k_enc_bwd_once's
// 11.8 with one token tile, 7.0 at T = 8) plus the partial sums' way out, as
// many bytes as the tiles at r = 32.  512 x 32 tiles (half of the g_b partials)
// were slower: 21.6 against 18.9 us at T = 2048, n = 4096, r = 32.

// decode_bwd for j-tiles [JT blockIdx.z, ...) of r: g_b partials of the block's columns (wave (cw, tw): a quarter
// of the columns, half of the tokens; the four column parts meet in LDS in order) and dW_d
// partials of the block's tokens (wave: an eighth of the columns).  Finished by k_dec_bwd_fin.
template <int JT>
__global__ __launch_bounds__(512) void k_dec_bwd_once(int64_t T, int n, int r, int RP, const io_t* __restrict__ b,
                                                      const float* __restrict__ W_d, const io_t* __restrict__ g_zt,
                                                      int64_t ld_g, float* __restrict__ gbp,
                                                      float* __restrict__ dwp, int nstep) {
  constexpr int RPT = 16 * JT, TS = kOnceTS, BC = kOnceBC, BQ = RPT / 8;
  constexpr int KSW = BC / 128, MTW = TS / 32;  // a wave's part of g_b: 32 KSW columns x 16 MTW tokens
  constexpr int CTW = BC / 128, KST = TS / 32;  // ... and of dW_d: 16 CTW columns, 32 KST tokens
  __shared__ __attribute__((aligned(16))) io_t s_g[TS * BC];
  __shared__ __attribute__((aligned(16))) io_t s_b[TS * RPT];
  __shared__ __attribute__((aligned(16))) float s_p[4][TS * gb_rowsz<RPT>()];
  const int l = lane_id(), row16 = l & 15, grp = l >> 4, wave = wave_id();
  const int cw = wave & 3, tw = wave >> 2;
  const int tg = blockIdx.x, cg = blockIdx.y, bc0 = cg * BC, bcv = min(BC, n - bc0);
  const int jb = blockIdx.z * RPT;
  const int64_t tb = (int64_t)tg * nstep * TS;
  const bool bthr = threadIdx.x < TS * BQ;
  const int btt = bthr ? threadIdx.x / BQ : 0, bch = threadIdx.x % BQ;

  XFrag gv[TS * BC / 4096], bv;
  auto load = [&](int s) {
    const int64_t t0 = tb + (int64_t)s * TS;  // steps past the range see no rows
    once_load<TS, BC>(gv, g_zt, ld_g, s < nstep ? t0 : T, T, bc0, bcv);
    const int64_t rows = s < nstep ? min((int64_t)TS, T - t0) : 0;
    const rsrc_t br = make_rsrc(b + t0 * r, rows * r * kEs);
    bv = bld_r8(br, bthr ? (uint32_t)(btt * r * kEs) : kOOB, r, jb + 8 * bch);
  };
  load(0);
  const rsrc_t wr = make_rsrc(W_d, (int64_t)r * n * 4);
  SFrag wdf[JT][KSW];  // W_d[jb + 16 jt + row16][bc0 + 32 KSW cw + 32 ks + 8 grp + e]
#pragma unroll
  for (int jt = 0; jt < JT; ++jt)
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks) {
      const int j = jb + 16 * jt + row16, c = bc0 + 32 * KSW * cw + 32 * ks + 8 * grp;
      const bool ok = j < r && c < n;
      const uint32_t o = (uint32_t)((j * n + c) * 4);
      const uint4 a = bld16(wr, ok ? o : kOOB), d = bld16(wr, ok ? o + 16 : kOOB);
      const float w[8] = {__builtin_bit_cast(float, a.x), __builtin_bit_cast(float, a.y),
                          __builtin_bit_cast(float, a.z), __builtin_bit_cast(float, a.w),
                          __builtin_bit_cast(float, d.x), __builtin_bit_cast(float, d.y),
                          __builtin_bit_cast(float, d.z), __builtin_bit_cast(float, d.w)};
      wdf[jt][ks] = sfrag_from(w);
    }
  f32x4 dw[CTW][JT];
#pragma unroll
  for (int ct = 0; ct < CTW; ++ct)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) dw[ct][jt] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int s = 0; s < nstep; ++s) {
    const int64_t t0 = tb + (int64_t)s * TS;
    if (t0 >= T) break;  // uniform over the block
    // the previous step's readers of the tile passed its second barrier
    once_put<TS, BC>(s_g, gv);
    if (bthr) tile_put8<RPT>(s_b, btt, 8 * bch, bv);
    load(s + 1);
    __syncthreads();
#pragma unroll
    for (int th = 0; th < MTW; ++th) {
      const int row = 16 * MTW * tw + 16 * th + row16;
      XFrag f[KSW];
#pragma unroll
      for (int ks = 0; ks < KSW; ++ks)
        f[ks].v = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(
                                                 s_g + row * BC + wide_col(row, 32 * KSW * cw + 32 * ks + 8 * grp)));
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KSW; ++ks) acc = mma_sx(wdf[jt][ks], f[ks], acc);
        *reinterpret_cast<float4*>(&s_p[cw][gb_pos<RPT>(row, 16 * jt + 4 * grp)]) =
            make_float4(acc[0], acc[1], acc[2], acc[3]);
      }
    }
#pragma unroll
    for (int ks = 0; ks < KST; ++ks) {
      XFrag bt[JT];
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) bt[jt] = tr_frag<RPT>(s_b + 32 * ks * RPT, 16 * jt, row16, grp);
#pragma unroll
      for (int ct = 0; ct < CTW; ++ct) {
        const XFrag a = tr_frag_wide<BC>(s_g, 32 * ks, 16 * CTW * wave + 16 * ct, row16, grp);
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) dw[ct][jt] = mma_xx(a, bt[jt], dw[ct][jt]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int idx0 = 0; idx0 < TS * RPT / 4; idx0 += 512) {
      const int idx = idx0 + threadIdx.x;
      const int tt = idx / (RPT / 4), j = 4 * (idx % (RPT / 4));
      if (idx < TS * RPT / 4 && t0 + tt < T && jb + j < r) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float4 p = *reinterpret_cast<const float4*>(&s_p[w][gb_pos<RPT>(tt, j)]);
          v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
        }
        *reinterpret_cast<float4*>(gbp + ((int64_t)cg * T + t0 + tt) * RP + jb + j) = v;
      }
    }
  }
  // dw[ct][jt][v] = dW_d partial [jb + 16 jt + row16][bc0 + 16 CTW wave + 16 ct + 4 grp + v]
  const int c0 = bc0 + 16 * CTW * wave;
  if (c0 >= n) return;
#pragma unroll
  for (int jt = 0; jt < JT; ++jt) {
    const int j = jb + 16 * jt + row16;
    if (j >= r) continue;
#pragma unroll
    for (int ct = 0; ct < CTW; ++ct)
      *reinterpret_cast<float4*>(dwp + ((int64_t)tg * RP + j) * n + c0 + 16 * ct + 4 * grp) =
          make_float4(dw[ct][jt][0], dw[ct][jt][1], dw[ct][jt][2], dw[ct][jt][3]);
  }
}

// encode_bwd, r <= 64, in one pass over z and g_z: g_h = g_b phi'(a) split in
// LDS, dW_e partials of the block's tokens and g_z of its tile (a wave: 32
// columns of either; ADD: + g_b I_{r x n}), g_z leaving through LDS as whole 512-byte row segments.
// Finished by k_enc_bwd_fin.
template <int JT, bool ADD>
__global__ __launch_bounds__(512) void k_enc_bwd_once(int64_t T, int n, int r, int RP, int silu,
                                                      const io_t* __restrict__ z, int64_t ld_z,
                                                      const float* __restrict__ W_e,
                                                      const float* __restrict__ a_save,
                                                      const io_t* __restrict__ g_b, io_t* __restrict__ g_z,
                                                      int64_t ld_gz, float* __restrict__ dwp, int nstep) {
  constexpr int KS = (JT + 1) / 2, KP = 32 * KS, TS = kOnceTS, BC = kOnceBC;
  constexpr int NCH = TS * KP / 4 / 512;  // 4-column pieces of g_h per thread
  __shared__ __attribute__((aligned(16))) io_t s_z[TS * BC];
  __shared__ __attribute__((aligned(16))) io_t s_o[TS * BC];
  __shared__ __attribute__((aligned(16))) GhTile<TS, KP> s_gh;
  const int l = lane_id(), row16 = l & 15, grp = l >> 4, wave = wave_id();
  const int tg = blockIdx.x, bc0 = blockIdx.y * BC, bcv = min(BC, n - bc0);
  const int c0 = bc0 + 32 * wave;  // this wave's columns: whole inside or outside [0, n)
  const int64_t tb = (int64_t)tg * nstep * TS;

  XFrag zv[TS * BC / 4096];
  uint2 gbv[NCH];
  uint4 av[NCH];
  uint2 iv[ADD ? TS / 16 : 1][2];  // ADD: g_b at this lane's 8 columns of g_z, zeros at or beyond r
  auto load = [&](int s) {
    const int64_t t0 = tb + (int64_t)s * TS;
    const int64_t rows = s < nstep ? min((int64_t)TS, T - t0) : 0;
    once_load<TS, BC>(zv, z, ld_z, s < nstep ? t0 : T, T, bc0, bcv);
    const rsrc_t gbr = make_rsrc(g_b + t0 * r, rows * r * kEs);
    const rsrc_t ar = make_rsrc(silu ? a_save + t0 * r : a_save, silu ? rows * r * 4 : 0);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int q = threadIdx.x + 512 * i, tt = q / (KP / 4), j = 4 * (q % (KP / 4));
      gbv[i] = bld8(gbr, j < r ? (uint32_t)((tt * r + j) * kEs) : kOOB);
      av[i] = bld16(ar, j < r ? (uint32_t)((tt * r + j) * 4) : kOOB);
    }
    if constexpr (ADD) {
#pragma unroll
      for (int mt = 0; mt < TS / 16; ++mt)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int c = c0 + 8 * grp + 4 * h;
          iv[mt][h] = bld8(gbr, c < r ? (uint32_t)(((16 * mt + row16) * r + c) * kEs) : kOOB);
        }
    }
  };
  load(0);
  const rsrc_t wr = make_rsrc(W_e, (int64_t)n * r * 4);
  SFrag wf[KS][2];  // W_e[expand_col(c0, ct, row16)][32 ks + 8 grp + e]
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      const int col = expand_col<2>(c0, ct, row16), k = 32 * ks + 8 * grp;
      const uint32_t o = (uint32_t)((col * r + k) * 4);
      const uint4 a = bld16(wr, c0 < n && k < r ? o : kOOB), d = bld16(wr, c0 < n && k + 4 < r ? o + 16 : kOOB);
      const float w[8] = {__builtin_bit_cast(float, a.x), __builtin_bit_cast(float, a.y),
                          __builtin_bit_cast(float, a.z), __builtin_bit_cast(float, a.w),
                          __builtin_bit_cast(float, d.x), __builtin_bit_cast(float, d.y),
                          __builtin_bit_cast(float, d.z), __builtin_bit_cast(float, d.w)};
      wf[ks][ct] = sfrag_from(w);
    }
  f32x4 dw[2][JT];
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) dw[ct][jt] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int s = 0; s < nstep; ++s) {
    const int64_t t0 = tb + (int64_t)s * TS;
    if (t0 >= T) break;  // uniform over the block
    // the previous step's readers of the tile and of g_h passed its second barrier
    once_put<TS, BC>(s_z, zv);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int q = threadIdx.x + 512 * i, tt = q / (KP / 4), j = 4 * (q % (KP / 4));
      const float gb4[4] = {bf16_bits_to_f32(gbv[i].x & 0xffffu), bf16_bits_to_f32(gbv[i].x >> 16),
                            bf16_bits_to_f32(gbv[i].y & 0xffffu), bf16_bits_to_f32(gbv[i].y >> 16)};
      const float a4[4] = {__builtin_bit_cast(float, av[i].x), __builtin_bit_cast(float, av[i].y),
                           __builtin_bit_cast(float, av[i].z), __builtin_bit_cast(float, av[i].w)};
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = silu ? gb4[e] * silu_grad(a4[e]) : gb4[e];
      gh_put4(s_gh, tt, j, v);
    }
    uint2 id[ADD ? TS / 16 : 1][2];
    if constexpr (ADD) {
#pragma unroll
      for (int mt = 0; mt < TS / 16; ++mt)
#pragma unroll
        for (int h = 0; h < 2; ++h) id[mt][h] = iv[mt][h];
    }
    load(s + 1);
    __syncthreads();
    // dW_e: D[j][c] = sum_t g_h[t][j] z[t][c]
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      XFrag zb[2];
#pragma unroll
      for (int ct = 0; ct < 2; ++ct) zb[ct] = tr_frag_wide<BC>(s_z, 32 * ks, 32 * wave + 16 * ct, row16, grp);
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        const SFrag g = gh_tr(s_gh, 32 * ks, 16 * jt, row16, grp);
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) dw[ct][jt] = mma_sx(g, zb[ct], dw[ct][jt]);
      }
    }
    // g_z: D[c][t] = sum_j W_e[c][j] g_h[t][j]
#pragma unroll
    for (int mt = 0; mt < TS / 16; ++mt) {
      const int row = 16 * mt + row16;
      f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        SFrag g;
        const int pc = lds_col<KP>(row, 32 * ks + 8 * grp);
        g.hi = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&s_gh.hi[row][pc]));
        g.lo = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&s_gh.lo[row][pc]));
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) acc[ct] = mma_ss(wf[ks][ct], g, acc[ct]);
      }
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = acc[e >> 2][e & 3];
      // (no branch here: behind one the compiler of ROCm 7.2 read the products
      // before their registers were written)
      if constexpr (ADD) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t u = e & 2 ? id[mt][e >> 2].y : id[mt][e >> 2].x;
          v[e] += bf16_bits_to_f32(e & 1 ? u >> 16 : u & 0xffffu);
        }
      }
      bf16x8 h;
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = to_bf16(v[e]);
      *reinterpret_cast<uint4*>(s_o + row * BC + wide_col(row, 32 * wave + 8 * grp)) = __builtin_bit_cast(uint4, h);
    }
    __syncthreads();
    const rsrc_t gr = make_rsrc(g_z + t0 * ld_gz + bc0, rows_bytes(min((int64_t)TS, T - t0), bcv, ld_gz, kEs));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = 8 * wave + 2 * q + (l >> 5), c = 8 * (l & 31);
      bst16<kStStream>(gr, c < bcv ? (uint32_t)((row * ld_gz + c) * kEs) : kOOB,
                       *reinterpret_cast<const uint4*>(s_o + row * BC + wide_col(row, c)));
    }
  }
  // dw[ct][jt][v] = partial dW_e[c0 + 16 ct + row16][16 jt + 4 grp + v]
  if (c0 >= n) return;
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
      if (16 * jt < RP)
        *reinterpret_cast<float4*>(dwp + ((int64_t)tg * n + c0 + 16 * ct + row16) * RP + 16 * jt + 4 * grp) =
            make_float4(dw[ct][jt][0], dw[ct][jt][1], dw[ct][jt][2], dw[ct][jt][3]);
}

#endif  // !RESBM_IO_F32_BUILD

}  // namespace resbm
