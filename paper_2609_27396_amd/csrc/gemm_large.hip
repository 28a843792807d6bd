// bf16 projections over more than 64 rows: persistent, software-pipelined GEMMs.
//
// More than 320 rows (gemm_large_kernel).
// What bounds a 256 x 256 tile on a CU, per 64-deep K step: the MFMAs (0.98 us at the clock the
// chip holds), the LDS-DMA of its 64 KB of operands (0.97 us from L2 / Infinity Cache at the
// rate 256 CUs reach together) and 192 KB of LDS fragment reads (0.42 us).  The three must run
// side by side, so no wave may ever wait for all of its fragments before its first MFMA:
//  - A K step has two halves of 32.  The fragments of a half are read, a few at a time, while
//    the previous half's MFMAs issue; the order is pinned with scheduling barriers and the MFMA
//    groups run at raised wave priority (without: 605 against 572 us at 4096 x 24576 x 4096).
//  - One barrier per K step, between the halves: there every fragment of the step has been
//    read, so its ring slot is free, and the next step's DMA (issued one whole step earlier, the
//    weights' two) has landed.  The step after is then issued into the freed slot.
//  - One workgroup per CU walks a list of tiles.  The last K steps of a tile issue the first
//    ones of the next, so the epilogue and the next tile's first loads overlap.
// The MFMA operands are swapped (D = B A^T): a lane then holds four consecutive columns of one
// row, and every epilogue stores 8 or 16 bytes straight from registers, leaving the LDS ring to
// the DMA.
// Measured on MI355X, operands not in cache: 4096 x 24576 x 4096 with the SwiGLU epilogue 565 us
// = 1.46 PFLOP/s, 4624 rows 656 us against 821 for the LDS-pipeline kernel it replaced (which
// read every fragment of a K step before its first MFMA), 4096 x 4096 x 12288 288 us.
#include "common.h"
#include "internal.h"

namespace dpara {
namespace {

__device__ __forceinline__ float silu_l(float g) {
  return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.4426950408889634f));
}

__device__ __forceinline__ uint2 pack4(float a, float b, float c, float d) {
  return make_uint2((uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16), (uint32_t)f2bf(c) | ((uint32_t)f2bf(d) << 16));
}

// Sum over the four lanes l, l + 16, l + 32, l + 48 of a wave.
__device__ __forceinline__ float lanes4_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}

// The work of one launch: `full` tiles of BM x BN over every K split, then, where the last row
// tile holds few rows, its columns as `tails` tiles of 64 or 128 rows.  A tail costs less than
// a full tile (tail_cost), so the workgroups without a full tile in the last round take up to
// two of them each before the rest is dealt to all.
struct LargePlan {
  int mtf, NT;      // full row tiles, column tiles
  int full, tails;  // items
  int rem, nfree, tails1;
  int grid;
};

constexpr int kGroupM = 8;

// B slots of the ring: weights come from HBM, so their loads run a K step further ahead than the
// activations' (4096 x 4096 x 12288 with operands not in cache: 308 -> 288 us; 192-row tiles
// 433 -> 391).  The QKV epilogue's V^T staging (2 KB a wave) leaves no room for the third slot
// at 256 rows.  A tail tile's K step is short (36 KB of loads), so there both operands run two or
// three steps ahead.
__host__ __device__ constexpr int ring_depth(int epi, int bm) { return (epi == EPI_QKV || epi == EPI_KV) && bm == 256 ? 2 : 3; }
__host__ __device__ constexpr int tail_depth(int epi, int tail) { return epi == EPI_QKV || tail == 128 ? 3 : 4; }
constexpr int kStageWave = 2048;

// Row and column tile of item t among MT x NT tiles: 8 contiguous ranges, one per XCD
// (workgroups go round-robin over the XCDs), M fastest inside a range or, from 16 row tiles on,
// inside groups of 8 row tiles (the 32 tiles an XCD runs at once then share 8 A and 4 B tiles).
__device__ __forceinline__ void large_tile(int t, int total, int MT, int NT, int& s, int& mt, int& nt) {
  const int per = total >> 3;
  int L = t;
  if (t < (per << 3)) L = (t & 7) * per + (t >> 3);
  s = L / (MT * NT);
  L -= s * MT * NT;
  if (MT >= 2 * kGroupM) {
    const int grp = L / (kGroupM * NT), first = grp * kGroupM;
    const int gm = min(MT - first, kGroupM), r = L - grp * kGroupM * NT;
    mt = first + r % gm;
    nt = r / gm;
  } else {
    mt = L % MT;
    nt = L / MT;
  }
}

// Order of one half's MFMAs and fragment reads (FM x FN blocks, groups of GRP MFMAs).  The first
// FM / 2 row blocks go over all columns, then the others, so that a fragment whose last MFMA
// comes early (the first part's A, the first columns' B) has one register set and is re-read in
// the groups after it; the rest have two and are read for the next half in the first groups.
// 256 x 256: 72 fragment registers instead of 96, which leaves room for the accumulators
// without spilling.
template <int FM, int FN>
struct HalfPlan {
  static constexpr int GRP = FM * FN % 4 == 0 && FM * FN >= 8 ? 4 : 2, NG = FM * FN / GRP, LO = FM / 2, HI = FM - LO;
  static_assert(FM * FN % GRP == 0 && NG >= 2, "whole groups of MFMAs");
  static constexpr int mi(int t) { return t < LO * FN ? t % LO1 : LO + (t - LO * FN) % HI; }
  static constexpr int ni(int t) { return t < LO * FN ? t / LO1 : (t - LO * FN) / HI; }
  static constexpr int LO1 = LO > 0 ? LO : 1;
  // group of the last MFMA that uses column block n / a row block of the first part
  static constexpr int last_b(int n) { return (LO * FN + (n + 1) * HI - 1) / GRP; }
  static constexpr int last_a() { return (LO * FN - 1) / GRP; }
  static constexpr int singles() {  // B blocks 0 .. singles - 1 have one register set
    int n = 0;
    while (n < FN && last_b(n) + 1 <= NG - 2) ++n;
    return n;
  }
  static constexpr int SB = singles(), DB = FN - SB;
  static constexpr int NBF = SB + 2 * DB, NAF = LO + 2 * HI;
  static constexpr int bslot(int h, int n) { return n < SB ? n : SB + (n - SB) + h * DB; }
  static constexpr int aslot(int h, int m) { return m < LO ? m : m + h * HI; }
  // group before which the next half's fragment is read
  static constexpr int RATE = (DB + HI + NG - 2) / (NG - 1);
  static constexpr int read_b(int n) { return n < SB ? last_b(n) + 1 : (n - SB) / RATE; }
  static constexpr int read_a(int m) { return m < LO ? (last_a() + 1 < NG ? last_a() + 1 : NG - 1) : (DB + m - LO) / RATE; }
};

// Parts of the epilogues that hold one 128-wide head a wave column: x[ni] are a row's columns
// ni * 16 + lc * 4 .., the rest of its 128 sits in the three lanes 16 apart.
// x * (1 / sqrt(ss / 128 + eps)) * g; gain: the lane's first.
__device__ __forceinline__ void head_norm(f32x4_t (&x)[8], const float* gain, float eps) {
  float ss = 0.f;
#pragma unroll
  for (int ni = 0; ni < 8; ++ni)
#pragma unroll
    for (int r = 0; r < 4; ++r) ss += x[ni][r] * x[ni][r];
  ss = lanes4_sum(ss);
  const float rn = 1.0f / sqrtf(ss / 128.0f + eps);
#pragma unroll
  for (int ni = 0; ni < 8; ++ni) {
    const float4 g = *(const float4*)(gain + ni * 16);
    x[ni][0] = x[ni][0] * rn * g.x;
    x[ni][1] = x[ni][1] * rn * g.y;
    x[ni][2] = x[ni][2] * rn * g.z;
    x[ni][3] = x[ni][3] * rn * g.w;
  }
}

// x_d cos - x_{d+64} sin and x_{d+64} cos + x_d sin (both operands in the lane) as bf16; cs, dst: the
// lane's first (cos, sin) and destination.
__device__ __forceinline__ void head_rope(const f32x4_t (&x)[8], const float2* cs, bf16_t* dst) {
#pragma unroll
  for (int ni = 0; ni < 4; ++ni) {
    const float4 c01 = *(const float4*)(cs + ni * 16), c23 = *(const float4*)(cs + ni * 16 + 2);
    const float co[4] = {c01.x, c01.z, c23.x, c23.z}, si[4] = {c01.y, c01.w, c23.y, c23.w};
    float lo[4], hi[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float l = x[ni][r], h = x[ni + 4][r];
      lo[r] = l * co[r] + -1.f * h * si[r];
      hi[r] = h * co[r] + 1.f * l * si[r];
    }
    *(uint2*)(dst + ni * 16) = pack4(lo[0], lo[1], lo[2], lo[3]);
    *(uint2*)(dst + ni * 16 + 64) = pack4(hi[0], hi[1], hi[2], hi[3]);
  }
}

// The wave's WM rows as columns of a [128][stride] matrix: 16 head dimensions at a time through its
// LDS, so that a store covers consecutive rows.  Lane l stores row l at dst where `on`.
template <int WM>
__device__ __forceinline__ void head_transposed(const f32x4_t (&acc)[WM / 16][8], bf16_t* stg, int lane, bool on,
                                                bf16_t* dst, int stride) {
  const int lr = lane & 15, lc = lane >> 4;
#pragma unroll
  for (int ni = 0; ni < 8; ++ni) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mi = 0; mi < WM / 16; ++mi)
#pragma unroll
      for (int r = 0; r < 4; ++r) stg[(lc * 4 + r) * 64 + mi * 16 + lr] = f2bf(acc[mi][ni][r]);
    wave_lds_fence();
    if (on)
#pragma unroll 8
      for (int d = 0; d < 16; ++d) dst[(int64_t)(ni * 16 + d) * stride] = stg[d * 64 + lane];
    wave_lds_fence();
  }
}

// Epilogue of one BM x BN tile whose wave (wm, wn) holds rows m0 + wm * WM .. and columns
// wn * WN .. of column tile nt: lane (lr, lc) has row .. + mi * 16 + lr and the four columns
// ni * 16 + lc * 4 .. of every fragment (mi, ni); rows from m_end on are not the tile's.  stg: kStageWave bytes of LDS of this wave alone.
template <int BN, int WM, int WN, int WNW, int EPI>
__device__ __forceinline__ void large_epilogue(const GemmArgs& a, f32x4_t (&acc)[WM / 16][WN / 16], int s, int row0,
                                               int m_end, int nt, int wn, int lane, bf16_t* stg) {
  constexpr int FM = WM / 16, FN = WN / 16;
  const int lr = lane & 15, lc = lane >> 4;
  const int row_w = row0 + lr;
  if constexpr (EPI == EPI_KV) {
    static_assert(WN == 128, "one 128-wide head per wave column");
    // as EPI_QKV below, at each row's position in the caches
    const KvEpi& e = a.kv;
    const int head = nt * WNW + wn, l = head / (2 * e.n_kv), slot = head - l * 2 * e.n_kv;
    if (head * 128 >= a.N) return;
    // this lane's row: its request, position, and whether it is stored
    auto place = [&](int row, int& b, int& pos) {
      const int r = e.r0 + min(row, m_end - 1);
      b = r / e.n_max;
      const int c = r - b * e.n_max;
      pos = max(e.ctx_len[b], 0) + c;
      return row < m_end && c < min(e.n_new[b], e.n_max) && pos < e.cap;
    };
    if (slot < e.n_kv) {
      const float* gain = e.kn[0];
#pragma unroll
      for (int j = 1; j < 8; ++j) gain = l == j ? e.kn[j] : gain;  // (an indexed argument goes to scratch)
      gain += lc * 4;
#pragma unroll
      for (int mi = 0; mi < FM; ++mi) {
        __builtin_amdgcn_sched_barrier(0);
        const int row = row_w + mi * 16;
        int b, pos;
        const bool on = place(row, b, pos);
        if (e.qk_norm) head_norm(acc[mi], gain, e.eps);
        if (on)
          head_rope(acc[mi], e.table + (int64_t)row * 64 + lc * 4,
                    (bf16_t*)e.Kc + l * e.layer_elems + ((int64_t)(b * e.n_kv + slot) * e.cap + pos) * 128 + lc * 4);
      }
    } else {
      int b, pos;
      const bool on = place(row0 + lane, b, pos) && lane < WM;
      bf16_t* dst = (bf16_t*)e.Vc + l * e.layer_elems + (int64_t)(b * e.n_kv + slot - e.n_kv) * 128 * e.cap + pos;
      head_transposed<WM>(acc, stg, lane, on, dst, e.cap);
    }
    return;
  }
  if constexpr (EPI == EPI_QKV) {
    static_assert(WN == 128, "one 128-wide head per wave column");
    const QkvEpi& e = a.qkv;
    const int slot = nt * WNW + wn, grp = e.n_q / e.n_kv;
    if (slot >= e.n_q + 2 * e.n_kv) return;
    if (slot < e.n_q + e.n_kv) {
      const bool isq = slot < e.n_q;
      const float* gain = (isq ? e.qn : e.kn) + lc * 4;
#pragma unroll
      for (int mi = 0; mi < FM; ++mi) {
        __builtin_amdgcn_sched_barrier(0);
        const int row = row_w + mi * 16, rc = min(row, m_end - 1), b = rc / e.R, rr = rc - b * e.R;
        if (e.qk_norm) head_norm(acc[mi], gain, e.eps);
        const float2* cs = e.table + ((int64_t)b * (2 * e.gamma + 1) + row_pos_offset(rr, e.gamma)) * 64 + lc * 4;
        bf16_t* dst = isq ? (bf16_t*)e.Q + (((int64_t)(b * e.n_kv + slot / grp) * grp + slot % grp) * e.R + rr) * 128
                          : (bf16_t*)e.Kb + ((int64_t)(b * e.n_kv + (slot - e.n_q)) * e.Rp + rr) * 128;
        if (row < m_end) head_rope(acc[mi], cs, dst + lc * 4);
      }
    } else {
      // V^T [128][Rp] per request
      const int row = row0 + lane, rc = min(row, m_end - 1), b = rc / e.R;
      bf16_t* dst = (bf16_t*)e.Vb + (int64_t)(b * e.n_kv + (slot - e.n_q - e.n_kv)) * 128 * e.Rp + (rc - b * e.R);
      head_transposed<WM>(acc, stg, lane, lane < WM && row < m_end, dst, e.Rp);
    }
    return;
  }
#pragma unroll
  for (int mi = 0; mi < FM; ++mi) {
    __builtin_amdgcn_sched_barrier(0);
    const int row = row_w + mi * 16;
    if constexpr (EPI == EPI_TOP2) {
      static_assert(WN == 128, "one 128-column top-2 tile per wave column");
      const int tile = nt * WNW + wn, n_tiles = (a.N + 127) / 128;
      // The values alone first: the largest three, v1 >= v2 >= v3, by a max and two medians a value,
      // then the columns of v1 and v2 by comparing with them.  Two equal values among the three, a
      // value that is not finite or columns past N: by keys (1088 rows x 151936 x 4096, keys for every
      // value 1270 us, so 1137).
      Top3 t{};
      float v1 = -INFINITY, v2 = -INFINITY, v3 = -INFINITY, zero = 0.f;
#pragma unroll
      for (int ni = 0; ni < FN; ++ni)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float x = acc[mi][ni][r];
          zero = fmaf(x, 0.f, zero);
          v3 = __builtin_amdgcn_fmed3f(v2, v3, x);
          v2 = __builtin_amdgcn_fmed3f(v1, v2, x);
          v1 = fmaxf(v1, x);
        }
#pragma unroll
      for (int o = 16; o <= 32; o *= 2) {
        const float u1 = __shfl_xor(v1, o, 64), u2 = __shfl_xor(v2, o, 64), u3 = __shfl_xor(v3, o, 64);
        for (const float x : {u1, u2, u3}) {
          v3 = __builtin_amdgcn_fmed3f(v2, v3, x);
          v2 = __builtin_amdgcn_fmed3f(v1, v2, x);
          v1 = fmaxf(v1, x);
        }
      }
      if (__any(row < m_end && (zero != 0.f || v1 == v2 || v2 == v3)) || (tile + 1) * 128 > a.N) {
#pragma unroll
        for (int ni = 0; ni < FN; ++ni) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int col = nt * BN + wn * WN + ni * 16 + lc * 4 + r;
            if (col < a.N) t.add(argmax_key(acc[mi][ni][r], (uint32_t)col));
          }
        }
#pragma unroll
        for (int o = 16; o <= 32; o *= 2) {
          Top3 u;
          u.k1 = __shfl_xor((unsigned long long)t.k1, o, 64);
          u.k2 = __shfl_xor((unsigned long long)t.k2, o, 64);
          u.v3 = __shfl_xor(t.v3, o, 64);
          t = Top3::merge(t, u);
        }
      } else {
        int c1 = -1, c2 = -1;
#pragma unroll
        for (int ni = 0; ni < FN; ++ni)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            c1 = acc[mi][ni][r] == v1 ? ni * 16 + r : c1;
            c2 = acc[mi][ni][r] == v2 ? ni * 16 + r : c2;
          }
        c1 = c1 < 0 ? -1 : c1 + lc * 4;
        c2 = c2 < 0 ? -1 : c2 + lc * 4;
#pragma unroll
        for (int o = 16; o <= 32; o *= 2) {
          c1 = max(c1, __shfl_xor(c1, o, 64));
          c2 = max(c2, __shfl_xor(c2, o, 64));
        }
        t.k1 = argmax_key(v1, (uint32_t)(tile * 128 + c1));
        t.k2 = argmax_key(v2, (uint32_t)(tile * 128 + c2));
        t.v3 = v3;
      }
      if (lc == 0 && row < m_end && tile < n_tiles) {
        uint64_t* o = (uint64_t*)a.C + ((int64_t)row * a.ldc + tile) * 3;
        o[0] = t.k1;
        o[1] = t.k2;
        o[2] = (uint64_t)__float_as_uint(t.v3);
      }
      continue;
    }
    if (row >= m_end) continue;
    if constexpr (EPI == EPI_SWIGLU) {
      const int f0 = nt * (BN / 2) + wn * (WN / 2) + lc * 4;
      bf16_t* c = (bf16_t*)a.C + (int64_t)row * a.ldc + f0;
#pragma unroll
      for (int ni = 0; ni < FN / 2; ++ni) {
        if (f0 + ni * 16 >= a.N) continue;
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = silu_l(acc[mi][ni][r]) * acc[mi][ni + FN / 2][r];
        *(uint2*)(c + ni * 16) = pack4(v[0], v[1], v[2], v[3]);
      }
    } else {
      bool vec = ((a.N | (int)a.ldc) & 3) == 0;  // four columns are one aligned store
      if constexpr (EPI == EPI_SCORE) vec = vec && (((uintptr_t)a.C | (uintptr_t)a.base) & 15) == 0;
      const int c0 = nt * BN + wn * WN + lc * 4;
#pragma unroll
      for (int ni = 0; ni < FN; ++ni) {
        f32x4_t v = acc[mi][ni];
        if constexpr (EPI == EPI_SCORE) {
          const float* l = a.base + (int64_t)row * a.ldc + c0 + ni * 16;
          f32x4_t x{0.f, 0.f, 0.f, 0.f};
          if (vec) {
            if (c0 + ni * 16 < a.N) x = *(const f32x4_t*)l;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (c0 + ni * 16 + r < a.N) x[r] = l[r];
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = (x[r] + v[r]) * a.scale;
        }
        if constexpr (EPI == EPI_STORE_BF16) {
          bf16_t* c = (bf16_t*)a.C + (int64_t)row * a.ldc + c0;
          if (vec) {
            if (c0 + ni * 16 < a.N) *(uint2*)(c + ni * 16) = pack4(v[0], v[1], v[2], v[3]);
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (c0 + ni * 16 + r < a.N) c[ni * 16 + r] = f2bf(v[r]);
          }
        } else {
          float* c = (float*)a.C + ((int64_t)s * a.M + row) * a.ldc + c0;
          if (vec) {
            if (c0 + ni * 16 < a.N) *(f32x4_t*)(c + ni * 16) = v;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (c0 + ni * 16 + r < a.N) c[ni * 16 + r] = v[r];
          }
        }
      }
    }
  }
}

// A list of n tiles of `rows` <= BM rows (item(i): K split s, first row m0, column tile nt) for
// WMW x WNW waves; K a multiple of 128, at least 256 per split.  NA, NB: ring slots of A and B;
// STREAM: the weights are read once, as non-temporal lines (the activations stay in L2).
// PL: planes of A; two are a float32 operand's bf16 hi and lo parts (lo_off apart), whose rows share a
// ring slot and which both meet every weight fragment, hi first.
template <int BM, int BN, int WMW, int WNW, int NA, int NB, int EPI, int STREAM, int PL, typename Item>
__device__ __forceinline__ void large_tiles(const GemmArgs& a, int n, int rows, const Item& item, unsigned char* smem) {
  constexpr int NW = WMW * WNW, WM = BM / WMW, WN = BN / WNW, FM = WM / 16, FN = WN / 16;
  constexpr int GR = 8 * NW;  // tile rows one DMA instruction of every wave loads
  constexpr int AG = BM / GR, AI = PL * AG, BI = BN / GR, ND = AI + BI;  // 1 KB DMA instructions per wave and K step
  constexpr int A_SLOT = PL * BM * 128, B_SLOT = BN * 128, B0 = NA * A_SLOT, RING = NA * A_SLOT + NB * B_SLOT;
  // loads a step's barrier may leave in flight: those issued after the next step's (vmcnt counts
  // in order)
  static_assert(NA == NB || (NA == 2 && NB == 3), "ring depths");
  constexpr int LATER = NA == NB ? (NB - 2) * ND : BI;
  using P = HalfPlan<PL * FM, FN>;
  static_assert(BM % GR == 0 && BN % GR == 0, "whole DMA groups");
  static_assert(EPI != EPI_SWIGLU || FN % 2 == 0, "gate and up fragments in pairs");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WNW, wn = wave % WNW;
  const int lr = lane & 15, lc = lane >> 4;

  // DMA sources.  One instruction of a wave loads 8 rows of 128 bytes; the waves' q-th
  // loads cover rows GR q .. of the tile's A or B rows (the same byte offsets for both: lda == K).
  // Rows past M or N lie outside the buffer descriptor: nothing is read for them, and what their
  // LDS rows hold only reaches rows and columns the epilogue does not store.  A row's 16-byte
  // chunk c sits in LDS slot c ^ (row % 8), so fragment reads (16 rows, one chunk) spread over
  // the banks.
  const int K2 = a.K * 2;
  const int lrow = lane >> 3;
  constexpr int BP = EPI == EPI_SWIGLU ? 2 : 1;  // B parts: gate and up rows
  constexpr int BG = BI / BP;  // groups of a part
  static_assert(BG * BP == BI, "whole groups of a part");
  int voff[AG > BG ? AG : BG];
#pragma unroll
  for (int q = 0; q < (AG > BG ? AG : BG); ++q)
    voff[q] = (q * GR + wave * 8 + lrow) * K2 + (((lane & 7) ^ lrow) * 16);
  const char *pa, *pb[BP];  // the tile the next A load and the next B load belong to
  unsigned na, nb;          // valid bytes from there
  int ka = 0, kb = 0;       // and their K steps within it
  // split s covers the 128-deep K units [s U / S, (s + 1) U / S), U = K / 128
  auto k_byte = [&](int s) { return (int)((int64_t)(a.K / 128) * s / a.splits) * 256; };
  auto a_source = [&](int s, int m0, const char*& p, unsigned& n) {
    p = (const char*)a.A + (int64_t)m0 * K2 + k_byte(s);
    n = (unsigned)(min(rows, a.M - m0) * K2 - k_byte(s));
  };
  auto b_source = [&](int s, int nt, const char* (&p)[BP], unsigned& n) {
    const int c = nt * (BN / BP), left = min(BN / BP, a.N - c);
    const void* m = a.B0;
    int r = c;  // the tile's first row of m
    if constexpr (EPI == EPI_SWIGLU) {
      p[BP - 1] = (const char*)a.B1 + (int64_t)c * K2 + k_byte(s);
    } else if (a.seg_rows > 0) {  // a tile lies within one segment (gemm_large_supported)
      const int si = c / a.seg_rows;
#pragma unroll
      for (int k = 0; k < kMaxGemmSegs; ++k) m = si == k ? a.seg[k] : m;  // (an indexed argument goes to scratch)
      r -= si * a.seg_rows;
    } else if (c >= a.n2) {
      m = a.B2;
      r -= a.n2;
    } else if (c >= a.n1) {
      m = a.B1;
      r -= a.n1;
    }
    p[0] = (const char*)m + (int64_t)r * K2 + k_byte(s);
    n = (unsigned)(left * K2 - k_byte(s));
  };
  // q-th load of A step ka into A slot `as`, or of B step kb into B slot `bs`
  auto dma = [&](int q, int as, int bs) {
#if defined(__HIP_DEVICE_COMPILE__)
    unsigned char* dst = smem + (q < AI ? as * A_SLOT : B0 + bs * B_SLOT) + (wave + NW * (q < AI ? q : q - AI)) * 1024;
    if (q < AI) {
      const char* p = PL > 1 && q >= AG ? pa + a.lo_off * 2 : pa;
      const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)na, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)dst, 16, voff[q % AG], ka * 128, 0, 0);
    } else {
      const int j = q - AI;
      const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)pb[j / BG], 0, (int)nb, 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)dst, 16, voff[j % BG], kb * 128, 0, STREAM ? 2 : 0);
    }
#endif
  };

  // Fragment addresses.  SwiGLU tiles hold BN/2 gate rows, then BN/2 up rows; a wave takes the
  // same FFN columns of both.
  const int x0 = (lc ^ (lr & 7)) * 16;
  constexpr bool kPair = EPI == EPI_SWIGLU;
  const unsigned char* ra[2];
  const unsigned char* rb[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    ra[h] = smem + (wm * WM + lr) * 128 + (x0 ^ (h * 64));
    rb[h] = smem + B0 + (wn * (kPair ? WN / 2 : WN) + lr) * 128 + (x0 ^ (h * 64));
  }
  bf16x8_t af[P::NAF], bf[P::NBF];
  f32x4_t acc[FM][FN];
  auto read_b = [&](int n, int bs, int h) {
    const int row = kPair && n >= FN / 2 ? BN / 2 + (n - FN / 2) * 16 : n * 16;
    bf[P::bslot(h, n)] = *(const bf16x8_t*)(rb[h] + bs * B_SLOT + row * 128);
  };
  auto read_a = [&](int m, int as, int h) {
    af[P::aslot(h, m)] = *(const bf16x8_t*)(ra[h] + as * A_SLOT + (m / FM) * BM * 128 + (m % FM) * 2048);
  };
  constexpr int DPG = (ND + P::NG - 1) / P::NG;
  // One half of a K step: the MFMAs of register set h, the fragment reads of the next half
  // (slots as, bs; set h ^ 1) and, in the second half, the DMA into slots da, db.
  auto half = [&](int h, int as, int bs, int da, int db) {
#pragma unroll
    for (int g = 0; g < P::NG; ++g) {
#pragma unroll
      for (int n = 0; n < FN; ++n)
        if (P::read_b(n) == g) read_b(n, bs, h ^ 1);
#pragma unroll
      for (int m = 0; m < PL * FM; ++m)
        if (P::read_a(m) == g) read_a(m, as, h ^ 1);
      if (h == 1) {
#pragma unroll
        for (int q = g * DPG; q < (g + 1) * DPG && q < ND; ++q) dma(q, da, db);
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int t = g * P::GRP; t < (g + 1) * P::GRP; ++t) {
        const int m = P::mi(t), mi = m % FM, ni = P::ni(t);
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[P::bslot(h, ni)], af[P::aslot(h, m)], acc[mi][ni], 0, 0, 0);
      }
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // the first NA steps of A and NB of B; a step's ring slot is its number, over the whole list's
  // steps, mod NA or NB
  int s, m0, nt;  // the tile being computed
  item(0, s, m0, nt);
  a_source(s, m0, pa, na);
  b_source(s, nt, pb, nb);
#pragma unroll
  for (int k = 0; k < NB; ++k) {
#pragma unroll
    for (int q = k < NA ? 0 : AI; q < ND; ++q) dma(q, k, k);
    if (k < NA) ++ka;
    ++kb;
  }
  wait_vmcnt<AI*(NA - 1) + BI * (NB - 1)>();
  __builtin_amdgcn_s_barrier();

  int as = 0, bs = 0;  // slots of the current step
  for (int it = 0; it < n; ++it) {
    int s1, m1, nt1;  // the next one (the list's end repeats its last tile)
    item(it + 1 < n ? it + 1 : it, s1, m1, nt1);
    const char *pa1, *pb1[BP];
    unsigned na1, nb1;
    a_source(s1, m1, pa1, na1);
    b_source(s1, nt1, pb1, nb1);
    const int KT = (k_byte(s + 1) - k_byte(s)) / 128;
#pragma unroll
    for (int j = 0; j < FN; ++j) read_b(j, bs, 0);
#pragma unroll
    for (int i = 0; i < PL * FM; ++i) read_a(i, as, 0);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int kt = 0; kt < KT; kt += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (NA == 2) as = u;  // (KT is even: a constant)
        const int an = as + 1 == NA ? 0 : as + 1, bn = bs + 1 == NB ? 0 : bs + 1;
        __builtin_amdgcn_sched_barrier(0);
        half(0, as, bs, 0, 0);
        // Every wave has its fragments of this step, and the next step's DMA has landed (after an
        // epilogue its stores are younger than the loads, so the wait is only longer).
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_vmcnt<LATER>();
        __builtin_amdgcn_s_barrier();
        // the last steps of a tile load the next one's first (KT is even and at least 4): scalar
        // selects, a branch here costs the loop twenty vector registers
        if (u == (NA & 1)) {
          pa = ka == KT ? pa1 : pa;
          na = ka == KT ? na1 : na;
          ka = ka == KT ? 0 : ka;
        }
        if (u == (NB & 1)) {
#pragma unroll
          for (int i = 0; i < BP; ++i) pb[i] = kb == KT ? pb1[i] : pb[i];
          nb = kb == KT ? nb1 : nb;
          kb = kb == KT ? 0 : kb;
        }
        __builtin_amdgcn_sched_barrier(0);
        half(1, an, bn, as, bs);
        ++ka;
        ++kb;
        as = an;
        bs = bn;
      }
    }
    // (the next tile's first fragments are read again after the epilogue: 48 registers less
    // while it runs)
    __builtin_amdgcn_sched_barrier(0);
    large_epilogue<BN, WM, WN, WNW, EPI>(a, acc, s, m0 + wm * WM, min(a.M, m0 + rows), nt, wn, lane, (bf16_t*)(smem + RING + wave * kStageWave));
    __builtin_amdgcn_sched_barrier(0);
    s = s1;
    m0 = m1;
    nt = nt1;
  }
  wait_vmcnt<0>();  // the last loads (the list's end repeats its last tile) have landed
}

template <int BM, int BN, int EPI, int TAIL>
__global__ __launch_bounds__(512, 2) void gemm_large_kernel(GemmArgs a, LargePlan p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if (a.only_if && *a.only_if == 0) return;
  const int w = blockIdx.x;
  constexpr int NB = ring_depth(EPI, BM);
  debug_poison_lds<(2 * BM + NB * BN) * 128>(smem);
  // full tiles w, w + grid, ..; then this workgroup's share of the tails
  const int n_full = w < p.full ? (p.full - w + p.grid - 1) / p.grid : 0;
  if (n_full > 0)
    large_tiles<BM, BN, 4, 2, 2, NB, EPI, 0, 1>(a, n_full, BM, [&](int i, int& s, int& m0, int& nt) {
      int mt;
      large_tile(w + p.grid * i, p.full, p.mtf, p.NT, s, mt, nt);
      m0 = mt * BM;
    }, smem);
  if constexpr (TAIL > 0) {
    const int fr = w - p.rem;
    const int n1 = fr >= 0 && fr < p.tails1 ? (p.tails1 - fr + p.nfree - 1) / p.nfree : 0;
    const int t2 = p.tails - p.tails1;
    const int n2 = w < t2 ? (t2 - w + p.grid - 1) / p.grid : 0;
    if (n1 + n2 == 0) return;
    __syncthreads();  // the ring is reused
    constexpr int TD = tail_depth(EPI, TAIL);
    // 64 rows: 2 x 4 waves where 64 columns a wave will do (a third fewer LDS reads)
    constexpr int WNW = TAIL == 64 && BN == 256 && EPI != EPI_QKV && EPI != EPI_TOP2 ? 4 : 2;
    large_tiles<TAIL, BN, 8 / WNW, WNW, TD, TD, EPI, 0, 1>(
        a, n1 + n2, TAIL, [&](int i, int& s, int& m0, int& nt) {
          const int t = i < n1 ? fr + p.nfree * i : p.tails1 + w + p.grid * (i - n1);
          s = t / p.NT;
          nt = t - s * p.NT;
          m0 = p.mtf * BM;
        }, smem);
  }
}

// 65 to 320 rows: weight streaming.  One or a few row tiles of equal height cover the rows, so the
// weights are read once from HBM; workgroups walk the tiles as above, one or two to a CU.
constexpr int mid_ring(int BM, int BN, int NA, int NB, int PL) { return (NA * PL * BM + NB * BN) * 128; }
template <int BM, int BN, int WMW, int WNW, int NA, int NB, int EPI, int STREAM, int PL>
__global__ __launch_bounds__(64 * WMW * WNW, mid_ring(BM, BN, NA, NB, PL) <= 81920 ? WMW * WNW / 2 : WMW * WNW / 4) void
gemm_mid_kernel(GemmArgs a, int MT, int NT, int rows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if (a.only_if && *a.only_if == 0) return;
  debug_poison_lds<mid_ring(BM, BN, NA, NB, PL)>(smem);
  const int w = blockIdx.x, grid = gridDim.x, total = MT * NT * a.splits;
  large_tiles<BM, BN, WMW, WNW, NA, NB, EPI, STREAM, PL>(a, (total - w + grid - 1) / grid, rows,
                                                     [&](int i, int& s, int& m0, int& nt) {
                                                       int mt;
                                                       large_tile(w + grid * i, total, MT, NT, s, mt, nt);
                                                       m0 = mt * rows;
                                                     },
                                                     smem);
}

// The context append over more than 320 feature rows (EPI_KV): all layers' K|V projections straight
// into the caches.  Row tiles whose rows are all past their request's count or the cache's end are
// left out: every workgroup finds the tiles that are not (at most 64, one a lane).  Bound by the
// MFMAs and the DMA, as above.  Three prompts of 1250, 955 and 478 rows, five Qwen3-8B layers: 246 us;
// fp32 planes in chunks of 867 rows, a copy of the features and a store pass took 490.
template <int BM>
__global__ __launch_bounds__(512, 2) void gemm_kv_kernel(GemmArgs a, int MT, int NT) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int NB = ring_depth(EPI_KV, BM), NA = BM == 256 ? 2 : 3;
  debug_poison_lds<(NA * BM + NB * 256) * 128>(smem);
  const KvEpi& e = a.kv;
  const int t = threadIdx.x & 63;
  bool live = false;
  if (t < MT) {
    const int r = e.r0 + t * BM, end = e.r0 + min((t + 1) * BM, a.M);
    int b = r / e.n_max, c = r - b * e.n_max;
    for (int left = end - r; left > 0 && !live; ++b) {
      live = c < min(e.n_new[b], e.n_max) && max(e.ctx_len[b], 0) + c < e.cap;
      left -= e.n_max - c;
      c = 0;
    }
  }
  const unsigned long long mask = __ballot(live);
  const int n_live = __popcll(mask), w = blockIdx.x, grid = gridDim.x, total = n_live * NT;
  if (w >= total) return;
  large_tiles<BM, 256, 4, 2, NA, NB, EPI_KV, 0, 1>(a, (total - w + grid - 1) / grid, BM,
                                                [&](int i, int& s, int& m0, int& nt) {
                                                  int mt;
                                                  large_tile(w + grid * i, total, n_live, NT, s, mt, nt);
                                                  unsigned long long m = mask;
                                                  for (; mt > 0; --mt) m &= m - 1;
                                                  m0 = (__ffsll(m) - 1) * BM;
                                                },
                                                smem);
}

constexpr int kCus = 256;

// Rows of the tail tiles (0: the last row tile runs as a full one) and their cost against a full
// tile: a 64-row tile is bound by its weight loads (36 KB of a full tile's 64 KB a K step).
int tail_rows(int M, int BM) {
  const int left = (M - 1) % BM + 1;
  return left <= 64 ? 64 : left <= 128 && BM > 128 ? 128 : 0;
}
double tail_cost(int rows, int BM) { return rows == 64 ? (BM == 256 ? 0.5 : 0.65) : (BM == 256 ? 0.65 : 0.8); }

LargePlan large_plan(int M, int NT, int BM, int S) {
  LargePlan p{};
  const int tail = tail_rows(M, BM);
  p.NT = NT;
  p.mtf = (M + BM - 1) / BM - (tail ? 1 : 0);
  p.full = p.mtf * NT * S;
  p.tails = tail ? NT * S : 0;
  p.grid = p.full + p.tails < kCus ? p.full + p.tails : kCus;
  p.rem = p.full % p.grid;
  p.nfree = p.grid - p.rem;
  const int cap = tail == 64 ? 2 : 1;
  p.tails1 = p.tails < cap * p.nfree ? p.tails : cap * p.nfree;
  return p;
}

// Estimated time of the launch, us (operands from HBM; fitted to measurements on MI355X over 400 to
// 4624 rows, within about 8%): a 64-deep K step of a 256 x 256 tile takes 1.44, of 192 x 256 and
// 256 x 192 1.18; each tile 1.5 more.  A round that fills only part of the CUs runs its tiles
// up to 22% faster.
double large_time(int M, int NT, int BM, int BN, int S, int K) {
  const LargePlan p = large_plan(M, NT, BM, S);
  const int steps = (K / 128 + S - 1) / S * 2;
  const double t = (BM == 256 && BN == 256 ? 1.44 : 1.18) * steps + 1.5;
  const double tc = tail_cost(tail_rows(M, BM), BM);
  const int whole = p.full / p.grid, n1 = (p.tails1 + p.nfree - 1) / p.nfree, t2 = p.tails - p.tails1;
  const double last = 0.78 + 0.22 * (p.rem + tc * p.tails1) / kCus;
  double r = whole * (p.grid < kCus ? 0.78 + 0.22 * p.grid / kCus : 1.0) + (p.rem > 0 ? last : 0.0);
  if (whole + n1 * tc > r) r = whole + n1 * tc;
  return (r + (t2 + p.grid - 1) / p.grid * tc) * t;
}

struct LargeTile {
  int BM, BN;
  double us;
};
// The tile with the least estimated time.  narrow: 256 x 192 is available.
LargeTile large_choice(int M, int N, int K, int S, int cols_per_256, bool narrow) {
  auto nt = [&](int bn) { const int c = bn * cols_per_256 / 256; return (N + c - 1) / c; };
  LargeTile best{256, 256, large_time(M, nt(256), 256, 256, S, K)};
  const double t1 = large_time(M, nt(256), 192, 256, S, K);
  if (t1 < best.us) best = {192, 256, t1};
  if (narrow) {
    const double t2 = large_time(M, nt(192), 256, 192, S, K);
    if (t2 < best.us) best = {256, 192, t2};
  }
  return best;
}

// Estimated time, us, of the LDS-pipeline kernel's 64 x 128 tiles (gemm.hip) over NT column tiles: two
// fit on a CU, so few rows of a short K, too few large tiles for the CUs, run them side by side.
// A 64-deep K step takes 0.48 while a CU has one and up to 0.72 with two (fitted to 325 to 1024 rows,
// K 1024 to 8192; only one round of the CUs).
double rows64_time(int M, int NT, int K) {
  if (M > 1024 || (M + 63) / 64 * NT > 2 * kCus) return 1e30;
  const double T = M / 64.0 * NT;
  return 0.5 + K / 64 * (T <= 256 ? 0.48 : T >= 352 ? 0.72 : 0.48 + 0.0025 * (T - 256));
}

// A float32 plane's store and its consumer's read (about 3.5 and 4 TB/s).
double plane_time(int M, int N) { return (double)M * N * 4.0 * (1 / 3.5e6 + 1 / 4e6); }

// Planes of the float32 store and their estimated time with the GEMM.  867 x 4096 x 12288: 195 us as
// one plane, 84 as three.
struct StoreChoice {
  int S;
  double us;
};
StoreChoice store_choice(int M, int N, int K) {
  StoreChoice best{1, 1e30};
  for (int S = 1; S <= 8 && K / 128 >= 2 * S; ++S) {
    const double t = large_choice(M, N, K, S, 256, true).us + S * plane_time(M, N);
    if (t < best.us) best = {S, t};
  }
  return best;
}

template <int BM, int BN, int EPI, int TAIL>
hipError_t run_large_tail(const GemmArgs& a, const LargePlan& p, hipStream_t st) {
  constexpr int ring = (2 * BM + ring_depth(EPI, BM) * BN) * 128;
  constexpr int tail = TAIL ? tail_depth(EPI, TAIL) * (TAIL + BN) * 128 : 0;
  constexpr int lds = (ring > tail ? ring : tail) + (EPI == EPI_QKV ? 8 * kStageWave : 0);
  static_assert(lds <= 163840, "LDS");
  auto kern = gemm_large_kernel<BM, BN, EPI, TAIL>;
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(p.grid), dim3(512), lds, st, a, p);
  return hipGetLastError();
}

template <int BM, int BN, int EPI>
hipError_t run_large(const GemmArgs& a, hipStream_t st) {
  constexpr int COLS = EPI == EPI_SWIGLU ? BN / 2 : BN;
  const LargePlan p = large_plan(a.M, (a.N + COLS - 1) / COLS, BM, a.splits);
  switch (tail_rows(a.M, BM)) {
    case 64: return run_large_tail<BM, BN, EPI, 64>(a, p, st);
    case 128: return run_large_tail<BM, BN, EPI, 128>(a, p, st);
    default: return run_large_tail<BM, BN, EPI, 0>(a, p, st);
  }
}

template <int EPI>
hipError_t pick_large(const GemmArgs& a, hipStream_t st) {
  const bool narrow = EPI == EPI_STORE_F32 && a.seg_rows == 0 && a.n1 >= a.N;
  const LargeTile t = large_choice(a.M, a.N, a.K, a.splits, EPI == EPI_SWIGLU ? 128 : 256, narrow);
  if constexpr (EPI == EPI_STORE_F32)
    if (t.BN == 192) return run_large<256, 192, EPI>(a, st);
  if (t.BM == 192) return run_large<192, 256, EPI>(a, st);
  return run_large<256, 256, EPI>(a, st);
}

template <int BM>
hipError_t run_kv(const GemmArgs& a, hipStream_t st) {
  constexpr int NB = ring_depth(EPI_KV, BM), NA = BM == 256 ? 2 : 3;
  constexpr int lds = (NA * BM + NB * 256) * 128 + 8 * kStageWave;
  static_assert(lds <= 163840, "LDS");
  auto kern = gemm_kv_kernel<BM>;
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr != hipSuccess) return attr;
  const int MT = (a.M + BM - 1) / BM, NT = (a.N + 255) / 256;
  hipLaunchKernelGGL(kern, dim3(MT * NT < kCus ? MT * NT : kCus), dim3(512), lds, st, a, MT, NT);
  return hipGetLastError();
}

// 256-row tiles, or 128 where the rounds over the CUs cost less (a K step of 128 x 256 takes about
// 0.6 of one of 256 x 256).
hipError_t pick_kv(const GemmArgs& a, hipStream_t st) {
  const int NT = (a.N + 255) / 256;
  const int r256 = ((a.M + 255) / 256 * NT + kCus - 1) / kCus, r128 = ((a.M + 127) / 128 * NT + kCus - 1) / kCus;
  if (a.M <= 64 * 128 && r128 * 0.6 < r256) return run_kv<128>(a, st);
  return run_kv<256>(a, st);
}

template <int BM, int BN, int WMW, int WNW, int NA, int NB, int EPI, int STREAM, int PL = 1>
hipError_t run_mid(const GemmArgs& a, hipStream_t st) {
  constexpr int lds = mid_ring(BM, BN, NA, NB, PL);
  static_assert(lds <= 163840, "LDS");
  auto kern = gemm_mid_kernel<BM, BN, WMW, WNW, NA, NB, EPI, STREAM, PL>;
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr != hipSuccess) return attr;
  constexpr int COLS = EPI == EPI_SWIGLU ? BN / 2 : BN, slots = lds <= 81920 ? 2 * kCus : kCus;
  const int MT = (a.M + BM - 1) / BM, NT = (a.N + COLS - 1) / COLS, T = MT * NT * a.splits;
  hipLaunchKernelGGL(kern, dim3(T < slots ? T : slots), dim3(64 * WMW * WNW), lds, st, a, MT, NT,
                     (a.M + MT - 1) / MT);
  return hipGetLastError();
}

// Tiles for 65 to 320 rows, measured on MI355X at Qwen3-8B widths with the weights in HBM (us of one
// product's launches back to back, and what the kernels used before took; between the other kernels of
// a layer gate/up at 289 rows takes 69, and took 72):
//  SwiGLU   : up to 128 rows 128 x 128 (192 workgroups at Qwen3-8B; 128 x 192 where that takes
//             fewer rounds): 102 rows 46 (63), Qwen3-14B 73.  Above, two equal row tiles x 192
//             columns by four waves, so that Qwen3-8B gives 256 workgroups and the two that share
//             a weight tile read it from one XCD's L2: 170 rows 54 (65), 238 59 (66), 289 63 (70).
//  fp32     : up to 192 rows one row tile x 128 columns, K split over up to 256 workgroups: 102 rows
//             down 25 (36), O 13 (17), Q|K|V 18 (24); 170 rows down 30, O 16, Q|K|V 21.  Above, two equal
//             row tiles x 128 columns where these and K's splits give 7/8 of the CUs a workgroup: half
//             the planes of the one 320-row tile, or workgroups on CUs it left idle (40 column tiles
//             take three splits, not four).  Drafter of 225 and 289 rows, Qwen3-14B: 1745 and 1867 us,
//             so 1639 and 1757; of 196 and 289 rows, Qwen3-8B: 989 and 1097, so 980 and 1084.
//  LM head  : wide tiles, so that the last round is nearly full: 102 rows x 320 columns 228 (371),
//             170 x 256 267, 238 x 192 340, 272 rows as two row tiles of 160 x 256 373 (382).
//  top-2    : 128-column wave tiles: 128, 192, 256 (or two of 160) rows x 256 columns.
template <int EPI>
hipError_t pick_mid(const GemmArgs& a, hipStream_t st) {
  if constexpr (EPI == EPI_SWIGLU) {
    if (a.M <= 128) {  // a K step's loads: the rows and the columns of the tile
      const int r128 = ((a.N + 63) / 64 + kCus - 1) / kCus, r192 = ((a.N + 95) / 96 + kCus - 1) / kCus;
      if (r128 * (a.M + 128) <= r192 * (a.M + 192)) return run_mid<128, 128, 4, 2, 3, 3, EPI, 1>(a, st);
      return run_mid<128, 192, 2, 2, 3, 3, EPI, 1>(a, st);
    }
    if (a.M <= 192) return run_mid<96, 192, 2, 2, 3, 3, EPI, 0>(a, st);
    if (a.M <= 256) return run_mid<128, 192, 2, 2, 3, 3, EPI, 0>(a, st);
    return run_mid<160, 192, 2, 2, 3, 3, EPI, 0>(a, st);
  } else if constexpr (EPI == EPI_TOP2) {
    if (a.M <= 128) return run_mid<128, 256, 4, 2, 2, 3, EPI, 1>(a, st);
    if (a.M <= 192) return run_mid<192, 256, 4, 2, 2, 3, EPI, 1>(a, st);
    if (a.M <= 256) return run_mid<256, 256, 4, 2, 2, 3, EPI, 1>(a, st);
    return run_mid<160, 256, 2, 2, 2, 3, EPI, 0>(a, st);
  } else {
    if (EPI == EPI_SCORE || a.N > 32768) {  // (S == 1: a vocabulary's columns)
      if constexpr (EPI == EPI_SCORE)
        if (a.M <= 64) return run_mid<64, 320, 4, 2, 2, 3, EPI, 1>(a, st);
      if (a.M <= 128) return run_mid<128, 320, 4, 2, 2, 3, EPI, 1>(a, st);
      if (a.M <= 192) return run_mid<192, 256, 4, 2, 2, 3, EPI, 1>(a, st);
      if (a.M <= 256) return run_mid<256, 192, 4, 2, 2, 3, EPI, 1>(a, st);
      return run_mid<160, 256, 2, 2, 2, 3, EPI, 0>(a, st);
    }
    if constexpr (EPI != EPI_SCORE) {
      if (a.M <= 128) return run_mid<128, 128, 4, 2, 3, 3, EPI, 1>(a, st);
      if constexpr (EPI == EPI_STORE_F32)
        if (a.M > 192) return run_mid<160, 128, 2, 2, 3, 3, EPI, 0>(a, st);
      return run_mid<192, 128, 4, 2, 3, 3, EPI, 1>(a, st);
    }
    return hipErrorInvalidValue;
  }
}

}  // namespace

bool gemm_mid_supported(int epi, const GemmArgs& a) {
  if (a.M <= 64 || a.M > 320 || a.splits < 1 || a.K % 128 != 0 || a.K / 128 < 2 * a.splits || a.lda != a.K) return false;
  if (a.splits > 1 && epi != EPI_STORE_F32) return false;
  if (epi == EPI_SWIGLU) return a.N % 8 == 0 && a.ldc % 4 == 0;
  if (epi == EPI_TOP2) return a.seg_rows == 0 && a.n1 >= a.N;
  if (epi != EPI_STORE_F32 && epi != EPI_STORE_BF16) return false;
  if (a.N > 32768) return a.splits == 1 && a.seg_rows == 0 && a.n1 >= a.N;
  // a 128-column tile comes from one weight segment
  const bool segs = a.seg_rows > 0 ? a.seg_rows % 128 == 0
                                   : (a.n1 >= a.N || a.n1 % 128 == 0) && (a.n2 >= a.N || a.n2 % 128 == 0);
  if (a.M <= 192) return segs;
  return segs && epi == EPI_STORE_F32 && gemm_mid_two_tiles(a.N, a.K) && a.splits == gemm_mid_splits(a.M, a.N, a.K);
}

bool gemm_mid_two_tiles(int N, int K) {
  return 2 * ((N + 127) / 128) * gemm_mid_splits(320, N, K) >= kCus * 7 / 8;
}

int gemm_mid_splits(int M, int N, int K) {
  int S = kCus / ((N + 127) / 128 * (M > 192 ? 2 : 1));
  if (S > 8) S = 8;  // the consumers' plane reads grow with S
  if (S > K / 256) S = K / 256;
  return S < 1 ? 1 : S;
}

hipError_t launch_gemm_mid(int epi, const GemmArgs& a, hipStream_t st) {
  if (epi == EPI_SCORE) return gemm_score_supported(a) ? pick_mid<EPI_SCORE>(a, st) : hipErrorInvalidValue;
  if (!gemm_mid_supported(epi, a)) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_SWIGLU: return pick_mid<EPI_SWIGLU>(a, st);
    case EPI_STORE_F32: return pick_mid<EPI_STORE_F32>(a, st);
    case EPI_STORE_BF16: return pick_mid<EPI_STORE_BF16>(a, st);
    default: return pick_mid<EPI_TOP2>(a, st);
  }
}

bool gemm_score_supported(const GemmArgs& a) {
  return a.M <= 320 && a.K % 128 == 0 && a.K >= 256 && a.lda == a.K && a.splits == 1 && a.seg_rows == 0 && a.n1 >= a.N;
}

bool gemm_dual_supported(const GemmArgs& a) {
  return a.M > 32 && a.K % 128 == 0 && a.K >= 256 && a.lda == a.K && a.splits == 1 && a.seg_rows == 0 && a.n1 >= a.N;
}

hipError_t launch_gemm_dual(const GemmArgs& a, hipStream_t st) {
  if (!gemm_dual_supported(a)) return hipErrorInvalidValue;
  // 320 columns: Qwen3's vocabulary in two rounds of the CUs, each weight fragment read from LDS for
  // both planes of all rows.  128 rows x 151936 x 4096: 290 us against 373 for 128 x 128 tiles with a
  // wait for every fragment of a K step; from 129 rows on two or more row tiles share a weight tile
  // from L2 (208 rows: the sampled head 1024 -> 949).
  if (a.M <= 64) return run_mid<64, 320, 4, 2, 2, 3, EPI_STORE_F32, 1, 2>(a, st);
  if (a.M <= 128) return run_mid<128, 320, 4, 2, 2, 2, EPI_STORE_F32, 1, 2>(a, st);
  return run_mid<128, 320, 4, 2, 2, 2, EPI_STORE_F32, 0, 2>(a, st);
}

bool gemm_large_supported(int epi, const GemmArgs& a) {
  if (a.M <= 320 || a.splits < 1 || a.K % 128 != 0 || a.K / 128 < 2 * a.splits || a.lda != a.K) return false;
  if (a.splits > 1 && epi != EPI_STORE_F32) return false;
  if (epi != EPI_SWIGLU) {  // a 256-column tile comes from one weight segment
    if (a.seg_rows % 256 != 0) return false;
    if (a.seg_rows == 0 && ((a.n1 < a.N && a.n1 % 256 != 0) || (a.n2 < a.N && a.n2 % 256 != 0))) return false;
  }
  switch (epi) {
    case EPI_SWIGLU: return a.N % 8 == 0 && a.ldc % 4 == 0;
    case EPI_STORE_F32:
    case EPI_STORE_BF16:
    case EPI_TOP2:
    case EPI_QKV: return true;
    case EPI_KV: return a.M <= kMaxKvRows && a.seg_rows == a.kv.n_kv * 128 && a.kv.n_max > 0;
    default: return false;
  }
}

int gemm_large_splits(int M, int N, int K) {
  const StoreChoice c = store_choice(M, N, K);
  return rows64_time(M, (N + 127) / 128, K) + plane_time(M, N) < c.us ? 1 : c.S;
}

bool gemm_large_fuses_qkv(int M, int N, int K) {
  // The fused epilogue has no split K: at few rows its tiles leave CUs idle, and the planes with the
  // q/k-norm pass (about 11 us of its own) are faster, or one plane of 64-row tiles.  Qwen3-8B, 340 / 578
  // / 867 / 1156 rows: fused 86 / 74 / 74 / 74 us, planes and pass 41 / 56 / 61 / 71 (64-row tiles 48 /
  // 61 / 94); K 1024, 340 and 867 rows: 35 and 31, 33 and 46, 24 and 38.
  const double us = large_choice(M, N, K, 1, 256, false).us;
  return us <= store_choice(M, N, K).us + 1 && us <= rows64_time(M, (N + 127) / 128, K) + plane_time(M, N) + 3;
}

bool gemm_large_prefers_rows64(int epi, const GemmArgs& a) {
  // gate/up 405 x 3072 x 1024 21 -> 13 us, Q|K|V 340 x 4096 x 2048 52 -> 31 with its pass
  if (a.splits != 1) return false;
  if (epi == EPI_SWIGLU)
    return rows64_time(a.M, (a.N + 63) / 64, a.K) < large_choice(a.M, a.N, a.K, 1, 128, false).us;
  return epi == EPI_STORE_F32 &&
         rows64_time(a.M, (a.N + 127) / 128, a.K) < large_choice(a.M, a.N, a.K, 1, 256, true).us;
}

hipError_t launch_gemm_large(int epi, const GemmArgs& a, hipStream_t st) {
  if (!gemm_large_supported(epi, a)) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_SWIGLU: return pick_large<EPI_SWIGLU>(a, st);
    case EPI_STORE_F32: return pick_large<EPI_STORE_F32>(a, st);
    case EPI_STORE_BF16: return run_large<256, 256, EPI_STORE_BF16>(a, st);
    case EPI_TOP2: return run_large<256, 256, EPI_TOP2>(a, st);
    case EPI_KV: return pick_kv(a, st);
    default: return pick_large<EPI_QKV>(a, st);
  }
}

}  // namespace dpara
