// Forward and input-gradient passes of the domain-parallel 3x3 conv tile (Sec. 2.2, pure
// domain parallelism: each process convolves its spatial tile with the halo supplied;
// the input gradient takes the output gradient with its own halo), for channel counts that
// are multiples of 64, as implicit GEMMs on the zero-padded (H+2) x (W+2) grid:
//   forward   D(P, o) = sum_{tap, c} x_pad[P + r*(W+2) + s][c] * W[o][tap][c]
//   input grad D(P, c) = sum_{tap, o} dy_pad[P + (2-r)*(W+2) + 2-s][o] * W[o][tap][c]
// with tap = 3r + s and P = (n (H+2) + h) (W+2) + w the row of the padded grid whose
// D(P, .) is the output at position (n, h, w). Each tap is a row shift of a dense
// [positions][channels] matrix, so a k-slab (64 channels of one tap) of the activation
// operand is 64 contiguous channels of shifted rows.
//
// What bounds it: with every byte loaded into LDS once per tap, a slab of 128 positions x
// 256 channels (48 KB) took 0.56 us for the loads alone, 0.54 us for the MFMAs with their
// fragment reads and 0.78 us for both, and each round of one-tile workgroups lost 6 us to
// its first loads and its write-out. So the three taps of one kernel row share one
// activation slab: per image row that the tile touches, its positions and the two columns
// after them (16-20% more rows than positions instead of three times as many; the loads of
// as many MFMAs then take 0.34 us); a tap is a shift of the fragment reads. And a workgroup
// walks through several tiles: its loaders run ahead into the next tile while the tile
// before is written from registers. What is left at 256 x 128 is power: a slab takes 0.58
// us on zeros and 0.76 us on normally distributed data (1.3 PFLOP/s, what a large library
// product reaches on the same card). Measured (forward / input gradient, us, before ->
// after; the other channel counts were on the tiled GEMM template):
//   32 x 56 x 56, 256 -> 256:  117 / 110 -> 106 / 107
//   64 x 13 x 13, 384 -> 384:   80 / 105 -> 27.6 / 29.6
//   32 x 56 x 56,  64 -> 128:   49 /  79 -> 21.2 / 23.2
//   32 x 14 x 14, 512 -> 512:   80 / 127 -> 33.6 / 35.2
//    8 x  7 x  7, 512 -> 512:   71 / 121 -> 18.5 / 19.8
//
// Work split: the positions, in blocks of 16, are dealt out evenly to 256 / (channel
// tiles) workgroups per channel tile, and each cuts its share into tiles of nearly equal
// height, so that no short last round of tiles remains. Eight MMA waves (two per SIMD)
// hold 64 positions x 64 channels each, laid out as WP position groups x WC channel groups
// x WK halves of each slab's k:
//   WP = 4, WC = 2: up to 256 positions x 128 channels (shares of more than 128 positions);
//   WP = 2, WC = 2, WK = 2: up to 128 positions x 128 channels: small grids, where shares
//     of 128 positions are all there is; the two k halves keep both waves of a SIMD busy
//     at 64 x 64 fragments each and are added through LDS at the end of a tile;
//   WP = 4, WC = 1, WK = 2: up to 256 positions x 64 channels, for 64 output channels.
// A channel count that is no multiple of 128 leaves half of its last tile's waves idle.
//
// Both operands travel through LDS in 64-k slabs written by buffer loads that go straight
// to LDS in whole 128-byte lines, XOR-swizzled in 16-byte chunks; one barrier per slab:
//  * waves 8-9 stream the activation slabs (one per kernel row and 64-channel chunk)
//    through two slots, a whole slab ahead;
//  * waves 10-11 stream the weight slabs (BN channels x 64 k of one tap) through five
//    slots: rows of W for the forward pass, k-rows of W (64 output channels of one tap x
//    BN input channels, in 64-channel quarters) for the input gradient, whose fragments
//    then come from the gfx950 LDS transpose read.
// Fragments are read between the MFMAs of the k-step before, block by block in place
// (activations) or into a second set (weights); reads stay in flight over the slab barrier,
// so the weight loaders keep one slot more of distance. With all reads ahead of the MFMAs
// and waited for at every barrier, the small-grid layout spilled registers and took 0.54
// instead of 0.41 us a slab (64 x 13 x 13, 384 channels: 36.8 instead of 27.6 us).
// The weights are the MFMA's row operand, so a lane's four sums are four consecutive
// channels of one position; a lane exchange makes them eight, and each store instruction
// writes 64-byte runs.

#include <algorithm>

#include "cdna4.h"

namespace imbd {
namespace {

constexpr int CV_NW = 5;               // weight ring slots
constexpr int CV_QSLOT = 64 * 128;     // one 64-channel quarter of a transposed weight slab
constexpr int CV_CUS = 256;            // compute units of the chip: one workgroup each
constexpr int CV_XBUF = 32 * 1024;     // exchange of the two k halves' sums

struct CvArgs {
  const uint16_t *act;  // x_pad (forward) or dy_pad (input gradient): [N][H+2][W+2][Ck]
  const uint16_t *w;    // [C_out][3][3][C_in]
  void *out;            // [N][H][W][Cn]
  int out_bf16;
  int N, H, W;
  int Ck, Cn, Ci;       // channels of act (the reduction), of out, and C_in (W's channel stride)
  int64_t w_bytes;
  int M, nblk;          // output positions N*H*W, blocks of 16 of them
  int nct, groups;      // channel tiles; workgroups (shares of the blocks) per channel tile
  int tmax;             // position blocks per tile at most
};

// Rows of an activation slab in LDS: the image rows' pieces of the tile one after another,
// each with two columns more than the tile has positions in it.
constexpr int cv_slab_rows(int wp) { return wp == 4 ? 304 : 160; }

__device__ __forceinline__ int cv_swz_kc(int r) { return r & 7; }
__device__ __forceinline__ int cv_swz_tr(int r) { return 2 * ((r >> 1) & 1) + 4 * ((r >> 3) & 1); }
template <int V>
struct CvInt {
  static constexpr int value = V;
};
// x / d for 0 <= x < 2^16 (inv = 1 / d): the half keeps the quotient's error away from whole numbers
__device__ __forceinline__ int cv_div(int x, float inv) { return (int)(((float)x + 0.5f) * inv); }

// TR: input gradient (W read transposed); else forward.
template <bool TR, int WP, int WK>
__global__ void __launch_bounds__(768, 1) conv_nt_kernel(CvArgs a) {
  constexpr int WC = 8 / (WP * WK);
  constexpr int BN = 64 * WC;
  constexpr int RA = cv_slab_rows(WP);
  constexpr uint32_t OOB = 0x80000000u;
  constexpr int WSLOT = BN * 128, ASLOT = RA * 128;
  constexpr int WRING = CV_NW * WSLOT, ARING = 2 * ASLOT;
  constexpr int LDS = WRING + ARING + (WK == 2 ? CV_XBUF : 0);
  static_assert(WP * WC * WK == 8 && (WK == 1 || WP * WC == 4), "eight waves");
  static_assert(LDS <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) char smem[LDS];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // consecutive shares, and the channel tiles of one share, run on one XCD
  const int G = gridDim.x;
  const int l = (int)(blockIdx.x & 7) * (G >> 3) + (int)(blockIdx.x >> 3);
  if (l >= a.groups * a.nct) return;
  const int gr = l / a.nct, n0 = (l - gr * a.nct) * BN;
  const int b0 = (int)((int64_t)gr * a.nblk / a.groups);
  const int nb = (int)((int64_t)(gr + 1) * a.nblk / a.groups) - b0;
  const int nt = (nb + a.tmax - 1) / a.tmax;
  auto tile0 = [&](int t) { return b0 + t * nb / nt; };  // first block of tile t (tile nt: the end)
  const int Hp = a.H + 2, Wp = a.W + 2;
  const int nch = a.Ck / 64, ntr = 3 * nch, nsl = 3 * ntr;  // chunks; triples and slabs of a tile
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  const uint32_t ldsw = lds0, ldsa = lds0 + WRING, ldsx = ldsa + ARING;

  if (wave >= 10) {
    // --------------------------------------------------------------- weight loaders
    constexpr int QW = WSLOT / 2048;  // 1 KB blocks per wave
    const int ww = wave - 10;
    const i32x4 rw = buf_rsrc(a.w, (uint32_t)a.w_bytes);
    uint32_t base[QW], dst[QW];
#pragma unroll
    for (int q = 0; q < QW; ++q) {
      const int blk = QW * ww + q;
      if constexpr (!TR) {
        // W row n0 + 8 blk + lane/8 (rows past C_out: past the buffer), chunk (lane%8) ^ swz
        const int r = 8 * blk + (lane >> 3);
        const int c = (lane & 7) ^ cv_swz_kc(r);
        base[q] = n0 + r < a.Cn ? (uint32_t)(((int64_t)(n0 + r) * 9 * a.Ck + 8 * c) * 2) : OOB;
        dst[q] = (uint32_t)(blk * 1024);
      } else {
        // quarter h (input channels n0 + 64h ..), k-row (output channel) r of the slab
        const int h = blk >> 3, g = blk & 7;
        const int r = 8 * g + (lane >> 3);
        const int c = (lane & 7) ^ cv_swz_tr(r);
        base[q] = n0 + 64 * h < a.Cn ? (uint32_t)(((int64_t)r * 9 * a.Ci + n0 + 64 * h + 8 * c) * 2) : OOB;
        dst[q] = (uint32_t)(h * CV_QSLOT + g * 1024);
      }
    }
    // the slab to issue next: tap column s of (kernel row r, chunk ch); its ring slot
    int s = 0, ch = 0, r = 0, left = nt * nsl;
    uint32_t slot = ldsw;
    auto issue = [&]() {
      const uint32_t off = TR ? (uint32_t)(((int64_t)ch * 64 * 9 + 3 * r + s) * a.Ci * 2)
                              : (uint32_t)(((3 * r + s) * a.Ck + ch * 64) * 2);
      // (a channel past the last one: OOB plus any slab's offset stays past the buffer)
      if (left-- > 0) {
#pragma unroll
        for (int q = 0; q < QW; ++q) dma16(rw, base[q] + off, slot + dst[q]);
      } else {  // no slab left: as many loads, all out of range
#pragma unroll
        for (int q = 0; q < QW; ++q) dma16(rw, OOB, slot + dst[q]);
      }
      slot = slot + WSLOT == ldsw + WRING ? ldsw : slot + WSLOT;
      if (++s == 3) {
        s = 0;
        if (++ch == nch) {
          ch = 0;
          r = r == 2 ? 0 : r + 1;
        }
      }
    };
#pragma unroll
    for (int S = 0; S < CV_NW - 2; ++S) issue();
    for (int t = 0; t < nt; ++t) {
      for (int S = 0; S < nsl; ++S) {
        vm_barrier<QW * (CV_NW - 3)>();  // slab S landed: B_S
        issue();                         // into the slot of S-2 (reads of S-1 may be in flight)
        if (WK == 2 && S == 0 && t > 0) {
          lds_barrier();  // the exchange of the tile before
          lds_barrier();
        }
      }
    }
    vm_barrier<0>();
    if (WK == 2) {
      lds_barrier();
      lds_barrier();
    }
  } else if (wave >= 8) {
    // ----------------------------------------------------------- activation loaders
    // LDS row u of a tile's slab is column e % (W+2) of the image row e / (W+2) rows after
    // the tile's first, e = u + (the first position's column): a piece ends with the two
    // columns after its last position, and the next row's piece starts at column 0.
    constexpr int QA = RA / 16;  // 8-row blocks per wave: blocks aw, aw + 2, ...
    const int aw = wave - 8;
    const i32x4 ra = buf_rsrc(a.act, (uint32_t)((int64_t)a.N * Hp * Wp * a.Ck * 2));
    const float invw = 1.0f / (float)Wp, invh = 1.0f / (float)a.H;
    uint32_t base[QA];
    int rows = 0;
    auto set_tile = [&](int t) {
      const int m0 = tile0(t) * 16, cnt = min(tile0(t + 1) * 16, a.M) - m0;
      const int hr0 = m0 / a.W, w0 = m0 - hr0 * a.W;
      const int img0 = hr0 / a.H, h0 = hr0 - img0 * a.H;
      rows = cnt + 2 * ((w0 + cnt - 1) / a.W) + 2;
#pragma unroll
      for (int q = 0; q < QA; ++q) {
        const int u = 8 * (2 * q + aw) + (lane >> 3);
        const int c = (lane & 7) ^ cv_swz_kc(u);
        const int e = u + w0, seg = cv_div(e, invw), col = e - seg * Wp;
        const int dn = cv_div(h0 + seg, invh), h = h0 + seg - dn * a.H;
        base[q] = u < rows ? (uint32_t)(((int64_t)(((img0 + dn) * Hp + h) * Wp + col) * a.Ck + 8 * c) * 2) : OOB;
      }
    };
    int ch = 0, r = 0;  // the triple to issue next
    uint32_t slot = ldsa;
    auto issue = [&]() {
      const uint32_t off = (uint32_t)(((int64_t)(TR ? 2 - r : r) * Wp * a.Ck + ch * 64) * 2);
      int left = rows - 8 * aw;
      asm volatile("" : "+s"(left));  // keeps the blocks' tests here: hoisted, they take 2 QA scalar registers
#pragma unroll
      for (int q = 0; q < QA; ++q)
        if (16 * q < left) dma16(ra, base[q] + off, slot + (uint32_t)((2 * q + aw) * 1024));
      slot = slot == ldsa ? ldsa + ASLOT : ldsa;
      if (++ch == nch) {
        ch = 0;
        r = r == 2 ? 0 : r + 1;
      }
    };
    set_tile(0);
    issue();
    for (int t = 0; t < nt; ++t) {
      for (int q = 0; q < ntr; ++q) {
        vm_barrier<0>();  // triple q landed: B_{3q}
        // into the slot of the triple before
        if (q + 1 < ntr) {
          issue();
        } else if (t + 1 < nt) {
          set_tile(t + 1);
          issue();
        }
        if (WK == 2 && q == 0 && t > 0) {
          lds_barrier();
          lds_barrier();
        }
        lds_barrier();
        lds_barrier();
      }
    }
    vm_barrier<0>();
    if (WK == 2) {
      lds_barrier();
      lds_barrier();
    }
  } else {
    // --------------------------------------------------------------- MMA group
    // The waves w and w + 4 share a SIMD: their position groups differ, so that a tile
    // whose groups hold unequal numbers of blocks still loads the SIMDs evenly.
    const int fi = lane & 15, kg = lane >> 4;
    const int hi = wave >> 2;
    const int kh = WK == 2 ? hi : 0;
    const int c = WP == 4 ? (WK == 2 ? 0 : hi) : (wave >> 1) & 1;
    const int p = WP == 4 ? (wave + 2 * hi) & 3 : (wave ^ hi) & 1;
    const bool live = n0 + 64 * c < a.Cn;
    const float invw = 1.0f / (float)a.W;
    uint32_t fx;  // weight fragment of block 0, k-step kh
    if constexpr (!TR) {
      fx = (uint32_t)((64 * c + fi) * 128 + (((4 * kh + kg) ^ cv_swz_kc(fi)) * 16));
    } else {
      // k-rows 8kg + fi/4 (+4) at channels 16j + 4(fi%4) of quarter c: the transpose
      // read hands lane fi the four consecutive k of channel 16j + fi (block j: chunk ^ 2j)
      const int r = 8 * kg + (fi >> 2);
      fx = (uint32_t)(c * CV_QSLOT + (32 * kh + r) * 128 + ((((fi >> 1) & 1) ^ cv_swz_tr(r)) * 16) + 8 * (fi & 1));
    }
    uint32_t ws = ldsw, as = ldsa;  // slots of the slab being read
    auto next_w = [&]() { ws = ws + WSLOT == ldsw + WRING ? ldsw : ws + WSLOT; };
    lds_barrier();  // B_0: slab 0 landed

    auto tile = [&](auto nbtag, int t, int first) {
      constexpr int NB = decltype(nbtag)::value;  // position blocks of the wave, from block `first`
      const int m0 = tile0(t) * 16, w0 = m0 % a.W;
      uint32_t adr[3][NB];  // activation fragments of k-step kh (tap column, block)
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int pos = 16 * (first + i) + fi;
        const int u = pos + 2 * cv_div(w0 + pos, invw);
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const int row = u + (TR ? 2 - s : s);
          adr[s][i] = (uint32_t)(row * 128 + (((4 * kh + kg) ^ cv_swz_kc(row)) * 16));
        }
      }
      f32x4 acc[NB][4];
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      // Fragments: the activations' in place (block i is read anew as soon as its MFMAs have
      // been issued), the weights' in two sets.
      bf16x8 av[NB], wv[2][4];
      auto read_a = [&](int s, int k, int i) {
        const uint32_t kx = (uint32_t)(64 * k);  // four chunks on
        av[i] = __builtin_bit_cast(bf16x8, *(const __attribute__((address_space(3))) u32x4 *)(uintptr_t)(as + (adr[s][i] ^ kx)));
      };
      auto read_w = [&](int k, bf16x8 (&wd)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (!TR) {
            wd[j] = __builtin_bit_cast(bf16x8, *(const __attribute__((address_space(3))) u32x4 *)(uintptr_t)(ws + (fx ^ (uint32_t)(64 * k)) + (uint32_t)(2048 * j)));
          } else {
            lds_i16x4 *q = (lds_i16x4 *)(uintptr_t)(ws + (fx ^ (uint32_t)(32 * j)) + (uint32_t)(k * 4096));
            const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(q);
            const i16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(q + 4 * 128 / 8);
            wd[j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
          }
        }
      };
      // One k-step: the MFMAs of the fragments at hand (weight set `cur`), and between them
      // the reads of the next k-step (tap column s, step k of the slab at ws / as).
      auto step = [&](auto curtag, int s, int k) {
        constexpr int cur = decltype(curtag)::value;
        read_w(k, wv[cur ^ 1]);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[cur][j], av[i], acc[i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          read_a(s, k, i);
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      // The barrier between two slabs, B_{S+1}. A weight slot is written anew two slabs after
      // its last reads were issued (every one of them has been waited for by then), an
      // activation slot right after the barrier that ends its triple, which waits for them.
      auto slab_end = [&](int s) {
        if (s == 2) {
          lds_barrier();
          as = as == ldsa ? ldsa + ASLOT : ldsa;
        } else {
          asm volatile("s_barrier" : : : "memory");
        }
        next_w();
      };
#pragma unroll
      for (int i = 0; i < NB; ++i) read_a(0, 0, i);
      read_w(0, wv[0]);
      // (past a tile's last slab the next tile's slab is read at this tile's rows, unused)
      if constexpr (WK == 1) {
        for (int q = 0; q < ntr; ++q) {
#pragma unroll
          for (int s = 0; s < 3; ++s) {
            step(CvInt<0>{}, s, 1);
            slab_end(s);
            step(CvInt<1>{}, (s + 1) % 3, 0);
          }
        }
      } else {
        // the wave's k-step of each slab
        auto triple = [&](auto partag) {
          constexpr int par = decltype(partag)::value;
#pragma unroll
          for (int s = 0; s < 3; ++s) {
            slab_end(s);
            if ((par + s) & 1) step(CvInt<1>{}, (s + 1) % 3, 0);
            else step(CvInt<0>{}, (s + 1) % 3, 0);
          }
        };
        for (int q = 0;;) {
          triple(CvInt<0>{});
          if (++q == ntr) break;
          triple(CvInt<1>{});
          if (++q == ntr) break;
        }
        // the halves' sums: the second half's wave hands over its first two blocks and takes
        // the first's last two
        const uint32_t xs = ldsx + (uint32_t)((c * WP + p) * 8192 + lane * 16);
        auto xat = [&](int i, int j) {
          return (__attribute__((address_space(3))) f32x4 *)(uintptr_t)(xs + (uint32_t)(((i & 1) * 4 + j) * 1024));
        };
        auto give = [&](int i0) {
#pragma unroll
          for (int i = i0; i < i0 + 2; ++i)
            if (i < NB)
#pragma unroll
              for (int j = 0; j < 4; ++j) *xat(i, j) = acc[i < NB ? i : 0][j];
        };
        auto take = [&](int i0) {
#pragma unroll
          for (int i = i0; i < i0 + 2; ++i)
            if (i < NB)
#pragma unroll
              for (int j = 0; j < 4; ++j) acc[i < NB ? i : 0][j] += *xat(i, j);
        };
        if (kh == 1) give(0);
        lds_barrier();
        if (kh == 0) {
          take(0);
          give(2);
        }
        lds_barrier();
        if (kh == 1) take(2);
      }
      // ---- write the tile: lane (fi, kg) holds channels 16j + 4kg .. +3 of position fi of
      // each block; bf16: blocks 2t and 2t+1 exchanged between the lanes so that each
      // holds eight channels
      const int nc0 = n0 + 64 * c;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (WK == 2 && (i >> 1) != kh) continue;
        const int pos = m0 + 16 * (first + i) + fi;
        if (a.out_bf16) {
          uint16_t *o = reinterpret_cast<uint16_t *>(a.out) + (int64_t)pos * a.Cn + nc0 + 16 * (kg & 1) + 8 * (kg >> 1);
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const f32x4 x = acc[i][2 * b], y = acc[i][2 * b + 1];
            const auto lo = __builtin_amdgcn_permlane16_swap(cvt_pk_bf16(x[0], x[1]), cvt_pk_bf16(y[0], y[1]), false, false);
            const auto up = __builtin_amdgcn_permlane16_swap(cvt_pk_bf16(x[2], x[3]), cvt_pk_bf16(y[2], y[3]), false, false);
            if (pos < a.M) *reinterpret_cast<u32x4 *>(o + 32 * b) = u32x4{lo[0], up[0], lo[1], up[1]};
          }
        } else if (pos < a.M) {
          float *o = reinterpret_cast<float *>(a.out) + (int64_t)pos * a.Cn + nc0 + 4 * kg;
#pragma unroll
          for (int j = 0; j < 4; ++j) *reinterpret_cast<f32x4 *>(o + 16 * j) = acc[i][j];
        }
      }
    };

    for (int t = 0; t < nt; ++t) {
      // the tile's blocks over the position groups, as evenly as they go
      const int n = tile0(t + 1) - tile0(t);
      const int mine = live ? n / WP + (p < n % WP ? 1 : 0) : 0, first = p * (n / WP) + min(p, n % WP);
      switch (mine) {
        case 4: tile(CvInt<4>{}, t, first); break;
        case 3: tile(CvInt<3>{}, t, first); break;
        case 2: tile(CvInt<2>{}, t, first); break;
        case 1: tile(CvInt<1>{}, t, first); break;
        default:  // no block here: the slab barriers (and the exchange's)
          for (int S = 0; S < nsl + (WK == 2 ? 2 : 0); ++S) lds_barrier();
          // the ring positions after the tile
          for (int S = 0; S < nsl % CV_NW; ++S) next_w();
          if (ntr & 1) as = as == ldsa ? ldsa + ASLOT : ldsa;
      }
    }
  }
}


// ------------------------------------------------------------------ weight gradient
// dW[o][tap][c] = sum_p dy[p][o] * x_pad[P(p) + r*(W+2) + s][c] over the tile's output
// positions p = (n, h, w), P(p) = (n (H+2) + h) (W+2) + w (Sec. 2.2: the tile's partial of
// the weight gradient, which the all-reduce over the domain completes). Both operands are
// position-major, so K = positions and both fragments come from k-row-major LDS slabs
// through the transpose read. A workgroup owns 256 output channels x 128 input channels
// of one tap over one range of output positions; the ranges are K splits whose fp32
// partials the split-K reduce adds in split order. Slabs of 64 positions, each row's
// padded-grid row P(p) kept incrementally by the loader lane that fetches it:
//  * waves 6-7 load the Delta_Y slab (64 positions x 256 channels, four 64-channel
//    quarters);
//  * waves 4-5 load the shifted activation slab (64 positions x 128 channels);
//  * waves 0-3 each accumulate 128 output channels x 64 input channels.
// Rows past the split's range read as zero (their loads are out of range).
struct CwArgs {
  const uint16_t *x;    // x_pad [N][H+2][W+2][Ci]
  const uint16_t *dy;   // interior start of dy_pad: dy_pad + ((W+2) + 1) * Co
  float *partial;       // [split][Co][ldp]: element (tap*Ci + c, o) at o*ldp + tap*Ci + c
  int64_t ldp, sstride;
  int H, W, Ci, Co;
  int M, k_split, splits, tiles;  // output positions N*H*W; tiles = 9 * Ci / 128
  int Mp;                         // padded-grid rows up to the last output position's
};

constexpr int CW_XSLOT = 64 * 256;   // 16 KB: 64 positions x 128 channels
constexpr int CW_DSLOT = 64 * 512;   // 32 KB: 64 positions x 256 channels
constexpr int CW_NX = 4, CW_ND = 3;  // ring slots
constexpr int CW_PITCH = 128 + 4;    // staging row pitch in floats

// Output position p as (h, w) and its padded-grid row P(p); the step to position p + 64
// without a division (the rows that wrap past an image row or an image are counted).
__device__ __forceinline__ void cw_row_init(const CwArgs &a, int p, int *h, int *w, int *P) {
  const int HW = a.H * a.W, n = p / HW, rem = p - n * HW;
  *h = rem / a.W;
  *w = rem - *h * a.W;
  *P = (n * (a.H + 2) + *h) * (a.W + 2) + *w;
}
__device__ __forceinline__ void cw_row_next(const CwArgs &a, int *h, int *w, int *P) {
  const int Wp = a.W + 2, dh = 64 / a.W, dw = 64 - dh * a.W;
  *w += dw;
  *h += dh;
  *P += dh * Wp + dw;
  if (*w >= a.W) {
    *w -= a.W;
    ++*h;
    *P += 2;
  }
  while (*h >= a.H) {
    *h -= a.H;
    *P += 2 * Wp;
  }
}

__global__ void __launch_bounds__(512, 1) conv_wg_kernel(CwArgs a) {
  constexpr uint32_t OOB = 0x80000000u;
  constexpr int DRING = CW_ND * CW_DSLOT, XRING = CW_NX * CW_XSLOT;
  __shared__ __attribute__((aligned(1024))) char smem[DRING + XRING];
  static_assert(DRING + XRING <= 160 * 1024, "LDS");
  static_assert(256 * CW_PITCH * 4 <= DRING + XRING, "staging");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // padded to a multiple of 8: the tiles of one split (which read the same positions) run
  // on one XCD
  const int G = gridDim.x;
  const int b = (blockIdx.x & 7) * (G >> 3) + (blockIdx.x >> 3);
  if (b >= a.tiles * a.splits) return;
  const int split = b / a.tiles, tile = b - split * a.tiles;
  const int tap = tile / (a.Ci / 128), c0 = (tile - tap * (a.Ci / 128)) * 128;
  const int klo = split * a.k_split, krange = min(a.M, klo + a.k_split) - klo;
  const int nsl = krange > 0 ? (krange + 63) / 64 : 0;
  const int Wp = a.W + 2;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  const uint32_t ldsd = lds0, ldsx = lds0 + DRING;

  if (wave >= 6) {
    // ---------------------------------------------------- Delta_Y loaders (6, 7)
    // blocks 16dw..16dw+15 of a slot: quarter h = blk/8, k-rows 8(blk%8)..+7
    const int dw = wave - 6;
    const i32x4 rd = buf_rsrc(a.dy, (uint32_t)((int64_t)a.Mp * a.Co * 2));
    // the wave's blocks cover quarters 2dw, 2dw+1 of the same 8 row groups g (k-rows
    // 8g + lane/8)
    uint32_t col[2][8];
    int hh[8], ww[8], pp[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const int r = 8 * g + (lane >> 3);
      const int c = (lane & 7) ^ cv_swz_tr(r);
      col[0][g] = (uint32_t)((64 * (2 * dw) + 8 * c) * 2);
      col[1][g] = (uint32_t)((64 * (2 * dw + 1) + 8 * c) * 2);
      cw_row_init(a, klo + r, &hh[g], &ww[g], &pp[g]);
    }
    auto issue = [&](int S) {
      const uint32_t slot = ldsd + (uint32_t)((S % CW_ND) * CW_DSLOT);
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        const int r = 8 * g + (lane >> 3);
        const bool ok = S < nsl && S * 64 + r < krange;
        const uint32_t off = (uint32_t)pp[g] * (uint32_t)(a.Co * 2);
#pragma unroll
        for (int hq = 0; hq < 2; ++hq)
          dma16(rd, ok ? off + col[hq][g] : OOB, slot + (uint32_t)((2 * dw + hq) * CV_QSLOT + g * 1024));
        cw_row_next(a, &hh[g], &ww[g], &pp[g]);
      }
    };
#pragma unroll
    for (int S = 0; S < CW_ND - 1; ++S) issue(S);
    for (int S = 0; S < nsl; ++S) {
      vm_barrier<16 * (CW_ND - 2)>();  // slab S landed: B_S
      issue(S + CW_ND - 1);            // into the slot of S-1
    }
    vm_barrier<0>();
  } else if (wave >= 4) {
    // --------------------------------------------------- activation loaders (4, 5)
    // quarter h = blk/8 (channels c0 + 64h ..), k-rows 8(blk%8).. of positions shifted by tap
    const int xw = wave - 4;
    const int r3 = tap / 3, s3 = tap - 3 * r3, shift = r3 * Wp + s3;
    const i32x4 rx = buf_rsrc(a.x, (uint32_t)((int64_t)(a.Mp + 2 * Wp + 2) * a.Ci * 2));
    // block q of the wave's quarter: k-rows 8q + lane/8
    uint32_t col[8];
    int hh[8], ww[8], pp[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = 8 * q + (lane >> 3);
      const int c = (lane & 7) ^ cv_swz_tr(r);
      col[q] = (uint32_t)((c0 + 64 * xw + 8 * c) * 2);
      cw_row_init(a, klo + r, &hh[q], &ww[q], &pp[q]);
    }
    auto issue = [&](int S) {
      const uint32_t slot = ldsx + (uint32_t)((S % CW_NX) * CW_XSLOT) + (uint32_t)(xw * CV_QSLOT);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int r = 8 * q + (lane >> 3);
        const bool ok = S < nsl && S * 64 + r < krange;
        const uint32_t off = (uint32_t)(pp[q] + shift) * (uint32_t)(a.Ci * 2);
        dma16(rx, ok ? off + col[q] : OOB, slot + (uint32_t)(q * 1024));
        cw_row_next(a, &hh[q], &ww[q], &pp[q]);
      }
    };
#pragma unroll
    for (int S = 0; S < CW_NX - 1; ++S) issue(S);
    for (int S = 0; S < nsl; ++S) {
      vm_barrier<8 * (CW_NX - 2)>();  // slab S landed: B_S
      issue(S + CW_NX - 1);           // into the slot of S-1
    }
    vm_barrier<0>();
  } else {
    // --------------------------------------------------------------- MMA group
    // wave (wm, wn): output channels 128wm.. (Delta_Y quarters 2wm, 2wm+1), input channels
    // 64wn.. (activation quarter wn)
    constexpr int FM = 8;
    const int fi = lane & 15, kg = lane >> 4;
    const int wm = wave & 1, wn = wave >> 1;
    const int r = 8 * kg + (fi >> 2);
    uint32_t fa[FM], fx[4];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int mb = 8 * wm + i, h = mb >> 2, ib = mb & 3;
      const int c = (2 * ib + ((fi >> 1) & 1)) ^ cv_swz_tr(r);
      fa[i] = (uint32_t)(h * CV_QSLOT + r * 128 + c * 16 + 8 * (fi & 1));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = (2 * j + ((fi >> 1) & 1)) ^ cv_swz_tr(r);
      fx[j] = (uint32_t)(wn * CV_QSLOT + r * 128 + c * 16 + 8 * (fi & 1));
    }
    f32x4 acc[FM][4];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto tr8 = [&](uint32_t addr) {
      lds_i16x4 *p = (lds_i16x4 *)(uintptr_t)addr;
      const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(p);
      const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(p + 4 * 128 / 8);
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    bf16x8 dv[2][FM], xv[2][4];
    auto read = [&](uint32_t ds, uint32_t xs, int s, bf16x8 (&dd)[FM], bf16x8 (&xd)[4]) {
#pragma unroll
      for (int i = 0; i < FM; ++i) dd[i] = tr8(ds + fa[i] + (uint32_t)(s * 4096));
#pragma unroll
      for (int j = 0; j < 4; ++j) xd[j] = tr8(xs + fx[j] + (uint32_t)(s * 4096));
    };
    // One 32-k step: its 32 MFMAs in eight groups (row block g against the four column
    // blocks), with the next step's twelve fragments (24 transpose reads) read two per group
    // in the first six, the column blocks and the first row blocks first (the next step's
    // first groups use them). Reading all 24 ahead of the MFMAs made every step wait for ten
    // of them: the LDS counter tracks at most 15 operations, so the wait that the older
    // fragments need also covers the oldest of the new reads. The last two groups' MFMAs
    // cover the reads before the next step or the slab barrier.
    auto step = [&](const bf16x8 (&df)[FM], const bf16x8 (&xf)[4], uint32_t dsn, uint32_t xsn, int sn,
                    bf16x8 (&dd)[FM], bf16x8 (&xd)[4]) {
#pragma unroll
      for (int g = 0; g < FM; ++g) {
        if (g < 6) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int f = 2 * g + h;
            if (f < 4) xd[f] = tr8(xsn + fx[f] + (uint32_t)(sn * 4096));
            else dd[f - 4] = tr8(dsn + fa[f - 4] + (uint32_t)(sn * 4096));
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[g][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(df[g], xf[j], acc[g][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    uint32_t ds = ldsd, xs = ldsx;
    if (nsl > 0) {
      lds_barrier();  // B_0
      read(ds, xs, 0, dv[0], xv[0]);
    }
    for (int S = 0; S < nsl; ++S) {
      step(dv[0], xv[0], ds, xs, 1, dv[1], xv[1]);
      lds_barrier();  // B_{S+1}
      ds = ldsd + (uint32_t)(((S + 1) % CW_ND) * CW_DSLOT);
      xs = ldsx + (uint32_t)(((S + 1) % CW_NX) * CW_XSLOT);
      step(dv[1], xv[1], ds, xs, 0, dv[0], xv[0]);  // past the last slab this reads a spent slot, unused
    }
    if (nsl == 0) lds_barrier();  // the loaders' B_0 (they pass vm_barrier<0> once)
    // ---- stage the tile as [output channel][input channel] fp32
    float *stg = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          stg[(16 * (8 * wm + i) + 4 * kg + e) * CW_PITCH + 16 * (4 * wn + j) + fi] = acc[i][j][e];
  }
  lds_barrier();
  // ---- partial tile out: 256 rows of 128 floats (512 B), device-scope stores
  const float *stg = reinterpret_cast<const float *>(smem);
  float *dst = a.partial + (int64_t)split * a.sstride + tap * a.Ci + c0;
  const __amdgpu_buffer_rsrc_t prs =
      __builtin_amdgcn_make_buffer_rsrc(dst, 0, (int)(((int64_t)(a.Co - 1) * a.ldp + 128) * 4), BUF_DW3);
  const int ch = tid & 31, sub = tid >> 5;
#pragma unroll
  for (int p = 0; p < 16; ++p) {
    const int o = 16 * p + sub;
    const f32x4 v = *reinterpret_cast<const f32x4 *>(stg + o * CW_PITCH + 4 * ch);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), prs, (uint32_t)((o * a.ldp + 4 * ch) * 4), 0, 16);
  }
}

}  // namespace

bool conv_nt_fits(int pass, int N, int H, int W, int Ci, int Co, const void *act, const void *w, const void *out) {
  if (opt(IMBD_OPT_CONV_NT) == 0) return false;  // the tiled GEMM template instead
  const int Cn = pass == 1 ? Co : Ci, Ck = pass == 1 ? Ci : Co;
  auto al = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) % 16) == 0; };
  // byte offsets of both operands within one buffer descriptor; image rows and columns
  // within the range of the kernel's short divisions
  return (pass == 1 || pass == 2) && N >= 1 && H >= 1 && W >= 1 && Cn >= 64 && Cn % 64 == 0 && Ck >= 64 &&
         Ck % 64 == 0 && al(act) && al(w) && al(out) && H < 32768 && W < 32768 &&
         (int64_t)N * (H + 2) * (W + 2) * Ck * 2 < ((int64_t)1 << 31) &&
         (int64_t)9 * Ci * Co * 2 < ((int64_t)1 << 31);
}

bool conv_wg_fits(int N, int H, int W, int Ci, int Co, const void *x, const void *dy, const void *dw) {
  if (opt(IMBD_OPT_CONV_NT) == 0) return false;
  auto al = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) % 16) == 0; };
  const int64_t rows = (int64_t)N * (H + 2) * (W + 2) + 2 * (W + 2) + 2 + 64;
  return N >= 1 && H >= 1 && W >= 1 && Co == 256 && Ci >= 128 && Ci % 128 == 0 && al(x) && al(dy) && al(dw) &&
         rows * (Ci > Co ? Ci : Co) * 2 < ((int64_t)1 << 31);
}

void conv_wg_plan(int N, int H, int W, int Ci, int *splits, int *k_split) {
  const int64_t M = (int64_t)N * H * W;
  const int tiles = 9 * Ci / 128;
  int s = 256 / tiles;
  if (s < 1) s = 1;
  int ks = (int)((M + s - 1) / s + 63) / 64 * 64;
  if (ks < 64) ks = 64;
  *k_split = ks;
  *splits = (int)((M + ks - 1) / ks);
}

int run_conv_wg(int N, int H, int W, int Ci, int Co, const void *x, const void *dy_pad, float *partial,
                int64_t ldp, int64_t sstride, hipStream_t s) {
  CwArgs a;
  a.x = reinterpret_cast<const uint16_t *>(x);
  a.dy = reinterpret_cast<const uint16_t *>(dy_pad) + (int64_t)(W + 3) * Co;
  a.partial = partial;
  a.ldp = ldp;
  a.sstride = sstride;
  a.H = H;
  a.W = W;
  a.Ci = Ci;
  a.Co = Co;
  a.M = N * H * W;
  a.Mp = (int)((int64_t)(N - 1) * (H + 2) * (W + 2) + (int64_t)(H - 1) * (W + 2) + W);
  conv_wg_plan(N, H, W, Ci, &a.splits, &a.k_split);
  a.tiles = 9 * Ci / 128;
  const int grid = (a.tiles * a.splits + 7) / 8 * 8;
  {
    LaunchTimer t(IMBD_K_CONV_WGRAD, 0, s);
    hipLaunchKernelGGL(conv_wg_kernel, dim3(grid), dim3(512), 0, s, a);
  }
  return check_launch("conv_wg");
}

int run_conv_nt(int pass, int N, int H, int W, int Ci, int Co, const void *act, const void *w, void *out,
                int out_dtype, hipStream_t s) {
  CvArgs a;
  a.act = reinterpret_cast<const uint16_t *>(act);
  a.w = reinterpret_cast<const uint16_t *>(w);
  a.out = out;
  a.out_bf16 = out_dtype == IMBD_BF16 ? 1 : 0;
  a.N = N;
  a.H = H;
  a.W = W;
  a.Ck = pass == 1 ? Ci : Co;
  a.Cn = pass == 1 ? Co : Ci;
  a.Ci = Ci;
  a.w_bytes = (int64_t)9 * Ci * Co * 2;
  a.M = N * H * W;
  a.nblk = (a.M + 15) / 16;
  const bool narrow = a.Cn == 64;
  a.nct = narrow ? 1 : (a.Cn + 127) / 128;
  // one workgroup per CU (the LDS of each), every one with a share of the position blocks
  a.groups = std::max(1, std::min(a.nblk, CV_CUS / a.nct));
  const int share = (a.nblk + a.groups - 1) / a.groups;
  const int o = opt(IMBD_OPT_CONV_NT);
  const bool tall = narrow || share > 8 || o >= 2;
  // blocks per tile: what the MMA waves hold and what the activation slab's rows allow (a
  // tile of n positions touches at most (W - 1 + n - 1) / W + 1 image rows)
  const int cap = cv_slab_rows(tall ? 4 : 2);
  a.tmax = tall ? 16 : 8;
  if (o >= 2) a.tmax = o == 2 ? 8 : 7;
  while (a.tmax > 1 && 16 * a.tmax + 2 * ((W + 16 * a.tmax - 2) / W) + 2 > cap) --a.tmax;
  const int grid = (a.groups * a.nct + 7) / 8 * 8;
  {
    LaunchTimer t(pass == 1 ? IMBD_K_CONV_FWD : IMBD_K_CONV_DGRAD, 0, s);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(768), 0, s, a); };
    if (narrow) pass == 1 ? go(conv_nt_kernel<false, 4, 2>) : go(conv_nt_kernel<true, 4, 2>);
    else if (tall) pass == 1 ? go(conv_nt_kernel<false, 4, 1>) : go(conv_nt_kernel<true, 4, 1>);
    else pass == 1 ? go(conv_nt_kernel<false, 2, 2>) : go(conv_nt_kernel<true, 2, 2>);
  }
  return check_launch("conv_nt");
}

}  // namespace imbd
