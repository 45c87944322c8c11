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
//  * waves 10-11 stream the weight slabs (BN channels x 64 k of one tap) through five (four)
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
// NARROW (images of few columns, whose tiles touch many image rows): more of them, and four
// weight slots instead of five.
constexpr int cv_slab_rows(int wp, bool narrow = false) { return narrow ? 384 : wp == 4 ? 304 : 160; }
constexpr int cv_weight_slots(bool narrow) { return narrow ? 4 : 5; }

__device__ __forceinline__ int cv_swz_kc(int r) { return r & 7; }
__device__ __forceinline__ int cv_swz_tr(int r) { return 2 * ((r >> 1) & 1) + 4 * ((r >> 3) & 1); }
template <int V>
struct CvInt {
  static constexpr int value = V;
};
// x / d for 0 <= x < 2^22 (inv = 1 / d, rounded): the half keeps the quotient 0.5 / d away from
// whole numbers, its two roundings move it by less than (x / d) 2^-23
constexpr int CV_SIDE_MAX = 1 << 21;  // image rows and columns of the kernels, which add a tile's to them
__device__ __forceinline__ int cv_div(int x, float inv) { return (int)(((float)x + 0.5f) * inv); }

// TR: input gradient (W read transposed); else forward.
template <bool TR, int WP, int WK, bool NARROW = false>
__global__ void __launch_bounds__(768, 1) conv_nt_kernel(CvArgs a) {
  constexpr int WC = 8 / (WP * WK);
  constexpr int BN = 64 * WC;
  constexpr int RA = cv_slab_rows(WP, NARROW), CV_NW = cv_weight_slots(NARROW);
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
// through the transpose read.
//
// A workgroup owns OB = 64 WO output channels x 64 input channels x the three taps of one
// kernel row over one range of positions. The three taps share both slabs: the Delta_Y slab
// (64 positions x OB channels) and the activation slab (per image row piece of the slab its
// positions and the two columns after them, 64 channels), of which a tap reads the rows
// from its column on: 27 KB into LDS per 48 x 16 MFMAs, where one tap of 128 input
// channels with slabs of its own took 32 KB per 32 x 16. The ranges are K splits, whose
// fp32 partials a flat reduce adds in split order (one range writes dW itself).
//
// Eight MMA waves, each 64 output channels x 32 input channels x 3 taps:
//   WO = 2, WK = 2: 128 output channels, the two 32-position steps of each slab to two
//     halves of the waves, whose sums are added through LDS at the end (five slabs of ring);
//   WO = 4, WK = 1: 256 output channels, every wave both steps (three slabs).
// Images of one to three columns (NARROW, the former layout): 64 positions touch up to 64
// image rows, so an activation slab has up to 192 rows in a slot twice as large, and three
// slabs fit.
// What bounds it is the issue of the MMA waves' other instructions, which the two waves of
// a SIMD, in step through the slab barriers, do not hide from each other. Left to them are
// the fragment reads and ten instructions per slab for the fragments' rows; four loader
// waves do the rest. At 32 x 56 x 56, 256 -> 256 (kernel and reduce): every wave issuing an
// eighth of the loads and working out swizzled rows per tap 148 us, the rows linear (160
// bytes apart instead of swizzled, a tap then is an offset) 123, the loads on waves of
// their own and both operands' fragments read anew in place 110 (with a second Delta_Y
// set the registers spilled: 170), the reduce with four loads instead of eight in flight
// on a sixth of the registers 104; the one-tap kernel before 118. Measured (us, before ->
// after; other channel counts than 256 were on the tiled GEMM template):
//   64 x 13 x 13, 384 -> 384: 137 -> 40.5      32 x 14 x 14, 512 -> 512: 179 -> 41.7
//   32 x 56 x 56,  64 -> 128: 200 -> 26.9      16 x 56 x 56, 192 -> 320: 685 -> 62.4
// Rows past the range read as zero in Delta_Y, and the positions there read a zero row of
// the activation slab, so no infinity of a neighbouring row reaches a sum.
struct CwArgs {
  const uint16_t *x;    // x_pad [N][H+2][W+2][Ci]
  const uint16_t *dy;   // dy_pad [N][H+2][W+2][Co]
  float *out;           // [split][Co][3][3][Ci], or dW when there is one split
  int64_t sstride;      // floats from one split to the next
  uint32_t x_bytes, dy_bytes, out_bytes;
  int H, W, Ci, Co;
  int M, k_split, splits, tiles;  // output positions N*H*W; tiles of one split
  int tco;                        // output-channel tiles
  int xblk;                       // 1 KB blocks of an activation slab in use
  int dh, dw;                     // 64 / W, 64 % W: 64 positions on
};

// An activation slab: up to 98 rows of 64 channels and three zero rows, 160 bytes apart (ten
// 16-byte chunks, the last two unused): a transpose read of 16 consecutive rows x 16 channels
// touches every bank twice whatever row it starts at, and a tap is an offset of 160 bytes.
constexpr int CW_XPITCH = 160;
constexpr int cw_xrows(bool narrow) { return narrow ? 192 : 98; }
constexpr int cw_xslot(bool narrow) { return (narrow ? 32 : 16) * 1024; }
static_assert((cw_xrows(false) + 3) * CW_XPITCH <= cw_xslot(false) && (cw_xrows(true) + 3) * CW_XPITCH <= cw_xslot(true),
              "activation slab");

// rows of a slab: 64 positions touch at most (w + 62) / w + 1 image rows
constexpr int cw_slab_rows(int w) { return 64 + 2 * ((w + 62) / w) + 2; }
constexpr bool cw_narrow(int w) { return cw_slab_rows(w) > cw_xrows(false); }
static_assert(cw_slab_rows(1) <= cw_xrows(true) && cw_narrow(3) && !cw_narrow(4), "every width fits a slab");

// 16-byte chunk swizzle of a Delta_Y row (128 bytes apart), to the same end.
__device__ __forceinline__ int cw_swz(int r) { return ((r >> 1) & 3) << 1; }

template <int WO, int WK, bool NARROW>
__global__ void __launch_bounds__(768, 1) conv_wg_kernel(CwArgs a) {
  static_assert((WO == 2 && WK == 2) || (WO == 4 && WK == 1), "eight waves, two per 64-channel half");
  constexpr uint32_t OOB = 0x80000000u;
  static_assert(!NARROW || WK == 2, "three slots fit");
  constexpr int CW_XROWS = cw_xrows(NARROW);
  constexpr int DSLOT = WO * CV_QSLOT, SLOT = DSLOT + cw_xslot(NARROW);
  constexpr int NS = WK == 2 && !NARROW ? 5 : 3;
  // slabs issued ahead of the one being read: a slot is written anew two slabs after its last
  // reads were issued (they need not have landed at the barrier in between), or, with three
  // slots, after a barrier that waits for them
  constexpr int AHEAD = NS == 5 ? NS - 2 : NS - 1;
  __shared__ __attribute__((aligned(1024))) char smem[NS * SLOT];
  static_assert(NS * SLOT <= 160 * 1024, "LDS");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the tiles of one split (which read the same positions) run on one XCD
  const int G = gridDim.x;
  const int l = (int)(blockIdx.x & 7) * (G >> 3) + (int)(blockIdx.x >> 3);
  if (l >= a.tiles * a.splits) return;
  const int split = l / a.tiles;
  int tile = l - split * a.tiles;
  const int o0 = (tile % a.tco) * 64 * WO;
  tile /= a.tco;
  const int r3 = tile % 3, c0 = (tile / 3) * 64;
  const int klo = split * a.k_split, kend = min(a.M, klo + a.k_split);
  const int nsl = (kend - klo + 63) / 64;
  const int Hp = a.H + 2, Wp = a.W + 2;
  const float invw = 1.0f / (float)a.W;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  auto up = [&](uint32_t slot) { return slot + SLOT == lds0 + NS * SLOT ? lds0 : slot + SLOT; };

  // the zero rows of each activation slot
  for (int i = tid; i < NS * 32; i += 768)
    if ((i & 31) < 30)
      *reinterpret_cast<u32x4 *>(smem + (i >> 5) * SLOT + DSLOT + CW_XROWS * CW_XPITCH + (i & 31) * 16) = u32x4{0u, 0u, 0u, 0u};
  lds_barrier();

  if (wave >= 8) {
    // ---- loaders: Delta_Y (waves 8, 9) and activations (10, 11). The rows of an activation
    // slab are one run of the padded grid (two halo rows more at each image's end), so within
    // an image their offsets are a lane constant plus a scalar; Delta_Y's skip two columns
    // per image row.
    const float invwp = 1.0f / (float)Wp, invh = 1.0f / (float)a.H;
    const int w2 = wave & 1;
    // the slab to issue: its first position q0 = (row h0 of its image, column w0), row P0 of
    // the padded grid
    int q0 = klo, h0, w0, P0;
    {
      const int hr = klo / a.W, n = hr / a.H;
      w0 = klo - hr * a.W;
      h0 = hr - n * a.H;
      P0 = (n * Hp + h0) * Wp + w0;
    }
    uint32_t slot = lds0;
    auto crosses = [&]() {  // whether the 64 positions reach another image: row h0 + (w0 + 63) / W
      const int t63 = w0 + a.dw - 1;
      return h0 + a.dh + (t63 >= a.W ? 1 : 0) - (t63 < 0 ? 1 : 0) >= a.H;
    };
    auto next = [&]() {
      slot = up(slot);
      q0 += 64;
      w0 += a.dw;
      h0 += a.dh;
      P0 += a.dw + a.dh * Wp;
      if (w0 >= a.W) {
        w0 -= a.W;
        ++h0;
        P0 += 2;
      }
      while (h0 >= a.H) {
        h0 -= a.H;
        P0 += 2 * Wp;
      }
    };
    auto run = [&](auto ntag, auto issue) {  // N loads a slab
      constexpr int N = decltype(ntag)::value;
#pragma unroll
      for (int S = 0; S < AHEAD; ++S) issue(ntag);
      for (int S = 0; S <= nsl; ++S) {
        vm_barrier<N * (AHEAD - 1)>();  // slab S landed: B_S
        issue(ntag);
      }
    };
    if (wave < 10) {
      // row groups 4 w2 .. 4 w2 + 3 (8 positions each) of every 64-channel quarter
      const i32x4 rd = buf_rsrc(a.dy, a.dy_bytes);
      const uint32_t d2 = (uint32_t)(a.Co * 2);
      uint32_t base[4];
      float rowf[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int r = 32 * w2 + 8 * g + (lane >> 3);
        base[g] = (uint32_t)(r + Wp + 1) * d2 + (uint32_t)((o0 + 8 * ((lane & 7) ^ cw_swz(r))) * 2);
        rowf[g] = (float)r + 0.5f;
      }
      run(CvInt<4 * WO>{}, [&](auto) {
        const uint32_t dP = (uint32_t)P0 * d2;
        const bool far = crosses(), last = q0 + 64 > kend;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int seg = (int)((rowf[g] + (float)w0) * invw);
          uint32_t off = base[g] + dP + (uint32_t)__umul24((uint32_t)seg, 2 * d2);
          if (far) off += (uint32_t)cv_div(h0 + seg, invh) * (uint32_t)(2 * Wp) * d2;
          if (last && 32 * w2 + 8 * g + (lane >> 3) >= kend - q0) off = OOB;
#pragma unroll
          for (int q = 0; q < WO; ++q)
            dma16(rd, o0 + 64 * q < a.Co ? off + (uint32_t)(128 * q) : OOB,
                  slot + (uint32_t)(q * CV_QSLOT + (4 * w2 + g) * 1024));
        }
        next();
      });
    } else {
      // 1 KB blocks w2, w2 + 2, .. of the slab: chunk L = 64 (w2 + 2q) + lane is chunk L % 10
      // (the last two unused) of row L / 10
      const i32x4 rx = buf_rsrc(a.x, a.x_bytes);
      const uint32_t x2 = (uint32_t)(a.Ci * 2);
      auto row = [&](int q) { return (64 * (w2 + 2 * q) + lane) / 10; };
      constexpr int QX = NARROW ? 15 : 8;
      uint32_t base[QX];
#pragma unroll
      for (int q = 0; q < QX; ++q) {
        const int c = 64 * (w2 + 2 * q) + lane - 10 * row(q);
        // (OOB plus any row's offset stays past the buffer)
        base[q] = c < 8 && row(q) < CW_XROWS ? (uint32_t)(row(q) + r3 * Wp) * x2 + (uint32_t)((c0 + 8 * c) * 2) : OOB;
      }
      auto issue = [&](auto ntag) {
        constexpr int N = decltype(ntag)::value;
        const uint32_t xP = (uint32_t)P0 * x2;
        if (!crosses() && q0 + 64 <= kend) {
#pragma unroll
          for (int q = 0; q < N; ++q) dma16(rx, base[q] + xP, slot + (uint32_t)(DSLOT + (w2 + 2 * q) * 1024));
        } else {
          // the slab goes on in the next image (or past several), or is the range's last one
          // (or past it): rows behind its last position's read as zero
          const int cnt = min(64, kend - q0), rows = cnt > 0 ? cnt + 2 * ((w0 + cnt - 1) / a.W) + 2 : 0;
#pragma unroll
          for (int q = 0; q < N; ++q) {
            const uint32_t skip = (uint32_t)cv_div(h0 + cv_div(w0 + row(q), invwp), invh) * (uint32_t)(2 * Wp) * x2;
            dma16(rx, base[q] != OOB && row(q) < rows ? base[q] + xP + skip : OOB,
                  slot + (uint32_t)(DSLOT + (w2 + 2 * q) * 1024));
          }
        }
        next();
      };
      const int mine = (a.xblk + 1 - w2) / 2;  // of 11 to 16 blocks; 17, 21 or 30 of narrow images
      if constexpr (NARROW) {
        if (mine <= 9) run(CvInt<9>{}, issue);
        else if (mine <= 11) run(CvInt<11>{}, issue);
        else run(CvInt<15>{}, issue);
      } else {
        switch (mine) {
          case 8: run(CvInt<8>{}, issue); break;
          case 7: run(CvInt<7>{}, issue); break;
          case 6: run(CvInt<6>{}, issue); break;
          default: run(CvInt<5>{}, issue);
        }
      }
    }
    vm_barrier<0>();  // every load landed
    if constexpr (WK == 2) lds_barrier();
    return;
  }

  // ---- MMA waves. A fragment's lane reads cover rows lane/4 and lane/4 + 16 of a 32-position
  // step (the lane's eight k are four consecutive rows of each, in both operands).
  const int fi = lane & 15, kg = lane >> 4;
  const int kh = WK == 2 ? wave >> 2 : 0;
  const int wo = WK == 2 ? wave & 1 : wave & 3, wc = WK == 2 ? (wave >> 1) & 1 : wave >> 2;
  const bool live = o0 + 64 * wo < a.Co;
  const int R = 32 * kh + (lane >> 2);
  uint32_t fd[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    fd[i] = (uint32_t)(wo * CV_QSLOT + R * 128 + ((32 * i) ^ (16 * cw_swz(R))) + 8 * (lane & 3));
  auto tr8 = [&](uint32_t p0, uint32_t p1) {
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(uintptr_t)p0);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(uintptr_t)p1);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  f32x4 acc[6][4];  // [tap column, 16-channel block][output-channel block]
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 xv[6], dv[4];  // fragments, read anew in place as soon as their last MFMA is issued
  uint32_t rslot = lds0;  // the slab being read
  // the slab whose fragment rows are being worked out (ahead of the reads), its first
  // position's column and the positions from there to the end of the range
  uint32_t aslot = lds0;
  int aw0 = klo % a.W, acnt = kend - klo;
  uint32_t ax[2][2];  // activation fragments: set, half of the lane's k
  const float Rf = (float)R + 0.5f, Q16 = 16.0f * invw;
  const uint32_t xlane = (uint32_t)(DSLOT + 8 * (lane & 3) + 64 * wc);
  auto set_rows = [&](auto settag, int k) {
    constexpr int set = decltype(settag)::value;
    const float x = Rf + (float)aw0;  // exact
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = R + 32 * k + 16 * h;
      int u = j + 2 * (int)__builtin_fmaf(x, invw, (float)(2 * k + h) * Q16);  // (x + 16 (2k + h)) / W
      if (acnt < 64 && j >= acnt) u = CW_XROWS;  // past the range: a zero row
      ax[set][h] = (uint32_t)__umul24((uint32_t)u, CW_XPITCH) + (aslot + xlane);
      asm volatile("" : "+v"(ax[set][h]));  // worked out here, not where it is first used
    }
  };
  auto next_rows = [&]() {
    aslot = up(aslot);
    aw0 += a.dw;
    if (aw0 >= a.W) aw0 -= a.W;
    acnt -= 64;
  };
  auto read_d = [&](int k, int i) {
    const uint32_t p = rslot + fd[i] + (uint32_t)(4096 * k);
    dv[i] = tr8(p, p + 2048);
  };
  auto read_x = [&](auto settag, int b) {
    constexpr int set = decltype(settag)::value;
    const uint32_t d = (uint32_t)(CW_XPITCH * (b >> 1) + 32 * (b & 1));
    xv[b] = tr8(ax[set][0] + d, ax[set][1] + d);
  };
  // One step: the MFMAs of the fragments at hand, and between them the reads of the next step
  // (k of the slab at rslot, rows in set `nxt`) and the rows of the step after that (kn of
  // the slab at aslot, into the other set).
  auto step = [&](auto nxttag, int k, int kn) {
    constexpr int nxt = decltype(nxttag)::value;
#pragma unroll
    for (int b = 0; b < 6; ++b) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[b][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[b], dv[i], acc[b][i], 0, 0, 0);
        if (b == 5) {
          __builtin_amdgcn_sched_barrier(0);
          read_d(k, i);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      read_x(CvInt<nxt>{}, b);
      if (b == 1) set_rows(CvInt<nxt ^ 1>{}, kn);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  lds_barrier();  // B_0
  set_rows(CvInt<0>{}, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) read_d(0, i);
#pragma unroll
  for (int b = 0; b < 6; ++b) read_x(CvInt<0>{}, b);
  // (after the last slab the ring's next one, all zeros or spent, is read and not used)
  if constexpr (WK == 2) {
    auto slab_barrier = [&]() {
      if constexpr (NS == 5) asm volatile("s_barrier" : : : "memory");
      else lds_barrier();
    };
    next_rows();
    set_rows(CvInt<1>{}, 0);
    for (int S = 0;;) {
      slab_barrier();  // B_{S+1}
      rslot = up(rslot);
      next_rows();
      step(CvInt<1>{}, 0, 0);
      if (++S == nsl) break;
      slab_barrier();
      rslot = up(rslot);
      next_rows();
      step(CvInt<0>{}, 0, 0);
      if (++S == nsl) break;
    }
  } else {
    set_rows(CvInt<1>{}, 1);
    for (int S = 0; S < nsl; ++S) {
      next_rows();
      step(CvInt<1>{}, 1, 0);
      lds_barrier();  // B_{S+1}
      rslot = up(rslot);
      step(CvInt<0>{}, 0, 1);
    }
  }
  lds_barrier();  // every load landed, every read done
  if constexpr (WK == 2) {
    // the halves' sums through the ring: each gives the other the half of the blocks that the
    // other writes
    const uint32_t xs = lds0 + (uint32_t)((wo * 2 + wc) * 24 * 1024 + lane * 16);
    auto xat = [&](int b, int i) { return (__attribute__((address_space(3))) f32x4 *)(uintptr_t)(xs + (uint32_t)((b * 4 + i) * 1024)); };
    auto give = [&](auto b0tag) {
      constexpr int b0 = decltype(b0tag)::value;
#pragma unroll
      for (int b = b0; b < b0 + 3; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) *xat(b, i) = acc[b][i];
    };
    auto take = [&](auto b0tag) {
      constexpr int b0 = decltype(b0tag)::value;
#pragma unroll
      for (int b = b0; b < b0 + 3; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[b][i] += *xat(b, i);
    };
    if (kh == 0) give(CvInt<3>{});
    else give(CvInt<0>{});
    lds_barrier();
    if (kh == 0) take(CvInt<0>{});
    else take(CvInt<3>{});
  }
  // ---- out: lane (fi, kg) holds channels 4kg .. +3 of output channel fi of each block;
  // device-scope stores, read next by the reduce
  if (!live) return;
  const __amdgpu_buffer_rsrc_t ro =
      __builtin_amdgcn_make_buffer_rsrc(a.out + (int64_t)split * a.sstride, 0, (int)a.out_bytes, BUF_DW3);
  const uint32_t ob = (uint32_t)((((o0 + 64 * wo + fi) * 9 + 3 * r3) * a.Ci + c0 + 32 * wc + 4 * kg) * 4);
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    if (WK == 2 && (b / 3) != kh) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[b][i]), ro,
                                             ob + (uint32_t)((16 * i * 9 + (b >> 1)) * a.Ci * 4 + 64 * (b & 1)), 0, 16);
  }
}

// dW = the splits' partials added in split order: four floats a thread, SL slices of the
// splits per output (each summed in order, then added in slice order), so that many splits of
// a small dW are still read by enough threads at once.
template <int SL>
__global__ void __launch_bounds__(256) conv_wg_reduce(const float *__restrict__ part, int64_t sstride, int splits,
                                                      int n4, float *__restrict__ out) {
  constexpr int PER = 256 / SL;
  const int i = (int)blockIdx.x * PER + (int)threadIdx.x % PER, sl = (int)threadIdx.x / PER;
  const int s0 = sl * splits / SL, s1 = (sl + 1) * splits / SL;
  f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
  if (i < n4) {
    const float *p = part + (int64_t)i * 4;
#pragma unroll 1
    for (int s = s0; s < s1; s += 4) {  // four in flight
      f32x4 q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (s + u < s1) q[u] = *reinterpret_cast<const f32x4 *>(p + (int64_t)(s + u) * sstride);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (s + u < s1) t += q[u];
    }
  }
  if constexpr (SL > 1) {
    __shared__ f32x4 sums[SL][PER];
    sums[sl][threadIdx.x % PER] = t;
    __syncthreads();
    if (sl != 0) return;
#pragma unroll
    for (int v = 1; v < SL; ++v) t += sums[v][threadIdx.x];
  }
  if (i < n4) *reinterpret_cast<f32x4 *>(out + (int64_t)i * 4) = t;
}

}  // namespace

bool conv_nt_fits(int pass, int N, int H, int W, int Ci, int Co, const void *act, const void *w, const void *out) {
  if (opt(IMBD_OPT_CONV_NT) == 0) return false;  // the tiled GEMM template instead
  const int Cn = pass == 1 ? Co : Ci, Ck = pass == 1 ? Ci : Co;
  auto al = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) % 16) == 0; };
  // byte offsets of both operands within one buffer descriptor; image rows and columns
  // within the range of the kernel's short divisions
  const int64_t P = (int64_t)N * (H + 2) * (W + 2);
  // Tensors of 2^31 elements and more are left to the tiled template, which refuses them; at
  // 256 output channels they are taken while the activations, with the rows that the last
  // tile may touch, stay within the descriptor. So a workgroup's share is at most 2^13
  // position blocks (M * Cn < 2^31 over 256 workgroups of 128 channels; M < 2^24 at 256
  // channels), and the tile bounds' products fit 32 bits.
  if (P * (Ci > Co ? Ci : Co) >= ((int64_t)1 << 31) &&
      !(Cn == 256 && (P + 2 * (W + 2) + 130) * Ck * 2 < ((int64_t)1 << 31)))
    return false;
  return (pass == 1 || pass == 2) && N >= 1 && H >= 1 && W >= 1 && Cn >= 64 && Cn % 64 == 0 && Ck >= 64 &&
         Ck % 64 == 0 && al(act) && al(w) && al(out) && H < CV_SIDE_MAX && W < CV_SIDE_MAX && P * Ck * 2 < ((int64_t)1 << 31) &&
         (int64_t)9 * Ci * Co * 2 < ((int64_t)1 << 31);
}

bool conv_wg_fits(int N, int H, int W, int Ci, int Co, const void *x, const void *dy, const void *dw) {
  if (opt(IMBD_OPT_CONV_NT) == 0) return false;
  auto al = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) % 16) == 0; };
  // Up to three of the template's K tiles (64 positions of the padded grid) on its 64 x 64 tiles
  // (a channel count off 128), where those are all in flight at once: the template's chain is
  // the shorter (1 x 7 x 7, 64 -> 256: 7.0 us, here 10.1; three K tiles, 1 x 11 x 11: 9.0 and
  // 10.3; four, 1 x 13 x 13: 10.1 and 10.4, 512 -> 64 10.2 and 9.2. On its 128 x 128 tiles
  // 1 x 7 x 7, 128 -> 256 takes 11.6, here 10.4).
  const int64_t grid = (int64_t)(N - 1) * (H + 2) * (W + 2) + (int64_t)(H - 1) * (W + 2) + W;
  if (grid <= 3 * 64 && (Ci % 128 != 0 || Co % 128 != 0) && (int64_t)9 * (Ci / 64) * (Co / 64) <= 512) return false;
  // byte offsets within one buffer descriptor; short divisions
  return N >= 1 && H >= 1 && W >= 1 && Co >= 64 && Co % 64 == 0 && Ci >= 64 && Ci % 64 == 0 && al(x) && al(dy) &&
         al(dw) && H < CV_SIDE_MAX && W < CV_SIDE_MAX &&
         (int64_t)N * (H + 2) * (W + 2) * (Ci > Co ? Ci : Co) * 2 < ((int64_t)1 << 31) &&
         (int64_t)9 * Ci * Co * 4 < ((int64_t)1 << 31);
}

namespace {
// floats from one split's partials to the next (off powers of two)
int64_t cw_split_stride(int Ci, int Co) { return (int64_t)Co * 9 * Ci + 1088; }
struct CwPlan {
  int wo, tco, tiles, splits, k_split;
};
// The output channels per workgroup and the K splits with the least modelled time: a slab
// takes about 0.55 us with 128 output channels and 0.95 with 256 (measured at 32 x 56 x 56,
// 256 -> 256: 105 us on 10 splits with the former, 108 on 21 with the latter; 1.0 us of a
// narrow image: 1.2 one column wide, 0.85 three), and the partials of every split are written
// and read once at about 4.5 TB/s together with the reduce's launch (4 us). Only as many splits
// as ws_bytes holds partials of.
CwPlan cw_best(int64_t M, int W, int Ci, int Co, size_t ws_bytes, double *time) {
  CwPlan best{};
  double &least = *time;
  least = 0;
  for (int wo : {2, 4}) {
    if (wo == 4 && (Co % 256 != 0 || cw_narrow(W))) continue;
    const int tco = (Co + 64 * wo - 1) / (64 * wo), tiles = tco * 3 * (Ci / 64);
    const int64_t slabs = (M + 63) / 64;
    const int most = (int)std::min<int64_t>(std::max(1, CV_CUS / tiles), (slabs + 3) / 4);
    for (int s = 1; s <= most; ++s) {
      if (s > 1 && (size_t)s * (size_t)cw_split_stride(Ci, Co) * sizeof(float) > ws_bytes) break;
      const int64_t per = (slabs + s - 1) / s;
      const double rounds = (double)((tiles * s + CV_CUS - 1) / CV_CUS);
      double t = rounds * (double)per * (cw_narrow(W) ? 1.0 : wo == 2 ? 0.55 : 0.95);
      if (s > 1) t += 4.0 + 2.0 * s * Co * 9 * Ci * 4 / 4.5e6;
      if (best.splits == 0 || t < least) {
        least = t;
        best = CwPlan{wo, tco, tiles, (int)((slabs + per - 1) / per), (int)(per * 64)};
      }
    }
  }
  return best;
}
// A plan within `prefer` bytes (what the tiled template's splits take) unless a larger
// workspace is more than a tenth faster.
CwPlan cw_plan(int64_t M, int W, int Ci, int Co, size_t ws_bytes, size_t prefer) {
  double t, tp;
  const CwPlan any = cw_best(M, W, Ci, Co, ws_bytes, &t);
  const CwPlan small = cw_best(M, W, Ci, Co, std::min(ws_bytes, prefer), &tp);
  return tp <= 1.1 * t ? small : any;
}
}  // namespace

size_t conv_wg_ws_bytes(int N, int H, int W, int Ci, int Co, size_t prefer) {
  const CwPlan pl = cw_plan((int64_t)N * H * W, W, Ci, Co, SIZE_MAX, prefer);
  return pl.splits > 1 ? (size_t)pl.splits * (size_t)cw_split_stride(Ci, Co) * sizeof(float) : 0;
}

int run_conv_wg(int N, int H, int W, int Ci, int Co, const void *x, const void *dy_pad, float *dw, void *ws,
                size_t ws_bytes, size_t prefer, hipStream_t s) {
  const CwPlan pl = cw_plan((int64_t)N * H * W, W, Ci, Co, ws ? ws_bytes : 0, prefer);
  CwArgs a;
  a.x = reinterpret_cast<const uint16_t *>(x);
  a.dy = reinterpret_cast<const uint16_t *>(dy_pad);
  a.out = pl.splits > 1 ? reinterpret_cast<float *>(ws) : dw;
  a.sstride = pl.splits > 1 ? cw_split_stride(Ci, Co) : 0;
  a.x_bytes = (uint32_t)((int64_t)N * (H + 2) * (W + 2) * Ci * 2);
  a.dy_bytes = (uint32_t)((int64_t)N * (H + 2) * (W + 2) * Co * 2);
  a.out_bytes = (uint32_t)((int64_t)Co * 9 * Ci * 4);
  a.H = H;
  a.W = W;
  a.Ci = Ci;
  a.Co = Co;
  a.M = N * H * W;
  a.k_split = pl.k_split;
  a.splits = pl.splits;
  a.tiles = pl.tiles;
  a.tco = pl.tco;
  a.xblk = (cw_slab_rows(W) * 10 + 63) / 64;
  a.dh = 64 / W;
  a.dw = 64 % W;
  const int grid = (a.tiles * a.splits + 7) / 8 * 8;
  {
    LaunchTimer t(IMBD_K_CONV_WGRAD, 0, s);
    if (cw_narrow(W)) hipLaunchKernelGGL((conv_wg_kernel<2, 2, true>), dim3(grid), dim3(768), 0, s, a);
    else if (pl.wo == 2) hipLaunchKernelGGL((conv_wg_kernel<2, 2, false>), dim3(grid), dim3(768), 0, s, a);
    else hipLaunchKernelGGL((conv_wg_kernel<4, 1, false>), dim3(grid), dim3(768), 0, s, a);
  }
  const int rc = check_launch("conv_wg");
  if (rc != IMBD_OK || pl.splits == 1) return rc;
  {
    LaunchTimer t(IMBD_K_SPLITK, 0, s);
    const int n4 = Co * 9 * Ci / 4;
    if (pl.splits <= 8)
      hipLaunchKernelGGL(conv_wg_reduce<1>, dim3((n4 + 255) / 256), dim3(256), 0, s, a.out, a.sstride, pl.splits, n4, dw);
    else
      hipLaunchKernelGGL(conv_wg_reduce<4>, dim3((n4 + 63) / 64), dim3(256), 0, s, a.out, a.sstride, pl.splits, n4, dw);
  }
  return check_launch("conv_wg_reduce");
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
  const int most = o == 2 ? 8 : o == 3 ? 7 : tall ? 16 : 8;
  auto tile_max = [&](int cap) {
    int t = most;
    while (t > 1 && 16 * t + 2 * ((W + 16 * t - 2) / W) + 2 > cap) --t;
    return t;
  };
  a.tmax = tile_max(cv_slab_rows(tall ? 4 : 2));
  // the larger slabs where a share then takes fewer tiles: each tile of 128 channels streams all
  // of its weights anew (32 x 224 x 4, 256 -> 256, shares of 14 blocks, forward / input gradient:
  // 41.5 / 44.3 us in two tiles, 35.6 / 39.2 in one)
  const int tn = tile_max(cv_slab_rows(4, true));
  const bool few_columns = tall && !narrow && (share + tn - 1) / tn < (share + a.tmax - 1) / a.tmax;
  if (few_columns) a.tmax = tn;
  const int grid = (a.groups * a.nct + 7) / 8 * 8;
  {
    LaunchTimer t(pass == 1 ? IMBD_K_CONV_FWD : IMBD_K_CONV_DGRAD, 0, s);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(768), 0, s, a); };
    if (narrow) pass == 1 ? go(conv_nt_kernel<false, 4, 2>) : go(conv_nt_kernel<true, 4, 2>);
    else if (few_columns) pass == 1 ? go(conv_nt_kernel<false, 4, 1, true>) : go(conv_nt_kernel<true, 4, 1, true>);
    else if (tall) pass == 1 ? go(conv_nt_kernel<false, 4, 1>) : go(conv_nt_kernel<true, 4, 1>);
    else pass == 1 ? go(conv_nt_kernel<false, 2, 2>) : go(conv_nt_kernel<true, 2, 2>);
  }
  return check_launch("conv_nt");
}

}  // namespace imbd
