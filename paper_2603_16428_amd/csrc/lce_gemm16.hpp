// The contractions on the 16x16 MFMAs, in tiles of several sizes (gemm_xs_kernel).
//
// The same three contractions, operand layouts and epilogues as gemm_xb_kernel (lce_gemm.hpp), with
// two differences that its fixed 256 x 256 tile of 32x32 MFMAs by one wave per SIMD cannot have:
//   * v_mfma_f32_16x16x32 does the same flops as v_mfma_f32_32x32x16 at less power, and these
//     kernels run against the chip's power limit.
//   * A wave's sub-tile is at most 128 x 64 (128 accumulator registers), so two waves fit a SIMD:
//     from two workgroups of 128 x 256, whose epilogues, pipeline fills and waits then pass under each
//     other's MFMAs, or from one of 256 x 256 with eight waves.
//
// A 16x16x32 fragment is 16 rows (columns) by 64 bytes of K, lane l holding row l%16, bytes
// [16 (l/16), +16); a K-quad below is those 64 bytes, two K-pairs. fp32 takes the same fragments in
// four 16x16x4 steps, step s using element s of every lane's four (K = 4 (l/16) + s).
//
// B's blocked layout is that of lce_gemm.hpp, 1 KB fragments of 32 columns by 32 bytes: lane l of a
// 16-column fragment finds chunk l/16 of column l%16 in the K-quad's K-pair l/32, half (l/16)%2:
// four runs of 256 bytes per load, every one whole cache lines.
#pragma once
#include <utility>

#include "lce_gemm.hpp"

namespace lce {

// A workgroup's tile: BM x BN of C by WM x WN waves, each with kI x kJ blocks of 16 x 16.
template <int BM, int BN, int WM, int WN>
struct Tile {
  static constexpr int kBM = BM, kBN = BN, kWM = WM, kWN = WN;
  static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves;
  static constexpr int kI = BM / WM / 16, kJ = BN / WN / 16;
  static constexpr int kSlice = BM / WM;          // vocabulary rows per log-sum-exp partial
  static constexpr int kSlot = BM * kTileBytes;   // A's K-tile in LDS
  static constexpr int kNL = BM / (8 * kWaves);   // LDS-DMA loads per wave and K-tile of A
  static constexpr int kSmem = kXbASlots * kSlot + 1024;  // the A ring, then the tile's references
  static_assert(kI % 2 == 0 && kJ % 2 == 0 && 4 * BN <= 1024);
};
using Tile256 = Tile<256, 256, 2, 4>;
using Tile128 = Tile<128, 256, 1, 4>;
using Tile64 = Tile<64, 64, 2, 2>;
using Tile128x64 = Tile<128, 64, 1, 2>;

template <typename F, int... I>
__device__ __forceinline__ void for_each_index(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

template <typename T>
__device__ __forceinline__ void mfma_quad(f32x4& c, const f32x4& a, const f32x4& b);
template <>
__device__ __forceinline__ void mfma_quad<bf16>(f32x4& c, const f32x4& a, const f32x4& b) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mfma_quad<f16>(f32x4& c, const f32x4& a, const f32x4& b) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mfma_quad<float>(f32x4& c, const f32x4& a, const f32x4& b) {
#pragma unroll
  for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], c, 0, 0, 0);
}

// A segment of 32 consecutive 16-bit elements held by the four lanes l%16 + 16 g: lane group g has
// elements 4g .. 4g + 3 of its first half in x and of its second half in y. v_permlane32_swap and
// v_permlane16_swap regroup them so that group g ends with elements 8g .. 8g + 7: whole 16-byte
// pieces, 64 contiguous bytes of a row per store instruction.
template <typename T>
__device__ __forceinline__ u32x4 regroup16(const f32x4& x, const f32x4& y) {
  typedef T t4 __attribute__((ext_vector_type(4)));
  const u32x2 a = __builtin_bit_cast(u32x2, (t4){(T)x[0], (T)x[1], (T)x[2], (T)x[3]});
  const u32x2 b = __builtin_bit_cast(u32x2, (t4){(T)y[0], (T)y[1], (T)y[2], (T)y[3]});
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    // After the first swap: a = (a0, a1, b0, b1), b = (a2, a3, b2, b3) by groups; after the second
    // a = (a0, a2, b0, b2), b = (a1, a3, b1, b3).
    const auto r = __builtin_amdgcn_permlane32_swap(a[e], b[e], false, false);
    const auto q = __builtin_amdgcn_permlane16_swap(r[0], r[1], false, false);
    o[e] = q[0];
    o[2 + e] = q[1];
  }
  return o;
}
// Its inverse (both swaps are their own): the 8 elements of group g back to x and y.
template <typename T>
__device__ __forceinline__ void ungroup16(const u32x4& o, f32x4& x, f32x4& y) {
  typedef T t4 __attribute__((ext_vector_type(4)));
  u32x2 a, b;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const auto q = __builtin_amdgcn_permlane16_swap(o[e], o[2 + e], false, false);
    const auto r = __builtin_amdgcn_permlane32_swap(q[0], q[1], false, false);
    a[e] = r[0];
    b[e] = r[1];
  }
  const t4 u = __builtin_bit_cast(t4, a), v = __builtin_bit_cast(t4, b);
  x = (f32x4){(float)u[0], (float)u[1], (float)u[2], (float)u[3]};
  y = (f32x4){(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}

// The LDS object at byte address `a`.
template <typename V>
__device__ __forceinline__ __attribute__((address_space(3))) const V* lds_at(uint32_t a) {
  return (__attribute__((address_space(3))) const V*)(uintptr_t)a;
}

// MN-contig 16-bit tiles of BM rows: logical 16-byte slot s (0 .. BM/8 - 1) of K-row k sits in slot
// s ^ swz_mn16(k). A transposing read's 32-lane half takes two slots of each of eight K-rows, k%16 in
// {0 .. 3, 8 .. 11}: their slots fall into distinct banks (BM = 64: K-rows of 128 bytes, so the row's
// parity is one bank bit already).
template <int BM>
__device__ __forceinline__ int swz_mn16(int k) {
  if constexpr (BM == 64) return ((k & 2) ? 2 : 0) ^ ((k & 8) ? 4 : 0);
  else return ((k & 1) ? 2 : 0) ^ ((k & 2) ? 4 : 0) ^ ((k & 8) ? 8 : 0);
}

// Loads and fragment reads of operand A in layout AL; see Operand in lce_gemm.hpp for the layouts.
// Every load offset is a per-lane part (lane_offset) plus a uniform one, every fragment read a
// per-lane LDS address in the current pair of ring slots (xa) plus an immediate.
template <typename T, int AL, typename C>
struct Operand16 {
  static constexpr int kEsz = (int)sizeof(T);
  static constexpr int kBK = kTileBytes / kEsz;
  static constexpr int kBM = C::kBM, kW = C::kWaves, kNL = C::kNL;
  static constexpr bool MN = AL != A_K, BLK = AL == A_BLK;
  static constexpr int kPitch = kBM * kEsz;           // MN-contig: bytes per K-row in LDS
  static constexpr int kRowLanes = kPitch / 16;       // lanes (16-byte slots) per K-row
  static constexpr int kRowsLoad = 1024 / kPitch;     // K-rows per load

  const char* base;
  int64_t ld;
  int kb, ke;
  uint32_t skip;  // MN-contig: bytes of a K-row before the tile's first column
  uint32_t row_off, slot_x, row_step;
  __amdgpu_buffer_rsrc_t rsrc_k;

  // Addresses: K-contig one per XOR of the chunk (0, 2, 4, 6); 16-bit MN-contig one per block; 16-bit
  // blocked one per read of a fragment; fp32 MN-contig and blocked one.
  static constexpr int kXa = !MN ? 4 : kEsz == 4 ? 1 : BLK ? 2 : C::kI;
  uint32_t xa[kXa];

  __device__ __forceinline__ void init(const void* p, int64_t ld_, int mn0, int rows, int kb_, int ke_, int w,
                                       int lane, int wsub, uint32_t ring) {
    ld = ld_;
    kb = kb_;
    ke = ke_;
    skip = (uint32_t)mn0 * kEsz;
    const int g = lane >> 4, r16 = lane & 15;
    if constexpr (!MN) {
      base = (const char*)p + (size_t)mn0 * ld * kEsz;
      rsrc_k = make_rsrc((const void*)uniform64((uint64_t)base),
                         __builtin_amdgcn_readfirstlane((uint32_t)rows * (uint32_t)ld * kEsz));
      // n = kNL loads per wave. Load j of wave w covers LDS bytes [(n w + j) KB, +1 KB): lane l holds
      // row r = 8 n w + 8 j + l/8, slot l%8, which is logical chunk (l%8) ^ swz_k(r) of the row, and
      // swz_k(r) = (l/8) ^ (n w % 8) ^ j (j < n, n a power of two).
      row_off = (uint32_t)(8 * kNL * w + (lane >> 3)) * (uint32_t)ld * kEsz;
      row_step = 8u * (uint32_t)ld * kEsz;
      slot_x = (uint32_t)(((lane & 7) ^ (lane >> 3) ^ ((kNL * w) & 7)) << 4);
      // Fragment of block i, K-quad u of the K-tile: row wsub + 16 i + l%16, logical chunk 4u + l/16,
      // slot (l/16) ^ swz_k(wsub + l%16) ^ (4u ^ 2i%8): one of four addresses, 2 KB per block.
#pragma unroll
      for (int m = 0; m < 4; ++m)
        xa[m] = ring + (uint32_t)((wsub + r16) * kTileBytes + ((g ^ swz_k(wsub + r16) ^ (2 * m)) << 4));
    } else if constexpr (kEsz == 2 && BLK) {
      base = (const char*)p + (size_t)mn0 * 32 * kEsz;
      // The LDS K-tile holds the fragments (32 tokens by 16 ids, 1 KB) of the K-tile's two token blocks
      // b by the tile's BM/16 id fragments c in slot (BM/16) b + c, n = kNL per wave. Piece P of a
      // fragment (token P%32, id half P/32) sits at 16 (P ^ 4 (P/32)).
      row_off = (uint32_t)(w / (kW / 2)) * (uint32_t)ld * 1024u + (uint32_t)(w % (kW / 2)) * (uint32_t)(kNL * 1024);
      row_step = 1024u;
      slot_x = (uint32_t)((lane ^ (4 * (lane >> 5))) << 4);
      // Transposed reads of block i, K-quad u (token block u): group g, lane i' = l%16 reads token
      // 8g + 4s + i'/4, ids 16 i + 4 (i'%4) .. + 3: piece half h = (i'%4)/2 at 16 (8g + i'/4 + 4 (s ^ h)
      // + 32 h), byte 8 (i'%2). s flips bit 6.
      const int h = (r16 & 3) >> 1;
      xa[0] = ring + (uint32_t)((wsub / 16) * 1024 + 16 * (8 * g + (r16 >> 2) + 4 * h + 32 * h) + 8 * (r16 & 1));
      xa[1] = xa[0] ^ 64u;
    } else if constexpr (kEsz == 2) {
      base = (const char*)p + (size_t)mn0 * kEsz;
      // A load covers R = kRowsLoad K-rows of S = kRowLanes slots (2 x 32, 4 x 16, 8 x 8): lane l of load
      // j of wave w holds K-row kr = (64 / kW) w + R j + l/S, slot l%S, logical slot (l%S) ^ swz_mn16(kr).
      row_off = (uint32_t)(64 / kW * w + lane / kRowLanes) * (uint32_t)ld * 2;
      row_step = (uint32_t)kRowsLoad * (uint32_t)ld * 2;
      slot_x = (uint32_t)(((lane % kRowLanes) ^ swz_mn16<kBM>((64 / kW * w) | (lane / kRowLanes))) << 4);
      // Transposed reads of block i, K-quad u: group g, lane i' reads K-row 32u + 8g + 4s + i'/4 at columns
      // wsub + 16 i + 4 (i'%4) .. + 3. Neither u nor s changes the swizzle, and 2i flips slot bits that
      // wsub leaves clear.
      const int r0 = 8 * g + (r16 >> 2);
#pragma unroll
      for (int i = 0; i < C::kI; ++i)
        xa[i] = ring + (uint32_t)(r0 * kPitch + (((wsub / 8 + 2 * i + ((r16 & 3) >> 1)) ^ swz_mn16<kBM>(r0)) << 4) +
                                  8 * (r16 & 1));
    } else {
      base = (const char*)p + (size_t)mn0 * (BLK ? 32 : 1) * kEsz;
      // fp32: a load covers kRowsLoad K-rows of kRowLanes slots; blocked, K-row k is token k of the
      // K-tile's one token block, slot s at 512 s.
      const uint32_t kr = (uint32_t)(32 / kW * w + lane / kRowLanes);
      row_off = BLK ? kr * 16u : kr * (uint32_t)ld * 4;
      row_step = BLK ? (uint32_t)kRowsLoad * 16u : (uint32_t)kRowsLoad * (uint32_t)ld * 4;
      slot_x = (uint32_t)(lane % kRowLanes) << (BLK ? 9 : 4);
      xa[0] = ring + (uint32_t)(4 * g * kPitch + (wsub + r16) * 4);
    }
  }

  // The compile-time XOR part of load j's offset: what j adds to the swizzle.
  static __device__ __forceinline__ constexpr uint32_t xor_j(int j) {
    if constexpr (!MN) return (uint32_t)(j << 4);
    // 256 rows: kr = 8 w + 2 j + l/32; the wave gives bit 3, the lane bit 0.
    else if constexpr (kEsz == 2 && !BLK && kBM == 256) return (uint32_t)(((j & 1) ? 4 : 0) << 4);
    // 64 rows: kr = 16 w + 8 j + l/8.
    else if constexpr (kEsz == 2 && !BLK && kBM == 64) return (uint32_t)((j ? 4 : 0) << 4);
    // 128 rows: kr = 16 w + 4 j + l/16.
    else if constexpr (kEsz == 2 && !BLK) return (uint32_t)(((j & 2) ? 8 : 0) << 4);
    else return 0u;
  }
  __device__ __forceinline__ uint32_t lane_offset(int j) const { return (slot_x ^ xor_j(j)) + row_off; }
  // K-contig: the K-tile's start, kOOB at or past ke; whole K-tiles (see Operand::uniform_offset).
  __device__ __forceinline__ uint32_t uniform_offset(int t, int j) const {
    uint32_t o = (uint32_t)j * row_step;
    if constexpr (!MN) {
      const int k0 = kb + t * kBK;
      o = k0 < ke ? o + (uint32_t)k0 * kEsz : kOOB;
    }
    return __builtin_amdgcn_readfirstlane(o);
  }
  // K-contig with a check of every 16-byte chunk against ke.
  __device__ __forceinline__ uint32_t offset(int t, int j) const {
    const int k0 = kb + t * kBK;
    const int kc = (int)(((slot_x ^ xor_j(j)) >> 4) * (16 / kEsz));
    return k0 + kc < ke ? lane_offset(j) + (uint32_t)j * row_step + (uint32_t)k0 * kEsz : kOOB;
  }

  // Descriptor for K-tile t: its valid K-rows (MN-contig; the range ends with the last K-row's own
  // columns, what follows is other memory) or token blocks (blocked) only.
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int t) const {
    if constexpr (!MN) {
      return rsrc_k;
    } else {
      const int k0 = kb + t * kBK;
      uint32_t bytes;
      size_t start;
      if constexpr (BLK) {
        const uint32_t blk = (uint32_t)ld * 1024u;
        const int nblk = min(kBK / 32, (max(ke - k0, 0) + 31) >> 5);
        bytes = (uint32_t)nblk * blk - (uint32_t)min(nblk, 1) * (blk - (uint32_t)(kBM * kEsz * 32));
        start = (size_t)(k0 >> 5) * blk;
      } else {
        const int nrows = max(0, min(kBK, ke - k0));
        bytes = (uint32_t)nrows * (uint32_t)ld * kEsz - (uint32_t)min(nrows, 1) * skip;
        start = (size_t)(k0 < ke ? k0 : kb) * ld * kEsz;
      }
      return make_rsrc((const void*)uniform64((uint64_t)(base + start)), __builtin_amdgcn_readfirstlane(bytes));
    }
  }

  // Fragment of block I, K-quad U of slot SIP (0, 1) of the pair of ring slots that `a` points at.
  // 16-bit MN-contig and blocked reads are inline assembly (the compiler would wait for every
  // outstanding LDS-DMA load before the builtin): the caller waits for them (sync_frags).
  template <int SIP, int U, int I>
  static __device__ __forceinline__ f32x4 fragment(const uint32_t (&a)[kXa]) {
    constexpr int st = SIP * C::kSlot;
    if constexpr (!MN) {
      return *lds_at<f32x4>(a[((4 * U) ^ (2 * I % 8)) / 2] + (uint32_t)(st + 2048 * I));
    } else if constexpr (kEsz == 4) {
      f32x4 v;
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = *lds_at<float>(a[0] + (uint32_t)(st + (16 * U + s) * kPitch + 64 * I));
      return v;
    } else {
      i16x4 v[2];
      if constexpr (BLK) {
        asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%4\n\tds_read_b64_tr_b16 %1, %3 offset:%4"
                     : "=&v"(v[0]), "=&v"(v[1])
                     : "v"(a[0]), "v"(a[1]), "i"(st + 64 * kBM * U + 1024 * I));
      } else {
        asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                     : "=&v"(v[0]), "=&v"(v[1])
                     : "v"(a[I]), "i"(st + 32 * U * kPitch), "i"(st + (32 * U + 4) * kPitch));
      }
      return __builtin_bit_cast(f32x4, v);
    }
  }
};

// The epilogue: what a wave's sub-tile of NI x NJ 16 x 16 blocks at (mw, nw) becomes. Without the
// operand swap (LSE, STORE) element r of block (i, j) is row 16 i + 4 (l/16) + r, column 16 j + l%16 of
// the sub-tile; with it (DW) row 16 i + l%16, column 16 j + 4 (l/16) + r.
template <typename T, int EPI, bool PRELOADED, int NI, int NJ>
__device__ __forceinline__ void gemm_epilogue16(const GemmArgs& g, f32x4 (&acc)[NI][NJ], int mw, int nw, int split,
                                                int n0, const char* refs_lds, bool later_run) {
  constexpr int kEsz = (int)sizeof(T);
  const int lane = lane_id();
  const int l16 = lane & 15, grp = lane >> 4;
  if constexpr (EPI == EPI_LSE_FWD || EPI == EPI_LSE_BWD) {
    if (mw >= g.M) return;
    const int slice = mw / (16 * NI);
    const bool tref = EPI == EPI_LSE_BWD && g.ref != nullptr;
    auto body = [&](auto full_c) {
      constexpr bool FULL = decltype(full_c)::value;
      auto inside = [&](int i, int r) { return FULL || mw + 16 * i + 4 * grp + r < g.M; };
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int col = nw + 16 * j + l16;
        const bool in = col < g.N;
        float m_ref, ml, s = 0.f;
        if (tref) {  // as in gemm_epilogue: +inf for a token without a reference, so that its e is 0
          const float ref = *(const float*)(refs_lds + 4 * (col - n0));
          const bool keep = in && __builtin_isfinite(ref);
          m_ref = keep ? ref : 0.f;
          ml = keep ? ref * kLog2e : INFINITY;
        } else {
          float mx = -INFINITY;
#pragma unroll
          for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (inside(i, r)) mx = fmaxf(mx, acc[i][j][r]);
          mx = fmaxf(mx, __shfl_xor(mx, 16));
          mx = fmaxf(mx, __shfl_xor(mx, 32));
          m_ref = mx;
          ml = mx == -INFINITY ? 0.f : mx * kLog2e;  // a partial of -inf logits alone sums to 0
        }
        // Every token block that holds a token of the chunk is written whole. This lane's chunk of a
        // K-quad is in K-pair l/32, half (l/16)%2 of column l%16 (+ 16 for odd j).
        const bool store = EPI == EPI_LSE_BWD && ((nw + 16 * j) & ~31) < g.N;
        char* e_blk = (char*)g.out + (size_t)((nw + 16 * j) >> 5) * g.ldo * 1024 + (lane >> 5) * 1024 +
                      ((grp & 1) * 32 + l16 + 16 * (j & 1)) * 16;
#pragma unroll
        for (int i = 0; i < NI; i += 2) {
          f32x4 ev[2];
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float e = inside(i + h, r) ? __builtin_amdgcn_exp2f(fmaf(acc[i + h][j][r], kLog2e, -ml)) : 0.f;
              s += e;
              ev[h][r] = e * Storage<T>::kE;
            }
          if constexpr (EPI == EPI_LSE_BWD) {
            if (store) {
              if constexpr (kEsz == 2) {
                // Whole wave slices: the blocked rows cover M rounded up to 256, and rows at or beyond
                // M hold exp = 0 here.
                *(u32x4*)(e_blk + (size_t)((mw + 16 * i) >> 4) * 1024) = regroup16<T>(ev[0], ev[1]);
              } else {
                // fp32: 16 ids are a K-quad, this lane's four its chunk. Every K-quad that holds an id
                // below M is stored whole.
#pragma unroll
                for (int h = 0; h < 2; ++h)
                  if (FULL || mw + 16 * (i + h) < g.M)
                    *(f32x4*)(e_blk + (size_t)((mw + 16 * (i + h)) >> 3) * 1024) = ev[h];
              }
            }
          }
        }
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (in && lane < 16) {
          g.pmax[(size_t)slice * g.ldp + col] = m_ref;
          g.psum[(size_t)slice * g.ldp + col] = s;
        }
      }
    };
    if (mw + 16 * NI <= g.M) body(std::true_type{});
    else body(std::false_type{});
  } else if constexpr (EPI == EPI_STORE) {
    // C^T token-major: column n of C is row n of the output. M (the output's row length) is a multiple
    // of 8 for 16-bit types and of 4 for fp32. mode 1: fp32 partials, split s at out + s * N * ldo.
    const float sc = dz_epilogue_scale<T>(g.n_valid, g.mean);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int col = nw + 16 * j + l16;
      if (col >= g.N) continue;
      if (g.col_scale) {
        const float cs = g.col_scale[col];
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[i][j] *= cs;
      }
      if (g.mode == 1 || kEsz == 4) {
        float* o = (float*)g.out + ((size_t)(g.mode == 1 ? split : 0) * g.N + col) * g.ldo;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int row = mw + 16 * i + 4 * grp;
          if (row < g.M) *(f32x4*)(o + row) = acc[i][j];
        }
      } else if constexpr (kEsz == 2) {
        T* o = (T*)g.out + (size_t)col * g.ldo;
#pragma unroll
        for (int i = 0; i < NI; i += 2) {
          const int row = mw + 16 * i + 8 * grp;
          const u32x4 v = Storage<T>::kDzUnscaled ? regroup16<T>(acc[i][j] * sc, acc[i + 1][j] * sc)
                                                  : regroup16<T>(acc[i][j], acc[i + 1][j]);
          if (row < g.M) *(u32x4*)(o + row) = v;
        }
      }
    }
  } else {
    // DW. N (the output pitch) is a multiple of 8 (16-bit) or 4.
    const float sc = dz_epilogue_scale<T>(g.n_valid, g.mean);
    const bool acc32 = g.mode >= DW_ACC32_FIRST;
    // fp32 values land directly: acc32 (+)= sc C, at the last chunk dW = acc32 + sc C; fp32 dW itself
    // (no preload) likewise in one buffer, also from one run of the tokens to the next.
    const bool read = acc32 ? g.mode != DW_ACC32_FIRST : g.mode == DW_ACCUMULATE || later_run;
    const bool last = g.mode == DW_ACC32_LAST;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int row = mw + 16 * i + l16;
      if (row >= g.M) continue;
      T* o = (T*)g.out + (size_t)row * g.ldo;
      if (kEsz == 4 || acc32) {
        float* a = kEsz == 4 ? (float*)o : g.acc32 + (size_t)row * g.ldo;
        f32x4 base[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int col = nw + 16 * j + 4 * grp;
          base[j] = (read && col < g.N) ? *(const f32x4*)(a + col) : (f32x4){};
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int col = nw + 16 * j + 4 * grp;
          if (col >= g.N) continue;
          const f32x4 v = base[j] + sc * acc[i][j];
          if (last) store4(o + col, v[0], v[1], v[2], v[3]);
          else *(f32x4*)(a + col) = v;
        }
      } else if constexpr (kEsz == 2) {  // PRELOADED: the accumulators hold the earlier chunks' sum
#pragma unroll
        for (int j = 0; j < NJ; j += 2) {
          const int col = nw + 16 * j + 8 * grp;
          const u32x4 v = Storage<T>::kDzUnscaled ? regroup16<T>(acc[i][j] * sc, acc[i][j + 1] * sc)
                                                  : regroup16<T>(acc[i][j], acc[i][j + 1]);
          if (col < g.N) *(u32x4*)(o + col) = v;
        }
      }
    }
  }
}

// The pipeline of gemm_xb_kernel: A through a ring of four K-tiles in LDS, three ahead; B straight to
// registers, four K-quads of fragments, three ahead. A K-tile is four sections, K-quad p/2 by half p%2
// of the wave's row blocks; each section's A fragments are read during the one before it, and it issues
// a quarter of A's K-tile three ahead and half of B's fragments three K-quads ahead.
// fp32 dW is summed in runs of k_per_split tokens (an even number of K-tiles), one after the other: an
// entry's rounding error grows with the length of its running sum (2048 tokens, H = 2048: 7.7e-7 in one run,
// 5.5e-7 in two of half of them). 64 x 64 tiles have the registers for the sum of the earlier runs beside
// the accumulators (256 x 256 x 4096: a second pass over the pipeline cost 3 us of 43, this nothing); the
// others' kernel takes one run after the other through here, each added to dW.
template <typename T, int EPI, typename C>
constexpr bool kRunsInRegisters = EPI == EPI_DW && sizeof(T) == 4 && C::kBM == 64;
template <typename T, int EPI, typename C>
constexpr bool kRunsThroughDw = EPI == EPI_DW && sizeof(T) == 4 && C::kBM != 64;

// run: which run of K (kRunsThroughDw, else 0).
template <typename T, int EPI, int AL, bool KCHECK, typename C>
__device__ __forceinline__ void gemm_xs_tile(const GemmArgs& g, int bid, int run, char* smem) {
  constexpr int kEsz = (int)sizeof(T);
  constexpr int kBK = kTileBytes / kEsz;
  constexpr bool kSwap = EPI == EPI_DW;
  constexpr bool kAsmReads = AL != A_K && kEsz == 2;
  constexpr int NI = C::kI, NJ = C::kJ, NH = NI / 2, kNL = C::kNL;

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = w / C::kWN, wn = w % C::kWN;
  const int total = g.tiles_m * g.tiles_n * g.splits;
  int tm, rest;
  tile_coords(bid, total, g.tiles_m, g.group_m, tm, rest);
  tm = __builtin_amdgcn_readfirstlane(tm);
  rest = __builtin_amdgcn_readfirstlane(rest);
  const int tn = rest % g.tiles_n;
  const int split = rest / g.tiles_n;
  const int m0 = tm * C::kBM, n0 = tn * C::kBN;
  const int mw = m0 + wm * 16 * NI, nw = n0 + wn * 16 * NJ;
  constexpr bool kRegRuns = kRunsInRegisters<T, EPI, C>;
  const int kb = kRegRuns ? 0 : (split + run) * g.k_per_split;
  const int ke = kRegRuns ? g.K : min(g.K, kb + g.k_per_split);

  using Op = Operand16<T, AL, C>;
  Op opa;
  opa.init(g.A, g.lda, m0, min(C::kBM, g.M - m0), kb, ke, w, lane, wm * 16 * NI,
           (uint32_t)(uintptr_t)(lds_void*)smem);

  // B: the wave's 32-column blocks start at jb0 (the descriptor's base; blocks at or beyond NB read
  // zeros); K-quad q of this split is K-pairs q0 + 2q, + 1 of a block.
  const int KP = (int)g.ldb;
  const int NB = (g.N + 31) >> 5;
  const int jb0 = nw >> 5;
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(
      (const void*)uniform64((uint64_t)((const char*)g.B + (size_t)jb0 * KP * 1024)),
      __builtin_amdgcn_readfirstlane((uint32_t)max(0, min(NJ / 2, NB - jb0)) * (uint32_t)KP * 1024u));
  const uint32_t bvoff = (uint32_t)((lane >> 5) * 1024 + (((lane >> 4) & 1) * 32 + (lane & 15)) * 16);
  const int q0 = kb * kEsz / 32;
  const int qend = ((ke - kb) * kEsz + 63) / 64;

  uint32_t aoff[kNL];
#pragma unroll
  for (int j = 0; j < kNL; ++j) aoff[j] = opa.lane_offset(j);
  // Quarter pc of A K-tile t (its loads pc n/4 .. (pc + 1) n/4 - 1) into ring slot t % 4.
  auto load_a_q = [&](int t, auto pc) {
    constexpr int pq = decltype(pc)::value;
    const __amdgpu_buffer_rsrc_t r = opa.rsrc(t);
    char* st = smem + (t & (kXbASlots - 1)) * C::kSlot + w * kNL * 1024;
#pragma unroll
    for (int j = pq * kNL / 4; j < (pq + 1) * kNL / 4; ++j) {
      if constexpr (KCHECK && AL == A_K) dma16(r, st + j * 1024, opa.offset(t, j));
      else dma16(r, st + j * 1024, aoff[j], opa.uniform_offset(t, j));
    }
  };
  auto load_a = [&](int t) {
    load_a_q(t, std::integral_constant<int, 0>{});
    load_a_q(t, std::integral_constant<int, 1>{});
    load_a_q(t, std::integral_constant<int, 2>{});
    load_a_q(t, std::integral_constant<int, 3>{});
  };
  f32x4 vb[4][NJ];
  // Half h of B K-quad q's fragments into ring slot `slot` (a constant: the ring stays in registers).
  auto load_b = [&](int q, auto slot, auto h) {
    constexpr int j0 = decltype(h)::value * NJ / 2;
#pragma unroll
    for (int j = j0; j < j0 + NJ / 2; ++j) {
      const uint32_t so = q < qend ? (uint32_t)((j >> 1) * KP + q0 + 2 * q) * 1024u : kOOB;
      // The odd 16 columns of a block: 256 bytes further in each run.
      vb[decltype(slot)::value][j] =
          __builtin_bit_cast(f32x4, load16(rb, bvoff + (j & 1) * 256u, __builtin_amdgcn_readfirstlane(so)));
    }
  };

  f32x4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = (f32x4){};

  f32x4 fa[2][NH];
  uint32_t pair_delta = 2 * C::kSlot;  // current pair of slots 0-1: the next is two up, then down
  // The fragments of half H, K-quad U of slot SIP of the current pair (NEXT: of the other pair).
  auto read_frags = [&](auto sip, auto uc, auto hc, auto next, int buf) {
    constexpr int SIP = decltype(sip)::value, U = decltype(uc)::value, H = decltype(hc)::value;
    uint32_t a[Op::kXa];
#pragma unroll
    for (int k = 0; k < Op::kXa; ++k) a[k] = decltype(next)::value ? opa.xa[k] + pair_delta : opa.xa[k];
    for_each_index([&](auto i) { fa[buf][i] = Op::template fragment<SIP, U, H * NH + decltype(i)::value>(a); },
                   std::make_integer_sequence<int, NH>{});
  };
  // Inline-assembly reads are invisible to the compiler's waits: at the start of each section all
  // earlier LDS traffic is waited for, with the fragments as operands so that no MFMA moves above.
  auto sync_frags = [&]() {
    if constexpr (kAsmReads) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int i = 0; i < NH; ++i) asm volatile("" : "+v"(fa[0][i]), "+v"(fa[1][i]));
    }
  };
  auto mma = [&](int buf, auto slot, auto hc) {
    constexpr int H = decltype(hc)::value;
#pragma unroll
    for (int i = 0; i < NH; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if constexpr (kSwap) mfma_quad<T>(acc[H * NH + i][j], vb[decltype(slot)::value][j], fa[buf][i]);
        else mfma_quad<T>(acc[H * NH + i][j], fa[buf][i], vb[decltype(slot)::value][j]);
      }
  };
  constexpr int kReads = kAsmReads ? 0 : NH;  // compiler-visible LDS reads per section
  // 16-bit, 128 x 64 per wave: 16 MFMAs per section, the LDS reads after the first pairs of them, the
  // loads after the second, fourth and sixth pair. Nothing moves out of its section.
  auto sched = []() {
    if constexpr (kEsz == 2 && NI == 8) {
#pragma unroll
      for (int i = 0; i < NH * NJ / 2; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        if (i < kReads) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if ((i & 1) && i < 6) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // At p == 3, A(kt' + 1) has landed in LDS for every wave before its first fragments are read: its last
  // load went out in section 4 (kt' + 1 - ahead) + 3, and the 4 ahead - 5 sections since issued NJ / 2
  // loads of B each, ahead - 2 whole K-tiles of A and the first three quarters of one more (loads retire
  // in order).
  constexpr int kAWait = NJ / 2 * (4 * kXbAhead - 5) + kNL * (kXbAhead - 2) + 3 * kNL / 4;
  static_assert(kXbAhead >= 2 && kAWait <= 63, "vmcnt range");
  auto section = [&](int kt, auto sc) {
    constexpr int s = decltype(sc)::value;
    constexpr int p = s & 3, n = (s + 1) & 7;  // n: the section whose fragments are read now
    const int ktp = kt + (s >> 2);
    using Slot = std::integral_constant<int, (s >> 1)>;
    using Half = std::integral_constant<int, (s & 1)>;
    if constexpr (p == 3) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kAWait) : "memory");
    sync_frags();
    read_frags(std::integral_constant<int, (n >> 2)>{}, std::integral_constant<int, ((n >> 1) & 1)>{},
               std::integral_constant<int, (n & 1)>{}, std::integral_constant<bool, s == 7>{}, n & 1);
    if constexpr (AL != A_K) load_a_q(ktp + kXbAhead, std::integral_constant<int, p>{});
    mma(s & 1, Slot{}, Half{});
    load_b(2 * kt + (s >> 1) + 3, std::integral_constant<int, ((s >> 1) + 3) & 3>{}, Half{});
    if constexpr (AL == A_K) load_a_q(ktp + kXbAhead, std::integral_constant<int, p>{});
    sched();
  };

  // 16-bit dW accumulation: the wave's current dW values, the 16-byte row pieces that the epilogue
  // stores, loaded while the pipeline fills, are the accumulators' starting values (divided by the
  // factor that the epilogue applies). Rows at or beyond M read zeros, columns at or beyond N whatever
  // is there (the epilogue stores neither): a branch per piece made the compiler wait for each fp16
  // piece before it requested the next.
  constexpr bool kPreload = EPI == EPI_DW && kEsz == 2;
  const bool accumulate = EPI == EPI_DW && g.mode == DW_ACCUMULATE;
  u32x4 prev[kPreload ? NI : 1][NJ / 2];
  if constexpr (kPreload) {
    if (accumulate) {
      const uint32_t pitch = (uint32_t)g.ldo * 2u;
      const __amdgpu_buffer_rsrc_t rp = make_rsrc(
          (const void*)uniform64((uint64_t)((const T*)g.out + (size_t)mw * g.ldo)),
          __builtin_amdgcn_readfirstlane((uint32_t)max(0, min(16 * NI, g.M - mw)) * pitch));
      const uint32_t voff = (uint32_t)(lane & 15) * pitch + (uint32_t)(nw + 8 * (lane >> 4)) * 2u;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; j += 2)
          prev[i][j / 2] = load16(rp, voff + 32u * j, __builtin_amdgcn_readfirstlane((uint32_t)(16 * i) * pitch));
    }
  }
  const int nk = (ke - kb + kBK - 1) / kBK;
  // Target-referenced LSE_BWD: the tile's references into LDS, before the loads that are counted; past
  // N it reads zeros.
  if (EPI == EPI_LSE_BWD && g.ref != nullptr && w == 0) {
    const __amdgpu_buffer_rsrc_t rr = make_rsrc((const void*)uniform64((uint64_t)(g.ref + n0)),
                                                __builtin_amdgcn_readfirstlane((uint32_t)max(0, g.N - n0) * 4u));
    dma16(rr, smem + kXbASlots * C::kSlot, (uint32_t)lane * 16u);
  }
  if (nk > 0) {
    // A(0 .. ahead - 1), then B(0 .. 2). A(0) has landed for every wave before its first fragments are
    // read; the first waits at p == 3 find at least as many loads after A(1), A(2) as they allow.
#pragma unroll
    for (int t = 0; t < kXbAhead; ++t) load_a(t);
    if constexpr (kPreload) {
      if (accumulate) {
        const float inv = dw_prev_scale<T>(g);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; j += 2) {
            ungroup16<T>(prev[i][j / 2], acc[i][j], acc[i][j + 1]);
            if constexpr (Storage<T>::kDzUnscaled) {
              acc[i][j] *= inv;
              acc[i][j + 1] *= inv;
            }
          }
      }
    }
    using H0 = std::integral_constant<int, 0>;
    using H1 = std::integral_constant<int, 1>;
    load_b(0, std::integral_constant<int, 0>{}, H0{});
    load_b(0, std::integral_constant<int, 0>{}, H1{});
    load_b(1, std::integral_constant<int, 1>{}, H0{});
    load_b(1, std::integral_constant<int, 1>{}, H1{});
    load_b(2, std::integral_constant<int, 2>{}, H0{});
    load_b(2, std::integral_constant<int, 2>{}, H1{});
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(kNL * (kXbAhead - 1) + 3 * NJ) : "memory");
    read_frags(H0{}, H0{}, H0{}, std::false_type{}, 0);
    if constexpr (kRegRuns) {  // as below, run by run
      f32x4 sum[NI][NJ] = {};
      for (int kt = 0; kt < nk;) {
        const int end = min(nk, kt + g.k_per_split / kBK);
        for (; kt < end; kt += 2) {
          for_each_index([&](auto s) { section(kt, s); }, std::make_integer_sequence<int, 8>{});
#pragma unroll
          for (int k = 0; k < Op::kXa; ++k) opa.xa[k] += pair_delta;
          pair_delta = 0u - pair_delta;
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            sum[i][j] += acc[i][j];
            acc[i][j] = (f32x4){};
          }
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = sum[i][j];
    } else {
      for (int kt = 0; kt < nk; kt += 2) {  // an odd count runs one more K-tile of zeros
        section(kt, std::integral_constant<int, 0>{});
        section(kt, std::integral_constant<int, 1>{});
        section(kt, std::integral_constant<int, 2>{});
        section(kt, std::integral_constant<int, 3>{});
        section(kt, std::integral_constant<int, 4>{});
        section(kt, std::integral_constant<int, 5>{});
        section(kt, std::integral_constant<int, 6>{});
        section(kt, std::integral_constant<int, 7>{});
#pragma unroll
        for (int k = 0; k < Op::kXa; ++k) opa.xa[k] += pair_delta;
        pair_delta = 0u - pair_delta;
      }
    }
    // Loads past the end may still be in flight (they target no memory), and the last section's
    // fragment reads; their LDS and registers must not be reused before they retire.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    sync_frags();
  }
  gemm_epilogue16<T, EPI, kPreload>(g, acc, mw, nw, split, n0, smem + kXbASlots * C::kSlot, run > 0);
}


template <typename T, int EPI, int AL, bool KCHECK, typename C>
__global__ __launch_bounds__(C::kThreads, C::kBM == 256 ? 1 : C::kBM == 128 ? 2 : 4) void gemm_xs_kernel(const GemmArgs g) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  if (g.run_if != nullptr && __builtin_amdgcn_readfirstlane(*g.run_if) == 0) return;
  if constexpr (kRunsThroughDw<T, EPI, C>) {
    for (int run = 0; run * g.k_per_split < g.K; ++run) {
      // Every wave is done with the ring, and the tile's stores no longer count in vmcnt.
      if (run > 0) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      gemm_xs_tile<T, EPI, AL, KCHECK, C>(g, blockIdx.x, run, smem);
    }
  } else {
    gemm_xs_tile<T, EPI, AL, KCHECK, C>(g, blockIdx.x, 0, smem);
  }
}

}  // namespace lce
