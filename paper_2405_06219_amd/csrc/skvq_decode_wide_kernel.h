// Matrix-core kernel of skvq_decode_attention for more than four rows per kv head (query heads of the
// kv head x query tokens) over long caches: up to sixteen rows per workgroup.  The cache formats, the
// fp16 operands made of codes, the grid, the workgroups' shares and the partials are those of
// skvq_decode_mfma_kernel.h.  The later deals of tiles go to the older wavefronts first here too, where that
// kernel takes turns; all fp16 slices are of four tokens and plain vector arithmetic, two teams of wavefronts
// for them; no keys go through the matrix cores as FP4 or FP8 numbers.  (None of these three has been measured
// here.)  The products have another shape:
//
//   QK   S[token][row] by v_mfma_f32_16x16x32_f16: A = sixteen key rows, B = the rows' reordered
//        queries (sixteen columns, held in registers).  Lane (m = lane % 16, h = lane / 16) feeds a
//        quarter of one key row, loaded as such; product g of a tile takes the tokens
//        32 (g / 2) + 8 (m / 4) + 4 (g % 2) + m % 4, so that afterwards the lane holds, of ONE row
//        (its column), the scores of the tokens 8 h .. 8 h + 7 of both blocks of 32: the running
//        reference and the sums are plain registers of a lane, and
//   PV   O^T[channel][row] by v_mfma_f32_16x16x32_f16: A = the V unit, B = the lane's own weights as
//        they are (high and low fp16 parts, one chain of products): no weight goes through LDS.
//
// What the lane = token kernel does per row, in as many workgroups per chunk as there are four rows
// (each unpacking all codes again), is done once here: loads, unpacking, table reads, (scale, zero).
// The (scale, zero) factors of a tile are worked out with lane = token and read back by all sixteen
// rows of a token from LDS (1.25 KB per wavefront and group).  Bound by the vector instructions of
// the softmax (eleven per score, sixteen scores per lane and tile) and the LDS reads beside them.
// A call (with its merge) against the workgroups of four rows that this replaced, 32 q / 8 kv heads, us:
//   2-bit keys, 3-level values, one group, 131072 tokens: 4 query tokens 51.4 -> 27.8, 2: 31.5 -> 25.7
//   the same in two groups with FP8 (scale, zero), 100003 tokens, 4 query tokens: 44.2 -> 29.8
//   4-bit, two groups, 60000 tokens, 4 query tokens: 37.7 -> 28.4
// At short caches, and where the compute units have room for the other workgroups, four rows a workgroup are
// faster (up to twice: plan_decode in skvq_api.hip chooses).
// All 256 registers are in use.  With one group per head the tile loop spills nothing, and four of the 21
// instances one to five registers around it; with two groups every instance spills: 3 - 10 registers with 2-bit
// keys and 2-bit or 3-level values, 9 - 20 with 4 bits on one side, 17 - 26 on both, 25 - 31 with 3 bits.  With
// four groups or unequal ones it would be slower than the workgroups of four rows at any length (measured at
// 131072 and 60000 tokens: 46 -> 88 and 52 -> 54 us a call), so it is not built for them.
#pragma once
#include "skvq_decode_mfma_kernel.h"

namespace skvq {
namespace {

constexpr int kWideSlice = 4;                    // fp16 tokens per slice
// What one wavefront loads for one slice.
struct WideRing {
  uint4_t k;      // lane (token = l/16, piece = l%16): 8 channels of the token's key row
  unsigned v[4];  // lane = channel pair: the 4 tokens' values of channels 2l, 2l+1
};
constexpr int kRowQuad = 4;                      // rows that one wavefront serves in a fp16 slice
static_assert(kWideTeams == kNW / (kWideRows / kRowQuad), "wavefronts per row quad");
constexpr int kWideStride = kD + 4;  // floats per staged output row: sixteen rows on different banks
constexpr int kTokStride = 80;       // (factor pairs of) the 64 tokens of a tile: two of padding after every
                                     // eight, so that the four lane groups read different banks
__device__ __forceinline__ int tok_slot(int t) { return t + 2 * (t >> 3); }

template <bool TERNARY, int NG>
struct WideSmem {
  union {
    uint4_t lut[TERNARY ? 6561 : 1];  // 13-bit field -> operand, as in the lane = token kernel
    float stage[kNW][kWideRows][kWideStride];  // (after the last tile) per wave: its O, [row][reordered position]
  };
  float ring_o[kNW][kRowQuad][kD];  // per wave: its slices' outputs, original channel order
  alignas(16) int perm_v[kD];
  uint2_t lut4[TERNARY ? kNW : 1][81];
  // per wave and group, of the current tile's tokens: {key scale, dequantized centre} and {value scale,
  // value zero}, with the factors that the codes' places in the operands ask for
  alignas(16) float2 ktok[kNW][NG][kTokStride], vtok[kNW][NG][kTokStride];
  // B operands of the score product: [step][lane / 16][row][k slot]
  alignas(16) _Float16 qa[4][4][kWideRows][8];
  union {
    alignas(16) _Float16 qraw[kWideRows][kD];   // the query rows as loaded (rows that do not exist are zero)
    AppendScratch append;                       // (before them)
  };
  alignas(16) float qpart[kWideRows][8];        // sums of the reordered query over 16 positions each
  alignas(16) float wm[kWideRows][kNW], wl[kWideRows][kNW], wz[kWideRows][NG][kNW];
  float rm[kWideRows][kWideTeams], rl[kWideRows][kWideTeams];
};

// unpack_k3 with the key dword's place in its pair known at run time only.
__device__ __forceinline__ void unpack_k3_of(bool odd, unsigned w, unsigned h, half4_t b[4]) {
  const unsigned wl = w << 4, wr = w >> 6;
  const unsigned ha = odd ? h >> 1 : h << 6, hb = odd ? h >> 4 : h << 5, hc = odd ? h >> 7 : h;
  b[0] = h4((wl & kM4) | (ha & kB6), (wl & kM6) | (ha & kB8));
  b[1] = h4((w & kM4) | (hb & kB6), (w & kM6) | (hb & kB8));
  b[2] = h4((w & kM8) | (ha & kB10), (wr & kM4) | (hc & kB6));
  b[3] = h4((wr & kM6) | (hc & kB8), (wr & kM8) | (hb & kB10));
}
__device__ __forceinline__ half8_t join(half4_t a, half4_t b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

// 3- and 4-bit value fields, one shift more than in unpack_v3_field and unpack_v4_field: the token pairs at
// mantissa bits {6, 8, 8, 8}, or all at bit 6.  With the codes at those functions' places, and a row's high
// and low weights in one chain of products, the outputs were 2 % further from a 64-bit evaluation than the
// four-row kernel's; so they are nearer: 2.4e-6
// of the norm against 1.05e-5 (4-bit, two groups, 20000 tokens), 1.9e-6 against 6.4e-6 (3-bit).
constexpr unsigned kN6 = 0x03c003c0u;  // a 4-bit code at mantissa bit 6 of each half
__device__ __forceinline__ half8_t unpack_wide_v4(unsigned f) {
  return __builtin_bit_cast(half8_t, uint4_t{(f << 6) & kN6, (f << 2) & kN6, (f >> 2) & kN6, (f >> 6) & kN6});
}
template <int NN>
__device__ __forceinline__ half8_t unpack_wide_v3(unsigned f, unsigned h) {
  const unsigned a = f << 6, b = f << 4, c = f << 2;
  const unsigned ha = NN == 0 ? h << 8 : NN == 1 ? h << 7 : NN == 2 ? h << 2 : h << 1;  // token pairs 0, 1
  const unsigned hb = NN == 0 ? h << 6 : NN == 1 ? h << 5 : NN == 2 ? h : h >> 1;       // token pair 2
  const unsigned hc = h >> (2 + NN);                                                    // token pair 3
  return __builtin_bit_cast(half8_t, uint4_t{(a & kM6) | (ha & kB8), (a & kM8) | (ha & kB10), (b & kM8) | (hb & kB10),
                                             (c & kM8) | (hc & kB10)});
}

// A lane's quarter of a key row: `d` holds the dwords of steps 0, 1 and of steps 2, 3 (4-bit: one dword
// a step), `top` the 3-bit plane dwords that belong to them.
template <int KL>
struct KeyPiece {
  typedef uint2_t type;
};
template <>
struct KeyPiece<16> {
  typedef uint4_t type;
};
template <int KL, int VL, int META, int NG>
struct WideTile {
  typename KeyPiece<KL>::type k0, k1, k2, k3;  // products 0 .. 3
  uint2_t t0, t1, t2, t3;                      // 3-bit keys
  MetaBlock<META, NG> kmeta, vmeta;            // lane = token
  Unit16 v00, v01, v10, v11;                   // lane = unit, as in TileData
  uint2_t vt0, vt1;
};

template <int KL, int VL, int META, int NG>
__global__ __launch_bounds__(kThreads, 2) void decode_wide_kernel(Layout L, const __half *__restrict__ q,
                                                                  long long T, long long nq, int n_sink,
                                                                  int n_splits, int passes, int n_new,
                                                                  const __half *__restrict__ knew,
                                                                  const __half *__restrict__ vnew, long long te,
                                                                  ChunkPlan plan, MergeOut mo) {
  // grid (n_splits, Hk * passes, B), as in decode_mfma_kernel, sixteen rows per pass
  constexpr bool TERNARY = VL == 3, K4 = KL == 16, V4 = VL == 16, K3 = KL == 8, V3 = VL == 8;
  constexpr float kCentre = 0.5f * (KL - 1);
  // One group per head: a lane's quarter row is a run of 32 positions.  Two: it is the 16 positions h of
  // each half of the head (h = lane / 16), so that steps 0, 1 of a product lie in one group and steps 2,
  // 3 in the other.
  static_assert(NG == 1 || NG == 2, "one or two equal groups per head");
  constexpr bool SPLIT = NG == 2;
  __shared__ WideSmem<TERNARY, NG> sm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, h = lane >> 4;
  const int sp = blockIdx.x, by = blockIdx.y;
  const int hk = passes == 1 ? by : by / passes, b = blockIdx.z;
  const int n_rows = n_new * L.R;  // rows of this kv head: (query token, query head)
  const int row0 = passes == 1 ? 0 : (by % passes) * kWideRows;
  const int rows_here = min(n_rows - row0, kWideRows);
  const long long head = (long long)b * L.Hk + hk;
  const float c = L.sm_scale * kLog2e;
  auto row_index = [&](int x) {  // of the kv head's row x in q, the partials and the output
    const int j = n_new == 1 ? 0 : x / L.R;
    return ((long long)b * n_new + j) * L.Hq + hk * L.R + (x - j * L.R);
  };

  // ---- queries and permutations: the first requests.  Wavefront w stages rows w and w + 8. ----
  __half2 q2[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = wave + kNW * j;
    q2[j] = __floats2half2_rn(0.f, 0.f);
    if (row < rows_here) q2[j] = reinterpret_cast<const __half2 *>(q + row_index(row0 + row) * kD)[lane];
  }
  const int pk0 = L.perm_k[hk * kD + lane], pk1 = L.perm_k[hk * kD + 64 + lane];
  const int pv = L.perm_v[hk * kD + (tid & 127)];  // for the epilogue

  // ---- the new token taken along: by the same two wavefronts as in decode_mfma_kernel, but ahead of everything else:
  //      here the tiles hold the packed row too, so the last chunk's workgroup waits until it is stored (its chunk is
  //      the shorter for it: kAppendLagTiles) ----
  const bool fused = knew != nullptr;
  if (fused && sp == n_splits - 1) {
    if (wave < 2) append_token(L, knew, vnew, T - 1, plan.new_slot, -1, te, hk, b, wave, lane, sm.append);
    if (wave == 1 && te >= 0) {
      append_lds_sync();
      append_store_units(L, te, hk, b, lane, sm.append);
    }
    __threadfence_block();
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the stores have completed
    asm volatile("" ::: "memory");
    __syncthreads();
  }

  // ---- this chunk ----
  const int n_tiles = (int)((nq + 63) >> 6);
  const int n_long = sp > plan.first_long ? sp - plan.first_long : 0;
  const int tile_begin = sp * plan.tiles_q + n_long;
  const int tile_end = sp == n_splits - 1 ? n_tiles : tile_begin + plan.tiles_q + (sp >= plan.first_long ? 1 : 0);

  constexpr int kRowBytes = K4 ? 64 : K3 ? 48 : 32;
  const uint8_t *kc = L.k_codes + head * L.Tcap * kRowBytes;
  typedef WideTile<KL, VL, META, NG> Tile;
  typedef MetaBlock<META, NG> meta_block;
  const meta_block *km = reinterpret_cast<const meta_block *>(L.k_meta) + head * L.Tcap;
  const meta_block *vm = reinterpret_cast<const meta_block *>(L.v_meta) + head * L.Tcap;
  const uint8_t *vc = L.v_codes + head * L.n_vblocks * L.v_block_bytes;
  const int last_token = (int)(nq - 1);
  const int last_blk = last_token >> 5;
  constexpr int vbb = TERNARY ? kTernaryBlockBytes : V4 ? kFourBitBlockBytes : V3 ? kThreeBitBlockBytes : kTwoBitBlockBytes;
  const unsigned unit_off = TERNARY ? ((13 * lane) & ~3) : V4 ? 32 * lane : V3 ? 24 * lane : 16 * lane;
  const int unit_sh = TERNARY ? ((13 * lane) & 3) : 0;
  // token slot i = lane % 8 of a unit sits in register i / 2, at bits {4, 6, 8, 8} (2-bit) or {6, 8, 8, 8}
  // (3-bit); 3-level and 4-bit units hold all slots at one place: undo what is above the lowest place
  const int pair = (lane >> 1) & 3;
  const float kslot_scale = (TERNARY || V4 || pair == 0) ? 1.f : (V3 || pair == 1) ? 0.25f : 0.0625f;
  constexpr float kUnscale = TERNARY ? 65536.0f : V3 || V4 ? 262144.0f : 1048576.0f;  // codes carry 2^(place - 24)
  const int safe_last_tile = n_tiles > 0 ? n_tiles - 1 : 0;
  const int safe_last_token = last_token > 0 ? last_token : 0;
  const int safe_last_blk = last_blk > 0 ? last_blk : 0;
  // (streaming loads where one instruction takes whole cache lines: a product's quarter rows together
  // are four runs of four 32-byte key rows)
  constexpr bool kStreamK = KL == 4 && !SPLIT, kStreamV = VL == 3 || VL == 4, kStreamM = KL == 4;
  const int tile_cap = max(min(tile_end - 1, safe_last_tile), 0);
  const unsigned tok0 = 8 * (col >> 2) + (col & 3);  // this lane's token in product 0; + 4, 32, 36 in the others
  // where the lane's piece of a key row starts, and its (first) dword of the 3-bit plane
  const unsigned piece_off = (SPLIT ? (K4 ? 8u : 4u) : (K4 ? 16u : 8u)) * h, top_off = 32u + 4u * (SPLIT ? h >> 1 : h);
  auto load_tile = [&](const int tile) {
    Tile d;
    const unsigned rows_last = (unsigned)(safe_last_token - tile * 64);  // >= 0; rows past it repeat it
    const uint8_t *kt = kc + (size_t)tile * (64 * kRowBytes);
    auto load_key = [&](unsigned token, typename KeyPiece<KL>::type &k, uint2_t &top) {
      const unsigned row = min(token, rows_last) * (unsigned)kRowBytes, at = row + piece_off;
      if constexpr (K4) {
        if constexpr (SPLIT) {
          const uint2_t lo = *reinterpret_cast<const uint2_t *>(kt + at), hi = *reinterpret_cast<const uint2_t *>(kt + at + 32);
          k = uint4_t{lo.x, lo.y, hi.x, hi.y};
        } else {
          k = *reinterpret_cast<const uint4_t *>(kt + at);
        }
      } else if constexpr (SPLIT) {
        k = uint2_t{*reinterpret_cast<const unsigned *>(kt + at), *reinterpret_cast<const unsigned *>(kt + at + 16)};
        if constexpr (K3)
          top = uint2_t{*reinterpret_cast<const unsigned *>(kt + row + top_off),
                        *reinterpret_cast<const unsigned *>(kt + row + top_off + 8)};
      } else {
        k = load_as<kStreamK>(reinterpret_cast<const uint2_t *>(kt + at));
        if constexpr (K3) top.x = *reinterpret_cast<const unsigned *>(kt + row + top_off);
      }
    };
    load_key(tok0, d.k0, d.t0);
    load_key(tok0 + 4, d.k1, d.t1);
    load_key(tok0 + 32, d.k2, d.t2);
    load_key(tok0 + 36, d.k3, d.t3);
    const unsigned moff = min((unsigned)lane, rows_last) * (unsigned)sizeof(meta_block);
    d.kmeta = stream_load_block<kStreamM>(reinterpret_cast<const meta_block *>(
        reinterpret_cast<const uint8_t *>(km + (size_t)tile * 64) + moff));
    d.vmeta = stream_load_block<kStreamM>(reinterpret_cast<const meta_block *>(
        reinterpret_cast<const uint8_t *>(vm + (size_t)tile * 64) + moff));
    const int blk0 = min(2 * tile, safe_last_blk), blk1 = min(blk0 + 1, safe_last_blk);
    const uint8_t *vb0 = vc + (size_t)blk0 * vbb, *vb1 = vc + (size_t)blk1 * vbb;
    unsigned uoff = unit_off;  // (hidden from the compiler: the block's address stays scalar)
    asm("" : "+v"(uoff));
    d.v00 = stream_load_unit<kStreamV>(vb0 + uoff);
    d.v10 = stream_load_unit<kStreamV>(vb1 + uoff);
    if constexpr (V3) {
      d.vt0 = stream_load_pair<kStreamV>(vb0 + uoff + 16);
      d.vt1 = stream_load_pair<kStreamV>(vb1 + uoff + 16);
    }
    if constexpr (V4) {
      d.v01 = stream_load_unit<kStreamV>(vb0 + uoff + 16);
      d.v11 = stream_load_unit<kStreamV>(vb1 + uoff + 16);
    }
    return d;
  };

  // ---- the fp16 tokens: slices of four, slice j of the chunk's (j = sp, sp + n_splits, ...) goes to one
  //      team of wavefronts, and in it wavefront (row quad) serves four rows; the younger wavefronts'
  //      team is first in line ----
  const int n_win = (int)(T - nq) - n_sink, W = L.W;
  const int n_fp = n_sink + n_win;
  const int n_slices = (n_fp + kWideSlice - 1) / kWideSlice;
  const int ring_stride = n_splits * kWideTeams;
  const int quad = wave % (kNW / kWideTeams), team = kWideTeams - 1 - wave / (kNW / kWideTeams);
  const int ring_first = sp + n_splits * team;
  const bool ring_owner = ring_first < n_slices && kRowQuad * quad < rows_here;
  const int slot0 = plan.slot0;
  const __half *kwin = L.k_win + head * (W + L.S) * kD;
  const __half *vwin = L.v_win + head * (W + L.S) * kD;
  // (fp16 token t, clamped to the last one, sits in sink row W + t if it is a sink, else in ring slot
  // slot0 + t - n_sink modulo W; the newest token's row is the caller's when it is taken along)
  auto load_ring = [&](int slice) {
    WideRing d;
    const int t = min(slice * kWideSlice + (lane >> 4), n_fp - 1);
    const int s = slot0 + t - n_sink;
    const int slot = t < n_sink ? W + t : (s >= W ? s - W : s);
    const int fresh = fused && t >= n_fp - 1 ? 1 : 0;
    const unsigned row_bytes = (unsigned)slot * (unsigned)(kD * sizeof(__half));
    const char *krow = fresh ? reinterpret_cast<const char *>(knew + head * kD)
                             : reinterpret_cast<const char *>(kwin) + row_bytes;
    d.k = reinterpret_cast<const uint4_t *>(krow)[lane & 15];
#pragma unroll
    for (int k = 0; k < kWideSlice; ++k) {
      const unsigned vb = (unsigned)__builtin_amdgcn_readlane((int)row_bytes, 16 * k);
      const char *vrow = __builtin_amdgcn_readlane(fresh, 16 * k) ? reinterpret_cast<const char *>(vnew + head * kD)
                                                                   : reinterpret_cast<const char *>(vwin) + vb;
      d.v[k] = reinterpret_cast<const unsigned *>(vrow)[lane];
    }
    return d;
  };

  // ---- prologue: small loads, two tiles, the table and the queries' staging in their shadow ----
  WideRing ring = {};
  if (ring_owner) ring = load_ring(ring_first);
  asm volatile("" ::: "memory");
  const int share = wave < kNW / 2 ? kOldShare : kYoungShare;
  const int deal_base = wave < kNW / 2 ? wave : kOldShare * (kNW / 2) + (wave - kNW / 2);
  auto tile_of = [&](int n) {  // n-th tile of this wave
    const int r = n / share;
    return tile_begin + kDealPeriod * r + deal_base + (kNW / 2) * (n - share * r);
  };
  int n_a = 0, n_b = 1, n_c = 2;
  int tile_a = tile_of(n_a), tile_b = tile_of(n_b), tile_c = tile_of(n_c);
  Tile buf_a, buf_b, buf_c;
  buf_a = load_tile(min(tile_a, tile_cap));
  if constexpr (TERNARY) build_ternary_table(sm.lut4[wave], sm.lut, tid);
  asm volatile("" ::: "memory");
  buf_b = load_tile(min(tile_b, tile_cap));
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = wave + kNW * j;
    reinterpret_cast<__half2 *>(sm.qraw[row])[lane] = q2[j];
  }
  if (tid < 128) sm.perm_v[tid] = pv;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = wave + kNW * j;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int p = lane + 64 * half;
      int step, quarter, slot, shift;
      if constexpr (K4) {
        int x, kslot;
        k4_slot_of(p, x, kslot, shift);  // x = 2 * (dword of the row) + operand half
        const int dw = x >> 1;
        quarter = SPLIT ? (dw & 7) >> 1 : dw >> 2;
        step = SPLIT ? (dw & 1) + 2 * (dw >> 3) : dw & 3;
        slot = 4 * (x & 1) + kslot;
      } else {
        int x, kslot;
        k_slot_of(p, x, kslot, shift);  // x = 4 * (dword of the row) + quarter of its operands
        const int dw = x >> 2;
        quarter = SPLIT ? dw & 3 : dw >> 1;
        step = 2 * (SPLIT ? dw >> 2 : dw & 1) + ((x & 3) >> 1);
        slot = 4 * (x & 1) + kslot;
      }
      const float x = (float)sm.qraw[row][half ? pk1 : pk0];
      sm.qa[step][quarter][row][slot] = (_Float16)ldexpf(x, 8 - shift);  // exact: a power of two
      float s16 = x;  // sum over the 16 positions of this row of lanes
      s16 += row_move<kQuadSwap1>(s16);
      s16 += row_move<kQuadSwap2>(s16);
      s16 += row_move<kRowHalfMirror>(s16);
      s16 += row_move<kRowMirror>(s16);
      if ((lane & 15) == 0) sm.qpart[row][p >> 4] = s16;
    }
  }
  __syncthreads();
  // the score product's B operands: held in registers, or (two groups: registers) re-read from LDS
  half8_t qop[SPLIT ? 1 : 4];
  if constexpr (!SPLIT) {
#pragma unroll
    for (int s = 0; s < 4; ++s) qop[s] = *reinterpret_cast<const half8_t *>(sm.qa[s][h][col]);
  }
  // per group, for this lane's row: sm_scale*log2(e) * sum of the reordered query, and the start value
  // of the score accumulators (centred codes, see decode_mfma_kernel)
  float qsc[NG], dinit[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    float sum = 0.f;
#pragma unroll
    for (int x = 0; x < 8 / NG; ++x) sum += sm.qpart[col][g * (8 / NG) + x];
    qsc[g] = c * sum;
    dinit[g] = -kCentre * sum * (1.0f / 65536.0f);
  }

  // ---- fp16 slices of this wave: plain vector arithmetic, four rows ----
  {
    float rm[kRowQuad], rl[kRowQuad], ro[kRowQuad][2];  // reference, sum of weights, outputs
#pragma unroll
    for (int r = 0; r < kRowQuad; ++r) rm[r] = -INFINITY, rl[r] = 0.f, ro[r][0] = ro[r][1] = 0.f;
    if (ring_owner) {
      // query token j sees the fp16 tokens up to its own, index n_fp - n_new + j
      int ring_last[kRowQuad];
#pragma unroll
      for (int r = 0; r < kRowQuad; ++r)
        ring_last[r] = n_new == 1 ? n_fp - 1 : n_fp - n_new + (row0 + kRowQuad * quad + r) / L.R;
      auto ring_slice = [&](const WideRing &rd, const int slice) {
        const int tok = slice * kWideSlice + (lane >> 4), pc = lane & 15;
        const bool valid = tok < n_fp;
        const half8_t x = __builtin_bit_cast(half8_t, rd.k);
        float p[kRowQuad][kWideSlice];
#pragma unroll
        for (int r = 0; r < kRowQuad; ++r) {
          const half8_t qr = *reinterpret_cast<const half8_t *>(&sm.qraw[kRowQuad * quad + r][8 * pc]);
          float s = (float)qr[0] * (float)x[0];
#pragma unroll
          for (int e = 1; e < 8; ++e) s = fmaf((float)qr[e], (float)x[e], s);
          s += row_move<kQuadSwap1>(s);
          s += row_move<kQuadSwap2>(s);
          s += row_move<kRowHalfMirror>(s);
          s += row_move<kRowMirror>(s);  // all sixteen lanes of a token now hold its score
          s = valid && tok <= ring_last[r] ? c * s : -INFINITY;
          float sk[kWideSlice];
#pragma unroll
          for (int k = 0; k < kWideSlice; ++k)
            sk[k] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, s), 16 * k));
          const float mnew = fmaxf(rm[r], fmaxf(fmaxf(sk[0], sk[1]), fmaxf(sk[2], sk[3])));
          // (a row may see none of a slice's tokens, nor of the earlier ones: everything stays zero)
          const float mref = mnew == -INFINITY ? 0.f : mnew;
          const float f = fast_exp2(rm[r] - mref);
#pragma unroll
          for (int k = 0; k < kWideSlice; ++k) p[r][k] = fast_exp2(sk[k] - mref);
          rl[r] = rl[r] * f + (p[r][0] + p[r][1]) + (p[r][2] + p[r][3]);
          ro[r][0] *= f;
          ro[r][1] *= f;
          rm[r] = mnew;
        }
#pragma unroll
        for (int k = 0; k < kWideSlice; ++k) {
          const __half2 v2 = __builtin_bit_cast(__half2, rd.v[k]);
          const float vx = __low2float(v2), vy = __high2float(v2);
#pragma unroll
          for (int r = 0; r < kRowQuad; ++r) {
            ro[r][0] = fmaf(p[r][k], vx, ro[r][0]);
            ro[r][1] = fmaf(p[r][k], vy, ro[r][1]);
          }
        }
      };
      if (ring_first + ring_stride >= n_slices) {
        ring_slice(ring, ring_first);
      } else {
        for (int slice = ring_first; slice < n_slices; slice += ring_stride) {
          WideRing ring_next = ring;
          if (slice + ring_stride < n_slices) ring_next = load_ring(slice + ring_stride);
          ring_slice(ring, slice);
          ring = ring_next;
        }
        asm volatile("" ::"v"(ring.k.x), "v"(ring.k.y), "v"(ring.k.z), "v"(ring.k.w), "v"(ring.v[0]),
                     "v"(ring.v[1]), "v"(ring.v[2]), "v"(ring.v[3]));
      }
    }
#pragma unroll
    for (int r = 0; r < kRowQuad; ++r)
      *reinterpret_cast<float2 *>(&sm.ring_o[wave][r][2 * lane]) = make_float2(ro[r][0], ro[r][1]);
    if (lane == 0) {
#pragma unroll
      for (int r = 0; r < kRowQuad; ++r) sm.rm[kRowQuad * quad + r][team] = rm[r], sm.rl[kRowQuad * quad + r][team] = rl[r];
    }
  }

  float mref = 0.f, lsum = 0.f, zacc[NG];  // of this lane's row, over this lane's tokens
#pragma unroll
  for (int g = 0; g < NG; ++g) zacc[g] = 0.f;
  float beta = 1.f, vs_limit = kVsLimit;
  float minus_one = -1.0f;
  asm("" : "+v"(minus_one));
  float4_t acc[8];  // O^T: positions 16n + 4h .. + 3 of the row
#pragma unroll
  for (int n = 0; n < 8; ++n) acc[n] = float4_t{0.f, 0.f, 0.f, 0.f};
  bool first = true;

  auto compute_tile = [&](const Tile &cur, const int tile) {
    const bool tail = tile * 64 + 63 > last_token;  // (scalar) only the cache's last tile has tokens to drop

    // ---- lane = token: the factors of its (scale, zero) pairs ----
    float vs[NG], vz[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const float2 vmeta = meta_value(cur.vmeta.m[g]);
      vs[g] = vmeta.x, vz[g] = vmeta.y;
    }
    if (tail) {
      const bool valid = tile * 64 + lane <= last_token;
#pragma unroll
      for (int g = 0; g < NG; ++g) vs[g] = valid ? vs[g] : 0.f, vz[g] = valid ? vz[g] : 0.f;
    }
    float vs_top = vs[0];
#pragma unroll
    for (int g = 1; g < NG; ++g) vs_top = fmaxf(vs_top, vs[g]);
    if (first || __any(vs_top > vs_limit)) {
      const float vsmax = wave_max(vs_top);
      if (vsmax > 0.f) {
        int e;
        (void)frexpf(vsmax, &e);          // vsmax = fr * 2^e, fr in [0.5, 1)
        const float nb = ldexpf(1.f, 8 - e);  // vsmax * nb in [128, 256)
        const float g = nb / beta;
        beta = nb;
        vs_limit = kVsLimit / nb;
        if (!first) {
#pragma unroll
          for (int n = 0; n < 8; ++n) acc[n] *= g;
        }
      }
    }
    const float bk = beta * kslot_scale;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const float2 kmeta = meta_value(cur.kmeta.m[g]);
      sm.ktok[wave][g][tok_slot(lane)] = make_float2(kmeta.x * (c * 65536.0f), fmaf(kCentre, kmeta.x, kmeta.y));
      sm.vtok[wave][g][tok_slot(lane)] = make_float2(vs[g] * bk, vz[g]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // ---- scores, log2 domain, minus the running reference: u[4x + i] is token 32 (x/2) + 8h + 4 (x%2) + i ----
    float u[16];
    auto product = [&](const int x, const typename KeyPiece<KL>::type &k, const uint2_t &top) {
      half8_t a[4];
      if constexpr (K4) {
        const unsigned w[4] = {k.x, k.y, k.z, k.w};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          half4_t o[2];
          unpack_k4(w[s], o);
          a[s] = join(o[0], o[1]);
        }
      } else {
        half4_t lo[4], hi[4];
        if constexpr (K3 && SPLIT) {
          unpack_k3_of(h & 1, k.x, top.x, lo);
          unpack_k3_of(h & 1, k.y, top.y, hi);
        } else if constexpr (K3) {
          unpack_k3<0>(k.x, top.x, lo);
          unpack_k3<1>(k.y, top.x, hi);
        } else {
          unpack_k(k.x, lo);
          unpack_k(k.y, hi);
        }
        a[0] = join(lo[0], lo[1]), a[1] = join(lo[2], lo[3]), a[2] = join(hi[0], hi[1]), a[3] = join(hi[2], hi[3]);
      }
      float4_t d[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) d[g] = float4_t{dinit[g], dinit[g], dinit[g], dinit[g]};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        half8_t qs;
        if constexpr (SPLIT) qs = *reinterpret_cast<const half8_t *>(sm.qa[s][h][col]); else qs = qop[s];
        d[s * NG / 4] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s], qs, d[s * NG / 4], 0, 0, 0);
      }
      const int slot = tok_slot(32 * (x >> 1) + 8 * h) + 4 * (x & 1);
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        float u0 = -mref, u1 = -mref;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const float4_t f = *reinterpret_cast<const float4_t *>(&sm.ktok[wave][g][slot + i]);
          u0 = fmaf(d[g][i], f[0], fmaf(f[1], qsc[g], u0));
          u1 = fmaf(d[g][i + 1], f[2], fmaf(f[3], qsc[g], u1));
        }
        u[4 * x + i] = u0, u[4 * x + i + 1] = u1;
      }
      __builtin_amdgcn_sched_barrier(0);  // (else the factors of all products are read first: registers)
    };
    product(0, cur.k0, cur.t0);
    product(1, cur.k1, cur.t1);
    product(2, cur.k2, cur.t2);
    product(3, cur.k3, cur.t3);
    if (tail) {
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (tile * 64 + 32 * (x >> 1) + 8 * h + 4 * (x & 1) + i > last_token) u[4 * x + i] = -INFINITY;
    }
    float u_top = fmaxf(u[0], u[1]);
#pragma unroll
    for (int x = 2; x < 16; ++x) u_top = fmaxf(u_top, u[x]);
    if (first || __any(u_top > kRefSlack)) {
      // move the row's reference and rescale what is accumulated (the row's other tokens: lanes 16 apart)
      float umax = fmaxf(u_top, __shfl_xor(u_top, 16));
      umax = fmaxf(umax, __shfl_xor(umax, 32));
      const float delta = first ? umax : fmaxf(umax, 0.f);
      const float f = first ? 0.f : exp2f(-delta);
      mref += delta;
      lsum *= f;
#pragma unroll
      for (int g = 0; g < NG; ++g) zacc[g] *= f;
#pragma unroll
      for (int x = 0; x < 16; ++x) u[x] -= delta;
      if (!first) {
#pragma unroll
        for (int n = 0; n < 8; ++n) acc[n] *= f;
      }
      first = false;
    }

    // ---- weights: p * value scale as two fp16 numbers, its top 11 bits (toward zero) and the rest ----
    half8_t ph[2][NG], pl[2][NG];
    auto weights = [&](const int blk) {
      float p[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = fast_exp2(u[8 * blk + e]);
        lsum += p[e];
      }
      const int slot = tok_slot(32 * blk + 8 * h);
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const float4_t f = *reinterpret_cast<const float4_t *>(&sm.vtok[wave][g][slot + e]);
          const float wa = p[e] * f[0], wb = p[e + 1] * f[2];
          zacc[g] = fmaf(p[e], f[1], zacc[g]);
          zacc[g] = fmaf(p[e + 1], f[3], zacc[g]);
          const auto hi = __builtin_amdgcn_cvt_pkrtz(wa, wb);
          ph[blk][g][e] = (_Float16)hi[0], ph[blk][g][e + 1] = (_Float16)hi[1];
          pl[blk][g][e] = (_Float16)__builtin_fmaf((float)hi[0], minus_one, wa);
          pl[blk][g][e + 1] = (_Float16)__builtin_fmaf((float)hi[1], minus_one, wb);
        }
    };
    // ---- values.  The products of a tile go to accumulators of their own, low parts
    //      first, and these are added to the running ones: the matrix core truncates what it adds,
    //      and this way it truncates against one tile's sum, not against all tiles' so far. ----
    half8_t va[2][4];  // [block][channel tile of four]: A operands
    auto operands = [&](const int blk, const int n0) {
      const Unit16 raw = blk ? cur.v10 : cur.v00;
      if constexpr (V4) {
        const Unit16 w = n0 ? (blk ? cur.v11 : cur.v01) : raw;
        va[blk][0] = unpack_wide_v4(w.x), va[blk][1] = unpack_wide_v4(w.y);
        va[blk][2] = unpack_wide_v4(w.z), va[blk][3] = unpack_wide_v4(w.w);
      } else if constexpr (TERNARY) {
        unsigned f[8];
        ternary_fields(raw, unit_sh, f);
#pragma unroll
        for (int n = 0; n < 4; ++n)
          va[blk][n] = *reinterpret_cast<const half8_t *>(reinterpret_cast<const char *>(sm.lut) + f[n0 + n]);
      } else {
        const unsigned w0 = n0 ? raw.z : raw.x, w1 = n0 ? raw.w : raw.y;
        if constexpr (V3) {
          const uint2_t tops = blk ? cur.vt1 : cur.vt0;
          const unsigned top = n0 ? tops.y : tops.x;
          va[blk][0] = unpack_wide_v3<0>(w0, top), va[blk][1] = unpack_wide_v3<1>(w0 >> 8, top);
          va[blk][2] = unpack_wide_v3<2>(w1, top), va[blk][3] = unpack_wide_v3<3>(w1 >> 8, top);
        } else {
          va[blk][0] = unpack_v_field(w0), va[blk][1] = unpack_v_field(w0 >> 8);
          va[blk][2] = unpack_v_field(w1), va[blk][3] = unpack_v_field(w1 >> 8);
        }
      }
    };
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      weights(blk);
      if constexpr (NG > 1) __builtin_amdgcn_sched_barrier(0);  // (as above)
    }
#pragma unroll
    for (int n0 = 0; n0 < 8; n0 += 4) {
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) operands(blk, n0);
      float4_t t[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) t[n] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int blk = 0; blk < 2; ++blk)
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const int g = (n0 + n) * NG / 8;
            t[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va[blk][n], part ? ph[blk][g] : pl[blk][g], t[n], 0, 0, 0);
          }
#pragma unroll
      for (int n = 0; n < 4; ++n) acc[n0 + n] += t[n];
      if constexpr (NG > 1) __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_wave_barrier();
  };
  // (the loops of decode_mfma_kernel: no early exit, exact wait counters)
  if constexpr (K4 || V4 || K3 || V3 || NG > 1) {
    while (tile_b < tile_end) {
      compute_tile(buf_a, tile_a);
      tile_a = tile_of(n_a += 2);
      buf_a = load_tile(min(tile_a, tile_cap));
      compute_tile(buf_b, tile_b);
      tile_b = tile_of(n_b += 2);
      buf_b = load_tile(min(tile_b, tile_cap));
    }
  } else {
    while (tile_c < tile_end) {
      buf_c = load_tile(min(tile_c, tile_cap));
      compute_tile(buf_a, tile_a);
      tile_a = tile_of(n_a += 3);
      buf_a = load_tile(min(tile_a, tile_cap));
      compute_tile(buf_b, tile_b);
      tile_b = tile_of(n_b += 3);
      buf_b = load_tile(min(tile_b, tile_cap));
      compute_tile(buf_c, tile_c);
      tile_c = tile_of(n_c += 3);
    }
  }
#pragma unroll 1
  for (int k = 0; k < 2 && tile_a < tile_end; ++k) {
    compute_tile(buf_a, tile_a);
    buf_a = buf_b;
    tile_a = tile_b;
    tile_b = tile_end;
  }

  // ---- epilogue: fold the four lanes of a row, then the waves and the fp16 slices ----
  lsum += __shfl_xor(lsum, 16);
  lsum += __shfl_xor(lsum, 32);
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    zacc[g] += __shfl_xor(zacc[g], 16);
    zacc[g] += __shfl_xor(zacc[g], 32);
  }
  if (lane < kWideRows) {
    sm.wm[col][wave] = first ? -INFINITY : mref;
    sm.wl[col][wave] = lsum;
#pragma unroll
    for (int g = 0; g < NG; ++g) sm.wz[col][g][wave] = zacc[g];
  }
  __syncthreads();  // (the table's bytes become the stage)
  {
    const float unscale = kUnscale / beta;
#pragma unroll
    for (int n = 0; n < 8; ++n)
      *reinterpret_cast<float4_t *>(&sm.stage[wave][col][16 * n + 4 * h]) = acc[n] * unscale;
  }
  __syncthreads();
  // thread (row r, positions 4x .. 4x+3)
  const int r = tid >> 5, x = tid & 31;
  static_assert(kThreads == kWideRows * kD / 4, "one thread per row and four positions");
  if (r < rows_here) {
    float ref[kNW + kWideTeams], sum[kNW + kWideTeams], m = -INFINITY;
#pragma unroll
    for (int w = 0; w < kNW + kWideTeams; ++w) {
      sum[w] = w < kNW ? sm.wl[r][w] : sm.rl[r][w - kNW];
      const float y = w < kNW ? sm.wm[r][w] : sm.rm[r][w - kNW];
      ref[w] = sum[w] > 0.f ? y : -INFINITY;  // (without tokens: no meaningful reference)
      m = fmaxf(m, ref[w]);
    }
    float den = 0.f;
    float4_t num = {0.f, 0.f, 0.f, 0.f};
    const int4 pv4 = *reinterpret_cast<const int4 *>(&sm.perm_v[4 * x]);
    const int ch[4] = {pv4.x, pv4.y, pv4.z, pv4.w};
    const int zg = x * NG / 32;
#pragma unroll
    for (int w = 0; w < kNW; ++w) {
      const float e = sum[w] > 0.f ? fast_exp2(ref[w] - m) : 0.f;
      den = fmaf(e, sum[w], den);
      const float4_t o = *reinterpret_cast<const float4_t *>(&sm.stage[w][r][4 * x]);
      num += e * (o + sm.wz[r][zg][w]);
    }
#pragma unroll
    for (int t = 0; t < kWideTeams; ++t) {
      const float e = sum[kNW + t] > 0.f ? fast_exp2(ref[kNW + t] - m) : 0.f;
      den = fmaf(e, sum[kNW + t], den);
      const float *o = sm.ring_o[(kWideTeams - 1 - t) * (kNW / kWideTeams) + r / kRowQuad][r % kRowQuad];
#pragma unroll
      for (int k = 0; k < 4; ++k) num[k] = fmaf(e, o[ch[k]], num[k]);
    }
    const long long idx = row_index(row0 + r);
    if (mo.mode == kMergeDirect) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float o = num[k] / den;
        mo.out_f32[idx * kD + ch[k]] = o;
        if (mo.out_f16) mo.out_f16[idx * kD + ch[k]] = __float2half_rn(o);
      }
    } else {
      float *part = L.workspace + (idx * (SKVQ_MAX_SPLITS + 1) + sp) * kPartialStride;
#pragma unroll
      for (int k = 0; k < 4; ++k) part[4 + ch[k]] = num[k];
      if (x == 0) {
        part[0] = m;
        part[1] = den;
      }
    }
  }
}

}  // namespace
}  // namespace skvq
