// decode.hip -- single-query bifocal-RoPE decode on a raw KV cache, gfx950.
//
// Jet-Long (arXiv 2607.07740), Sec. 3.2: the cache keeps keys in their base
// coordinates and is never rewritten when G changes; the remote view of a key
// is formed on the fly by rotating it to f(k) (the correction rotation of
// Eqs. (5)-(6), applied here to raw keys as R(f(k)) x_k = R(Delta k) R(k) x_k).
// The query of sequence b sits at q = kv_len[b] - 1 and G follows from
// L = kv_len[b] (Eq. (2)), computed on the device, so one launch serves a
// ragged batch whose sequences have different G.
//
// Split-K: workgroup (group of up to 4 kv heads, w) streams the w-th equal
// part of the batch's 16-key steps, two waves per kv head, whatever sequences
// that part spans (SplitRange), so a ragged batch keeps every CU busy for
// the same time.  The Sec. 4.5 frequency map replaces the remote
// rotation by one at unchanged positions with rescaled frequencies.  The g query
// heads of a kv head are rotated twice (base and remote) and placed in the 16
// columns of a v_mfma_f32_16x16x32_bf16 B operand: columns 0..7 hold
// the base-rotated heads, 8..15 the remote-rotated ones.  Each key is rotated
// once, to the view its distance selects (Eq. (1)), and scored against both
// column groups; a column keeps only keys of its own view, so every column is
// the partial softmax state (m, l, O) of one (head, view) pair: the local
// window state and the remote-only state of Sec. 3.3.  Each split merges its
// head's two view states with the max-shifted, linear-space rule of Eq. (7)
// in fp32, and the reduce kernel merges the splits' states the same way.
#include <algorithm>
#include <climits>
#include <mutex>
#include <type_traits>

#include "jl_device.h"

namespace jl {

constexpr int kDecHeads = 4;  // kv heads per workgroup
constexpr int kDecWaves = 8;  // two waves per head: one takes the even steps, one the odd
constexpr int kDecThreads = 64 * kDecWaves;
constexpr int kDecTile = 16;  // keys per step
constexpr int kDecBufs = 4;   // LDS buffers: the two steps in use and the next two in flight
constexpr int kDecImgBytes = kDecTile * kDecHeads * kHeadDim * 2;  // K or V of one step: 16 KB
constexpr int kDecBufBytes = 2 * kDecImgBytes + 1024;  // K, V and the step's two query cos/sin rows
constexpr int kDecOffTab = kDecBufs * kDecBufBytes;
constexpr int kDecTabRow = kHalf * 8 + 16;  // one offset row: 64 (cos, sin) pairs + 16 B pad
constexpr int kDecOffTab2 = kDecOffTab + kDecTile * kDecTabRow;    // + 16 offset rows (base)
constexpr int kDecOffDummy = kDecOffTab2 + kDecTile * kDecTabRow;  // + 16 offset rows (freq map),
                                                                   // or the raw query rows
constexpr int kDecOffPages = kDecOffDummy + 1024;                  // + landing slot for padding copies
constexpr int kDecPageCap = 2048;  // paged caches: page indices of up to this many steps in LDS
constexpr int kDecSmem = kDecOffPages + kDecPageCap * 4;
constexpr int kDecCopies = 5;  // copies per step of wave 0: four K/V (padded to a fixed count) + rows
constexpr int kStateFloats = 132;  // m, l, the split count (int bits, B = 1), pad, O[128]
// What a workgroup pays for each further sequence it works on (refilling the
// copy pipeline, merging and writing the states), in steps of the copy stream.
constexpr int kDecSegCost = 4;

struct DecodeArgs {
  const uint16_t* q;
  const uint16_t* kc;
  const uint16_t* vc;
  const int32_t* kv_lens;
  float* ws;
  const float2* table;
  int B, Hq, Hkv, g, max_len;  // max_len: most keys a sequence can hold
  // paged caches: kc, vc are pools [n_pages][page_size][Hkv][128] and key k of
  // sequence b sits in page block_table[b][k >> page_shift]; nullptr: dense
  // caches [B][max_len][Hkv][128]
  const int32_t* block_table;
  int max_pages, n_pages, page_shift;
  int n_hgroups;  // groups of up to 4 kv heads
  int n_wg;       // workgroups per kv-head group
  int n_slots;    // state slots (see SplitRange)
  int w_pre, w0;
  float q_scale;
};

// Frequency-interpolation remote map (Sec. 4.5): omega_i and the ramp gamma_i
// of each frequency pair; every workgroup forms the cos/sin rows it needs from
// them and its sequence's length.  Kernel arguments of that map's kernels only:
// 1 KB that every other launch would carry too.
struct FreqRamp {
  double omega[kHalf];
  double gamma[kHalf];
};
struct NoRamp {};
template <bool FREQ>
using RampOf = std::conditional_t<FREQ, FreqRamp, NoRamp>;

__device__ inline int clamp_len(int n, int max_len) { return n < 1 ? 1 : (n > max_len ? max_len : n); }

// The batch's 16-key steps are one list, sequence after sequence, and
// workgroup w of a kv-head group takes an equal range of it: about one
// workgroup per CU, all finishing together whatever the lengths are.  A range
// may end one sequence and begin others; each (workgroup, sequence) pair is a
// split.  A batch's sequences are followed by kDecSegCost empty steps each in
// the list, so that a workgroup with more splits gets fewer keys.  The splits
// of one range are in list order, so w + b names a split: it is the slot of
// its states, and a sequence's slots are consecutive.  (Split counts rounded
// up per sequence, ceil(steps / u) of them, left the longest workgroup 10%
// above the mean at 32 sequences of 0.5K to 16K keys, and above 64 sequences
// every one was cut by max_len.)
//
// The range only counts a split's steps.  Where a sequence spans several whole
// ranges, their workgroups interleave: of n of them, the i-th takes every n-th
// step from its i-th on, so that at any moment they stream one narrow window
// of the cache.  Each streaming its own run of steps instead took 3% longer at
// 128K keys and 4% at 8 sequences of 32K to 128K.
struct SplitRange {
  int b;        // first sequence
  int off;      // first step of it (past its last one: inside its empty steps)
  int left;     // steps of the list, empty ones included; 0: nothing to do
  int n_wg;     // workgroups with a range
  uint32_t pos; // list entry of sequence b's first step
  uint32_t q, r;  // entries per range, and ranges (the first ones) with one more; q = 0: a list
                  // too long for 32 bits, whose splits all take runs of steps
};

__device__ inline int seq_steps(const DecodeArgs& a, int b) {
  return (clamp_len(a.kv_lens[b], a.max_len) + kDecTile - 1) / kDecTile;
}

// Ranges of a list of V < 2^32 entries, and where range w begins
__device__ inline uint32_t set_ranges(SplitRange& s, int n_wg, uint32_t V, int w) {
  s.n_wg = min((uint32_t)n_wg, V);
  s.q = V / (uint32_t)s.n_wg;
  s.r = V - s.q * s.n_wg;
  s.left = w < s.n_wg ? (int)(s.q + ((uint32_t)w < s.r ? 1 : 0)) : 0;
  return s.q * w + min((uint32_t)w, s.r);
}
// The workgroup whose range holds list entry x
__device__ inline int range_of(const SplitRange& s, uint32_t x) {
  const uint32_t head = s.r * (s.q + 1);
  return (int)(x < head ? x / (s.q + 1) : s.r + (x - head) / s.q);
}

__device__ inline SplitRange split_range(const DecodeArgs& a, int w) {
  SplitRange s;
  const int lane = threadIdx.x & 63;
  if (a.B == 1) {
    s.b = 0;
    s.pos = 0;
    s.off = (int)set_ranges(s, a.n_wg, (uint32_t)seq_steps(a, 0), w);
    return s;
  }
  if (a.B <= 64) {  // one lane per sequence, every wave for itself
    const int v = lane < a.B ? seq_steps(a, lane) + kDecSegCost : 0;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(incl, o);
      if (lane >= o) incl += x;
    }
    const int x0 = (int)set_ranges(s, a.n_wg, (uint32_t)__builtin_amdgcn_readlane(incl, 63), w);
    const int b = min((int)__popcll(__ballot(incl <= x0)), a.B - 1);
    s.b = __builtin_amdgcn_readfirstlane(b);
    s.pos = (uint32_t)__builtin_amdgcn_readlane(incl - v, s.b);
    s.off = x0 - (int)s.pos;
    return s;
  }
  // larger batches: one thread per run of ceil(B / threads) sequences
  __shared__ unsigned long long s_sum[kDecWaves];
  __shared__ int s_at[3];
  const int tid = threadIdx.x, wave = tid >> 6;
  const int per = (a.B + kDecThreads - 1) / kDecThreads;
  const long long b0 = (long long)tid * per;
  const int b1 = (int)min((long long)a.B, b0 + per);
  unsigned long long v = 0;
  for (long long b = b0; b < b1; ++b) v += seq_steps(a, (int)b) + kDecSegCost;
  unsigned long long incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long x = __shfl_up(incl, o);
    if (lane >= o) incl += x;
  }
  if (lane == 63) s_sum[wave] = incl;
  __syncthreads();
  unsigned long long V = 0, before = 0;
#pragma unroll
  for (int i = 0; i < kDecWaves; ++i) {
    if (i < wave) before += s_sum[i];
    V += s_sum[i];
  }
  unsigned long long x0;
  if (V <= 0xffffffffull) {
    x0 = set_ranges(s, a.n_wg, (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)V), w);
  } else {
    s.n_wg = a.n_wg;
    s.q = s.r = 0;
    x0 = V / (unsigned)a.n_wg * w + min((unsigned long long)w, V % (unsigned)a.n_wg);
    const unsigned long long len =
        V / (unsigned)a.n_wg + ((unsigned long long)w < V % (unsigned)a.n_wg ? 1 : 0);
    s.left = __builtin_amdgcn_readfirstlane((int)min(len, (unsigned long long)INT_MAX));
  }
  unsigned long long pos = before + incl - v;  // this thread's first list entry
  if (x0 >= pos && x0 < pos + v) {             // exactly one thread when the range is not empty
    long long b = b0;
    int n = seq_steps(a, (int)b) + kDecSegCost;
    while (x0 >= pos + n) {
      pos += n;
      ++b;
      n = seq_steps(a, (int)b) + kDecSegCost;
    }
    s_at[0] = (int)b;
    s_at[1] = (int)(x0 - pos);
    s_at[2] = (int)(uint32_t)pos;
  }
  __syncthreads();
  s.b = __builtin_amdgcn_readfirstlane(s_at[0]);  // not read when nothing is left
  s.off = __builtin_amdgcn_readfirstlane(s_at[1]);
  s.pos = (uint32_t)__builtin_amdgcn_readfirstlane(s_at[2]);
  return s;
}

// Rotate 8 (d, d + 64) pairs given in fp32 by the (cos, sin) pairs c4[0..3]
// (frequencies d..d+7).
__device__ inline void rotate8f(const float* lo, const float* hi, const float4* c4, bf16x8& olo,
                                bf16x8& ohi) {
  float ylo[8], yhi[8];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    float4 w = c4[t];
    int j = 2 * t;
    ylo[j] = lo[j] * w.x - hi[j] * w.y;
    yhi[j] = hi[j] * w.x + lo[j] * w.y;
    ylo[j + 1] = lo[j + 1] * w.z - hi[j + 1] * w.w;
    yhi[j + 1] = hi[j + 1] * w.z + lo[j + 1] * w.w;
  }
  olo = pack8(ylo);
  ohi = pack8(yhi);
}

// Rotate an 8-element pair of slices (d, d + 64) by the (cos, sin) pairs c4[0..3]
// (frequencies d..d+7), optional scale.
__device__ inline void rotate8(const u32x4 rlo, const u32x4 rhi, const float4* c4, float scale,
                               bf16x8& olo, bf16x8& ohi) {
  float lo[8], hi[8], ylo[8], yhi[8];
  unpack8(rlo, lo);
  unpack8(rhi, hi);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    float4 w = c4[t];
    int j = 2 * t;
    ylo[j] = (lo[j] * w.x - hi[j] * w.y) * scale;
    yhi[j] = (hi[j] * w.x + lo[j] * w.y) * scale;
    ylo[j + 1] = (lo[j + 1] * w.z - hi[j + 1] * w.w) * scale;
    yhi[j + 1] = (hi[j + 1] * w.z + lo[j + 1] * w.w) * scale;
  }
  olo = pack8(ylo);
  ohi = pack8(yhi);
}

__device__ inline f32x4 mfma16k16(bf16x4 a, bf16x4 b, f32x4 c) {
  typedef short i16x4v __attribute__((ext_vector_type(4)));
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(i16x4v, a),
                                                   __builtin_bit_cast(i16x4v, b), c, 0, 0, 0);
}

// Maximum over the lanes l, l ^ 16, l ^ 32, l ^ 48, by lane swaps in registers
// (an LDS permute pair in their place cost 2.3 us of a 128K-key call: this
// chain is on every step's critical path).
__device__ inline float max_xor16_32(float x) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Split-K workgroup (group of up to 4 kv heads, w): its splits one after
// another, each some 16-key steps of one sequence (SplitRange).  Every 16-key
// step copies the keys' contiguous head slices (K and V, one key's heads are
// adjacent in the cache) straight into LDS.  Waves w and w + 4 serve kv head
// 4 * group + w on the even and the odd steps, so two waves share each SIMD
// and hide each other's latency; their partial states are merged at the end.
// Four buffers hold the two steps being computed and the next two in flight.
// What the split needs besides its keys (the offset table, the raw query rows)
// is copied to LDS the same way, in front of the first steps, so nothing in
// the prologue is waited for on its own.
//
// Bound by HBM: 1.22 us per 32 KB step and CU at the 6.9 TB/s that the copies
// alone reach.  A call of 131072 keys, 32/8 heads, takes 85 us (6.3 TB/s in all;
// 89 before the prologue, the value reads and the maxima below left the critical
// path); 8 sequences of 32K to 128K 395 us (6.8 TB/s; 402); 32 paged ones of 0.5K
// to 16K 118 us (148).  Requesting every LDS operand of a step at once took 3.5 us more:
// the bursts hold up the copies' writes.
//
// Rotation by tile offset: with k0 the step's first key, a key at k0 + t is
// rotated by t only, R(t) x_k (base view) or by f(k0 + t) - f(k0) (remote
// view), from 16 cos/sin rows kept in LDS, and the query columns are rotated
// by q - k0 or f(q) - f(k0) instead: <R(a) x_q, R(b) x_k> = <R(a - c) x_q,
// R(b - c) x_k> for any c (rotations compose additively, Sec. 3.2 Eq. (6)).
// So no per-key cos/sin row is fetched from memory; the step's two query rows
// arrive with its copies.
//
// LDS layouts (16-byte slots inside one head's 256-byte row of a key t):
//   K: slot s holds chunk s ^ t          (16 keys read at one d: 16 bank groups)
//   V: slot s holds chunk s ^ 2 (t & 7)  (8 keys x 32 B of a transposing read)
//   offset table row r (512 B + 16 B pad, so the 16 rows start 4 banks
//   apart): slot s holds frequencies 2 s, 2 s + 1
// RMODE: 0 the vanilla kernel, 1 bifocal with the Eq. (3) map, 2 bifocal with
// the frequency map (remote rotations at unchanged positions by omega').
// PAGED: page pools and block tables instead of dense caches.
// The Sec. 4.5 map of a sequence of n keys: s = max(1, n / w_pretrained) and
// omega'_i = (1 - gamma_i) omega_i / s + gamma_i omega_i (freq_map_omega);
// the (cos, sin) of pos * omega'_i (freq_map_cs), with the angle formed and
// reduced modulo 2 pi in fp64 (exact to ~1e-11 rad at 1.3e5 rad) and its sine
// and cosine taken in fp32, within an ulp or two of the fp64 result rounded
// to fp32.
__device__ inline double freq_map_omega(const FreqRamp& f, int w_pre, int n, int i) {
#pragma clang fp contract(off)
  const double om = f.omega[i];
  const double sc = fmax(1.0, (double)n / (double)w_pre);
  return (1.0 - f.gamma[i]) * om / sc + f.gamma[i] * om;
}
__device__ inline double freq_map_omega(const NoRamp&, int, int, int) { return 0.0; }
__device__ inline float2 freq_map_cs(double omf, int pos) {
#pragma clang fp contract(off)
  const double two_pi = 6.283185307179586476925286766559;
  double ang = (double)pos * omf;
  ang -= two_pi * rint(ang * (1.0 / two_pi));
  float sn, cs;
  sincosf((float)ang, &sn, &cs);
  return make_float2(cs, sn);
}

// Wait until all but the last n steps' copies of this wave have landed: four
// K/V copies per step, and in wave 0 the step's query cos/sin row too.
__device__ inline void wait_steps(int wave, int n) {
  constexpr int k0 = kDecCopies, k = kDecCopies - 1;
  if (n >= 4) {
    if (wave == 0) wait_vmem_n<4 * k0>(); else wait_vmem_n<4 * k>();
  } else if (n == 3) {
    if (wave == 0) wait_vmem_n<3 * k0>(); else wait_vmem_n<3 * k>();
  } else if (n == 2) {
    if (wave == 0) wait_vmem_n<2 * k0>(); else wait_vmem_n<2 * k>();
  } else if (n == 1) {
    if (wave == 0) wait_vmem_n<k0>(); else wait_vmem_n<k>();
  } else {
    wait_vmem();
  }
}

// Per sequence of a batch, the workgroups (of one kv-head group) that hold its
// first and its last split: behind the states.
__device__ inline int* split_ends(const DecodeArgs& a) {
  return (int*)(a.ws + (size_t)a.n_slots * a.Hq * kStateFloats);
}

template <int RMODE, bool PAGED>
__global__ __launch_bounds__(kDecThreads, 1) void decode_split_kernel(DecodeArgs a, RampOf<RMODE == 2> f) {
  constexpr bool BIFOCAL = RMODE != 0;
  constexpr bool FREQ = RMODE == 2;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kDecSmem];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hw = wave & (kDecHeads - 1);  // head slot
  const int par = wave / kDecHeads;       // step parity
  const int i16 = lane & 15;
  const int g4 = lane >> 4;

  const int hgroup = blockIdx.x / a.n_wg;
  const int w = blockIdx.x - hgroup * a.n_wg;
  const uint32_t smem_base = lds_addr(smem);
  // ---- offset table: cos/sin of t * omega_i for t = 0..15 (table rows 0..15)
#pragma unroll
  for (int i = 0; i < kDecTile / kDecWaves; ++i) {
    const int r = wave + kDecWaves * i;
    if (lane < 32) dma16_s(a.table, (uint32_t)r * 512 + 16 * lane, smem_base + kDecOffTab + r * kDecTabRow);
  }
  SplitRange range = split_range(a, w);
  const int h0 = hgroup * kDecHeads;
  const int Hg = min(kDecHeads, a.Hkv - h0);  // heads in this group
  const int kvh = h0 + hw;
  const bool head_on = hw < Hg;
  const uint32_t row_bytes = (uint32_t)Hg * 256;
  const unsigned char* kbase = (const unsigned char*)(a.kc + (size_t)h0 * kHeadDim);
  const unsigned char* vbase = (const unsigned char*)(a.vc + (size_t)h0 * kHeadDim);
  const uint32_t kv_row_bytes = (uint32_t)a.Hkv * 256;
  int32_t* const pages_lds = (int32_t*)(smem + kDecOffPages);
  const unsigned char* const tab = smem + kDecOffTab;
  // query columns: col = (view, head) with view = col / 8
  const int col = i16;
  const int view = col >> 3;
  const int hj = col & 7;
  const bool col_on = head_on && hj < a.g && (BIFOCAL || view == 0);
  // distances q - k this column keeps: [keep_lo, keep_lo + keep_n) as one
  // unsigned compare; base view 0 .. w0 (every causal key for the vanilla
  // kernel), remote view w0 + 1 .. INT_MAX (Eq. (1)), none for unused columns
  const int keep_lo = BIFOCAL && view == 1 ? (int)min((uint32_t)a.w0 + 1u, (uint32_t)INT_MAX) : 0;
  const uint32_t keep_n = !col_on ? 0u
                          : !BIFOCAL ? 0x80000000u
                          : view == 0 ? (uint32_t)a.w0 + 1u
                                      : (uint32_t)INT_MAX - (uint32_t)a.w0;

  // ---- copies: a step's K image is 16 keys x Hg heads x 256 B = 4 Hg chunks
  // of 1 KB, V likewise; chunk n < 4 Hg is K, n < 8 Hg is V.  Wave w takes
  // chunks w + 8 i, i < 4; past 8 Hg it copies into a landing slot nobody
  // reads, so every wave has the same number of copies per step.  Lane ->
  // LDS slot 16 * lane of its chunk; it fetches the global chunk that slot
  // holds (keys past the chunk read the chunk's last key).
  // per copy i of this lane: the key row t it serves and the byte offset of its
  // chunk inside that key's slice of the cache (the same for every step)
  uint32_t cp_t[kDecCopies - 1], cp_off[kDecCopies - 1];
#pragma unroll
  for (int i = 0; i < kDecCopies - 1; ++i) {
    const int n = wave + kDecWaves * i;
    const bool is_v = n >= 4 * Hg;
    const bool real = n < 8 * Hg;
    const uint32_t o = (real ? (is_v ? n - 4 * Hg : n) : 0) * 1024 + 16 * lane;
    const uint32_t t = o / row_bytes;
    const uint32_t rem = o - t * row_bytes;
    const uint32_t h = rem >> 8, slot = (rem & 255) >> 4;
    cp_t[i] = t;
    cp_off[i] = h * 256 + 16 * (slot ^ (is_v ? 2 * (t & 7) : t));
  }
  uint32_t cp_full[kDecCopies - 1];  // byte offsets inside a step with 16 valid keys
#pragma unroll
  for (int i = 0; i < kDecCopies - 1; ++i) cp_full[i] = cp_t[i] * kv_row_bytes + cp_off[i];

  for (; range.left > 0 && range.b < a.B; ++range.b, range.off = 0) {
  const int b = range.b;
  // uniform and read-only for the kernel: a scalar load
  typedef __attribute__((address_space(4))) const int32_t const_i32;
  const int kv_len = clamp_len(((const const_i32*)a.kv_lens)[b], a.max_len);
  const int s_all = (kv_len + kDecTile - 1) / kDecTile;
  const int off = range.off;
  const int n_list = min(range.left, s_all + kDecSegCost - off);
  const uint32_t pos = range.pos;
  range.left -= n_list;
  range.pos += (uint32_t)(s_all + kDecSegCost);
  const int n_steps = min(off + n_list, s_all) - off;
  if (n_steps <= 0) continue;  // only empty steps of this sequence
  // this split: n_steps steps of sequence b from step0 on, `every` apart
  const bool seq_first = off == 0, seq_last = off + n_steps == s_all;
  int step0 = off, every = 1;
  if (a.B == 1) {
    step0 = w;
    every = range.n_wg;
  } else if (!seq_first && !seq_last && range.q != 0) {
    const int wf = range_of(range, pos), wl = range_of(range, pos + (uint32_t)s_all - 1);
    const uint32_t end_f = range.q * (wf + 1) + min((uint32_t)wf + 1, range.r);
    step0 = (int)(end_f - pos) + (w - wf - 1);
    every = wl - wf - 1;
  }
  const int c1 = kv_len;
  const int c0 = step0 * kDecTile;
  const int kstride = every * kDecTile;
  const int G = BIFOCAL ? group_size(kv_len, a.w_pre) : 1;
  const FastDiv gdiv = make_fastdiv((uint32_t)G);
  const int qpos = kv_len - 1;
  const int fq = BIFOCAL ? remote_pos(qpos, gdiv) : qpos;
  // the frequency map's omega'_i of this lane's frequency (wave 0 forms the
  // step rows, lane i taking frequency i)
  const double omf_lane = FREQ ? freq_map_omega(f, a.w_pre, kv_len, lane) : 0.0;
  const int n_iter = (n_steps + 1) / 2;

  // Byte offset of step jb's first key in its cache: a step's 16 keys are
  // consecutive rows (pages hold a multiple of 16 keys).  Dense caches: a
  // running offset.  Paged ones: the page index is read first (step_page) and
  // turned into an offset where the copies are issued (step_off), so the table
  // read overlaps the compute in between; page indices are clamped to the pool.
  size_t run_off = PAGED ? 0 : ((size_t)b * a.max_len + c0) * kv_row_bytes;
  const size_t run_inc = (size_t)kstride * kv_row_bytes;
  const bool pages_in_lds = PAGED && n_steps <= kDecPageCap;
  auto step_page = [&](int jb) __attribute__((always_inline)) {
    if (!PAGED) return 0;
    if (pages_in_lds) return (int)pages_lds[min(jb, n_steps - 1)];
    const int k0 = c0 + min(jb, n_steps - 1) * kstride;
    // the table is read-only for the kernel: read it through the constant
    // address space, so the load is a scalar one and its wait does not
    // drain the outstanding copies
    const const_i32* bt = (const const_i32*)a.block_table;
    return (int)bt[(size_t)b * a.max_pages + (k0 >> a.page_shift)];
  };
  auto step_off = [&](int jb, int pg) __attribute__((always_inline)) {
    if (!PAGED) {
      const size_t o = run_off;
      run_off += run_inc;
      return o;
    }
    const int k0 = c0 + jb * kstride;
    pg = min(max(__builtin_amdgcn_readfirstlane(pg), 0), a.n_pages - 1);
    return (((size_t)pg << a.page_shift) + (k0 & ((1 << a.page_shift) - 1))) * kv_row_bytes;
  };
  auto issue = [&](int jb, size_t off) __attribute__((always_inline)) {  // jb < n_steps, in order
    const int k0 = c0 + jb * kstride;
    const uint32_t buf = smem_base + (jb % kDecBufs) * kDecBufBytes;
    const unsigned char* kstep = kbase + off;
    const unsigned char* vstep = vbase + off;
    if (wave == 0) {
      // the cos/sin rows that rotate the query columns for this step: q - k0
      // (lanes 0..31) and f(q) - f(k0) (lanes 32..63) of the table, or the
      // step's row pair of the frequency map; one copy, by wave 0 alone (the
      // other waves wait for one copy fewer per step)
      const uint32_t dst = buf + 2 * kDecImgBytes;
      if (FREQ) {
        // the base row copied by lanes 0..31; the frequency map's row R'(q -
        // k0) formed here, lane i taking frequency i, and stored beside it
        if (lane < 32) dma16_s(a.table, (uint32_t)(qpos - k0) * 512 + 16 * lane, dst);
        const float2 cs = freq_map_cs(omf_lane, qpos - k0);
        *(float2*)(smem + (dst - smem_base) + 512 + 8 * lane) = cs;
      } else {
        const int fk0 = BIFOCAL ? remote_pos(k0, gdiv) : k0;
        const int row = lane < 32 ? qpos - k0 : fq - fk0;
        dma16_s(a.table, (uint32_t)row * 512 + 16 * (lane & 31), dst);
      }
    }
    // K and V are read exactly once per call: nontemporal.  A step whose 16
    // keys all lie below kv_len (every step but a sequence's last) takes the
    // precomputed offsets; the last one repeats its last key past kv_len.
    auto copy = [&](int i, uint32_t voff) __attribute__((always_inline)) {
      const int n = wave + kDecWaves * i;  // wave-uniform
      const bool is_v = n >= 4 * Hg;
      const bool real = n < 8 * Hg;
      const uint32_t dst = real ? buf + (is_v ? kDecImgBytes + (n - 4 * Hg) * 1024 : n * 1024)
                                : smem_base + kDecOffDummy;
      dma16_s_nt(is_v && real ? vstep : kstep, voff, dst);
    };
    if (k0 + kDecTile <= c1) {  // wave-uniform
#pragma unroll
      for (int i = 0; i < kDecCopies - 1; ++i) copy(i, cp_full[i]);
    } else {
#pragma unroll
      for (int i = 0; i < kDecCopies - 1; ++i)
        copy(i, (uint32_t)(min(k0 + (int)cp_t[i], c1 - 1) - k0) * kv_row_bytes + cp_off[i]);
    }
  };

  // ---- the raw query rows of the group's heads (contiguous, at most 8 KB),
  // beside the first steps' copies: into LDS where the frequency map's table
  // would lie, or straight into registers with that map
  // the raw query slices in fp32, scaled once (log2(e) / sqrt(d)): every
  // step rotates them by its own offset without unpacking or scaling again
  float qf[4][8];
  auto load_q = [&](const uint16_t* qrow) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      unpack8(load16(qrow + 32 * s + 8 * g4), qf[s]);
#pragma unroll
      for (int i = 0; i < 8; ++i) qf[s][i] *= a.q_scale;
    }
  };
  const int q_row = min(hw, Hg - 1) * a.g + min(hj, a.g - 1);  // row of the group's query heads
  const uint16_t* qgroup = a.q + ((size_t)b * a.Hq + h0 * a.g) * kHeadDim;
  if (FREQ) {
    for (int i = threadIdx.x; i < kDecTile * 32; i += kDecThreads) {
      const int r = i >> 5, s = i & 31;
      // the frequency map's rows t omega'_i, t = 0..15
      const float2 cs0 = freq_map_cs(freq_map_omega(f, a.w_pre, kv_len, 2 * s), r),
                   cs1 = freq_map_cs(freq_map_omega(f, a.w_pre, kv_len, 2 * s + 1), r);
      *(float4*)(smem + kDecOffTab2 + r * kDecTabRow + 16 * s) =
          make_float4(cs0.x, cs0.y, cs1.x, cs1.y);
    }
    load_q(qgroup + (size_t)q_row * kHeadDim);
  } else {
    const uint32_t off = 1024 * wave + 16 * lane;
    if (off < (uint32_t)(Hg * a.g) * 256)
      dma16_s(qgroup, off, smem_base + kDecOffTab2 + 1024 * wave);
  }

  // paged caches: the page index of every step of this split, into LDS
  if (pages_in_lds) {
    for (int j = threadIdx.x; j < n_steps; j += kDecThreads) {
      const int k0 = c0 + j * kstride;
      pages_lds[j] = a.block_table[(size_t)b * a.max_pages + (k0 >> a.page_shift)];
    }
    __syncthreads();
  }

  // the plain loads above complete before the first copy is requested, so the
  // compiler's waits for them never hold back the copies
  if (FREQ) wait_vmem();
  const int n_first = min(n_steps, 4);
  for (int jb = 0; jb < n_first; ++jb) issue(jb, step_off(jb, step_page(jb)));
  if (!FREQ) {
    // the query rows are older than the steps' copies
    wait_steps(wave, n_first);
    __syncthreads();
    load_q((const uint16_t*)(smem + kDecOffTab2) + (size_t)q_row * kHeadDim);
  }

  f32x4 acc_o[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc_o[i] = f32x4{};
  float m_run = -INFINITY, l_run = 0.f;

  // scalar loads still in flight would make the compiler drain every LDS read
  // of the loop (they share a counter and complete out of order)
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  for (int it = 0; it < n_iter; ++it) {
    // cache rows of the steps copied at the end of this iteration, looked up
    // now so the block-table reads are long done by then
    const int page4 = step_page(2 * it + 4), page5 = step_page(2 * it + 5);
    // this wave's copies of steps 2it, 2it+1 (the next pair may fly)
    if (2 * it + 3 < n_steps) {
      if (wave == 0)
        wait_vmem_n<2 * kDecCopies>();
      else
        wait_vmem_n<2 * (kDecCopies - 1)>();
    } else {  // the last iterations: fewer steps in flight
      wait_steps(wave, max(n_steps - (2 * it + 2), 0));
    }
    __syncthreads();  // everyone's copies (and the offset table)
    const int j = 2 * it + par;
    if (head_on && j < n_steps) {
      const int k0 = c0 + j * kstride;
      const unsigned char* sb = smem + (j % kDecBufs) * kDecBufBytes;
      const unsigned char* kb = sb + hw * 256;
      const unsigned char* vb = kb + kDecImgBytes;
      const int fk0 = BIFOCAL ? remote_pos(k0, gdiv) : k0;

      // query operand rotated by q - k0 (base columns) or f(q) - f(k0) (remote)
      bf16x8 qop[4];
      {
        const float4* c4 = (const float4*)(sb + 2 * kDecImgBytes + 512 * view);
#pragma unroll
        for (int s = 0; s < 2; ++s)
          rotate8f(qf[s], qf[s + 2], c4 + 16 * s + 4 * g4, qop[s], qop[s + 2]);
        if (!col_on) {
#pragma unroll
          for (int s = 0; s < 4; ++s) qop[s] = bf16x8{};
        }
      }

      // key t = i16 of this lane, rotated once, by its view's offset
      const int key = k0 + i16;
      // remote keys: offset f(k) - f(k0) in the base rows (Eq. (3)), or t in
      // the frequency map's rows
      int r = i16;
      if (BIFOCAL && qpos - key > a.w0)
        r = FREQ ? i16 + (kDecOffTab2 - kDecOffTab) / kDecTabRow : remote_pos(key, gdiv) - fk0;
      f32x4 sc = f32x4{};
      {
        u32x4 kr[4];
#pragma unroll
        for (int s = 0; s < 4; ++s)
          kr[s] = *(const u32x4*)(kb + i16 * row_bytes + 16 * ((4 * s + g4) ^ i16));
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          float4 cs[4];
#pragma unroll
          for (int u = 0; u < 4; ++u)
            cs[u] = *(const float4*)(tab + r * kDecTabRow + 16 * (16 * s + 4 * g4 + u));
          bf16x8 lo, hi;
          rotate8(kr[s], kr[s + 2], cs, 1.f, lo, hi);
          sc = mfma16(lo, qop[s], sc);
          sc = mfma16(hi, qop[s + 2], sc);
        }
      }

      // the values of the PV product, requested before the softmax needs time;
      // a transposing read gives lane i of group g4 the keys 4 g4 .. 4 g4 + 3
      // at d = 16 db + i
      i16x4 vr[8];
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        const int c = 2 * db + ((i16 & 3) >> 1);
        const int ta = 4 * g4 + (i16 >> 2);
        vr[db] = lds_read_tr4(vb + ta * row_bytes + 16 * (c ^ (2 * (ta & 7))) + 8 * (i16 & 1));
      }
      __builtin_amdgcn_sched_barrier(0);

      // each column keeps only the keys of its own view (q - k in [lo, lo +
      // keep)); lane holds keys 4 g4 + i
      float sv[4];
      const uint32_t dbase = (uint32_t)(qpos - k0 - 4 * g4) - (uint32_t)keep_lo;
#pragma unroll
      for (int i = 0; i < 4; ++i) sv[i] = dbase - (uint32_t)i < keep_n ? sc[i] : -INFINITY;

      // online softmax per column (the 4 lanes i16, i16+16, i16+32, i16+48)
      float mt = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
      mt = max_xor16_32(mt);
      const float m_new = fmaxf(m_run, mt);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      // 1 unless the maximum moved (a column with no key of its view yet
      // keeps m = -inf and must not take the rescale branch every step)
      const float alpha = m_new == m_run ? 1.f : fast_exp2(m_run - m_use);
      f32x4 p;
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = fast_exp2(sv[i] - m_use);
      l_run = l_run * alpha + (p[0] + p[1]) + (p[2] + p[3]);
      m_run = m_new;
      if (__ballot(alpha != 1.f) != 0) {  // most steps leave every column's maximum alone
#pragma unroll
        for (int db = 0; db < 8; ++db) acc_o[db] *= alpha;
      }
      // P^T operand of the k = 16 product: k index 4 g4 + i is key 4 g4 + i
      const bf16x4 pb = __builtin_convertvector(p, bf16x4);

      // O^T += V^T P^T
#pragma unroll
      for (int db = 0; db < 8; ++db)
        acc_o[db] = mfma16k16(__builtin_bit_cast(bf16x4, vr[db]), pb, acc_o[db]);
    }
    __syncthreads();  // steps 2it, 2it+1 consumed: their buffers take steps 2it+4, 2it+5
    if (2 * it + 4 < n_steps) issue(2 * it + 4, step_off(2 * it + 4, page4));
    if (2 * it + 5 < n_steps) issue(2 * it + 5, step_off(2 * it + 5, page5));
  }

  // ---- merge the odd-step wave's state into the even-step wave's (max-shifted)
  {
    float* xs = (float*)smem + ((size_t)hw * 64 + lane) * 34;
    if (par == 1) {
      xs[0] = m_run;
      xs[1] = l_run;
#pragma unroll
      for (int db = 0; db < 8; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) xs[2 + 4 * db + i] = acc_o[db][i];
    }
    __syncthreads();
    if (par == 0) {
      const float m_b = xs[0];
      const float M = fmaxf(m_run, m_b);
      const float wa = M == -INFINITY ? 0.f : fast_exp2(m_run - M);
      const float wb = M == -INFINITY ? 0.f : fast_exp2(m_b - M);
      l_run = wa * l_run + wb * xs[1];
#pragma unroll
      for (int db = 0; db < 8; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc_o[db][i] = wa * acc_o[db][i] + wb * xs[2 + 4 * db + i];
      m_run = M;
    }
  }

  // ---- one state per head: Eq. (7) over the local-window state (column hj)
  // and the remote-only state (column 8 + hj); the exclusion window is empty
  // because band keys never enter the remote view
  if (par == 0 && head_on) {
    float l_tot = l_run + __shfl_xor(l_run, 16);
    l_tot += __shfl_xor(l_tot, 32);
    float m_own = m_run, l_own = l_tot;
    float W_own = 1.f, W_oth = 0.f;
    float m_oth = -INFINITY, l_oth = 0.f;
    if (BIFOCAL) {
      m_oth = __shfl_xor(m_run, 8);
      l_oth = __shfl_xor(l_tot, 8);
      const float M = fmaxf(m_own, m_oth);
      W_own = M == -INFINITY ? 0.f : fast_exp2(m_own - M);
      W_oth = M == -INFINITY ? 0.f : fast_exp2(m_oth - M);
      m_own = M;
    }
    float* out = a.ws + ((size_t)(w + b) * a.Hq + kvh * a.g + hj) * kStateFloats;
    const bool writer = view == 0 && hj < a.g;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      f32x4 o4 = acc_o[db] * W_own;
      if (BIFOCAL) {
#pragma unroll
        for (int i = 0; i < 4; ++i) o4[i] += W_oth * __shfl_xor(acc_o[db][i], 8);
      }
      if (writer) *(f32x4*)(out + 4 + 16 * db + 4 * g4) = o4;
    }
    // the state's third word carries the split count of a single sequence, so
    // the reduce need not recompute it (slot 0 is written by every call)
    if (writer && g4 == 0)
      *(f32x4*)out = f32x4{m_own, W_own * l_own + W_oth * l_oth, __int_as_float(range.n_wg), 0.f};
  }
  // a batch's sequences: their first and last slots' workgroups, for the reduce
  if (a.B > 1 && hgroup == 0 && threadIdx.x == 0) {
    if (seq_first) split_ends(a)[2 * b] = w;
    if (seq_last) split_ends(a)[2 * b + 1] = w;
  }
  __syncthreads();  // the merged states are read: the next split may fill the buffers
  }
  // a workgroup without a split leaves its offset rows' copies to land while it
  // still holds the LDS they go to
  wait_vmem();
}

// Final merge over the splits of one head (Eq. (7) weights exp2(m - M)):
// O = sum W O~ / sum W l.
//
// One sequence: its splits are many (a slot per workgroup) and its first slot
// is known, so every slot is read at once.  Workgroup (head, quarter of the
// 128 channels): 32 groups of 8 threads; group grp takes splits grp, grp + 32,
// ..., thread c of a group owns channels 32 quarter + 4c .. +3; partial sums
// meet in LDS.
constexpr int kRedGroups = 32;
constexpr int kRedMaxPer = 8;
template <int PER>  // splits per group: at most kRedGroups * PER splits
__global__ __launch_bounds__(256) void decode_reduce_kernel(DecodeArgs a, uint16_t* o) {
  __shared__ float sMax[kRedGroups];
  __shared__ __attribute__((aligned(16))) float sAcc[kRedGroups][32];
  __shared__ float sDen[kRedGroups];
  const int h = blockIdx.x;
  const int quarter = blockIdx.y;
  const int tid = threadIdx.x;
  const float* base = a.ws + (size_t)h * kStateFloats;
  const size_t stride = (size_t)a.Hq * kStateFloats;
  const int c = tid & 7;
  const int grp = tid >> 3;

  // every slot is read at once, slot 0's state carrying the sequence's split
  // count; the slots past it hold stale states and are dropped below
  float m[PER], l[PER];
  f32x4 ov[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    // no branch: all loads are issued together (slots past the last read the
    // last slot again and are dropped with the rest)
    const float* stt = base + (size_t)min(grp + kRedGroups * i, a.n_slots - 1) * stride;
    const float2 ml = *(const float2*)stt;
    m[i] = ml.x;
    l[i] = ml.y;
    ov[i] = *(const f32x4*)(stt + 4 + 32 * quarter + 4 * c);
  }
  const int ns = __float_as_int(base[2]);  // splits with keys, from slot 0's state
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (grp + kRedGroups * i >= ns) {
      m[i] = -INFINITY;
      l[i] = 0.f;
      ov[i] = f32x4{};
    }
  }
  float M = -INFINITY;
#pragma unroll
  for (int i = 0; i < PER; ++i) M = fmaxf(M, m[i]);
  if (c == 0) sMax[grp] = M;
  __syncthreads();
#pragma unroll
  for (int g2 = 0; g2 < kRedGroups; ++g2) M = fmaxf(M, sMax[g2]);

  f32x4 acc = f32x4{};
  float den = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const float w = m[i] == -INFINITY ? 0.f : fast_exp2(m[i] - M);
    den += w * l[i];
    acc += w * ov[i];
  }
  *(f32x4*)&sAcc[grp][4 * c] = acc;
  if (c == 0) sDen[grp] = den;
  __syncthreads();
  if (tid < 32) {
    float num = 0.f, dsum = 0.f;
#pragma unroll
    for (int g2 = 0; g2 < kRedGroups; ++g2) {
      num += sAcc[g2][tid];
      dsum += sDen[g2];
    }
    const __bf16 r = (__bf16)(num / dsum);
    o[(size_t)h * kHeadDim + 32 * quarter + tid] = __builtin_bit_cast(uint16_t, r);
  }
}

// A batch: a sequence has about n_wg / B splits, from a first slot that the
// split kernel wrote, so only those are read (reading every slot a sequence
// could have moved 69 MB and took 20.8 us at 32 sequences of 32 heads).
// Workgroup = head: 16 groups of 16 threads; group grp takes splits grp,
// grp + 16, ..., thread c of a group owns channels 8c .. 8c+7.
constexpr int kRedBatchGroups = 16;
__global__ __launch_bounds__(256) void decode_reduce_batch_kernel(DecodeArgs a, uint16_t* o) {
  __shared__ float sM[kRedBatchGroups], sL[kRedBatchGroups];
  __shared__ __attribute__((aligned(16))) float sO[kRedBatchGroups][kHeadDim];
  const int b = blockIdx.x / a.Hq;
  const int h = blockIdx.x - b * a.Hq;
  const int tid = threadIdx.x;
  const int c = tid & 15, grp = tid >> 4;
  const int* ends = split_ends(a) + 2 * b;
  const int first = min(max(ends[0], 0), a.n_wg - 1);
  const int ns = min(max(ends[1], first), a.n_wg - 1) - first + 1;
  const float* base = a.ws + ((size_t)(first + b) * a.Hq + h) * kStateFloats;
  const size_t stride = (size_t)a.Hq * kStateFloats;

  float M = -INFINITY, den = 0.f;
  f32x4 acc0 = f32x4{}, acc1 = f32x4{};
  for (int s = grp; s < ns; s += kRedBatchGroups) {
    const float* stt = base + (size_t)s * stride;
    const float2 ml = *(const float2*)stt;
    const f32x4 o0 = *(const f32x4*)(stt + 4 + 8 * c), o1 = *(const f32x4*)(stt + 8 + 8 * c);
    const float m = fmaxf(M, ml.x);
    const float wa = M == -INFINITY ? 0.f : fast_exp2(M - m);
    const float wb = ml.x == -INFINITY ? 0.f : fast_exp2(ml.x - m);
    den = wa * den + wb * ml.y;
    acc0 = wa * acc0 + wb * o0;
    acc1 = wa * acc1 + wb * o1;
    M = m;
  }
  if (c == 0) {
    sM[grp] = M;
    sL[grp] = den;
  }
  *(f32x4*)&sO[grp][8 * c] = acc0;
  *(f32x4*)&sO[grp][8 * c + 4] = acc1;
  __syncthreads();
  if (tid < kHeadDim) {
    const int n = min(ns, kRedBatchGroups);  // groups past the splits hold nothing
    float mx = -INFINITY;
    for (int g2 = 0; g2 < n; ++g2) mx = fmaxf(mx, sM[g2]);
    float num = 0.f, dsum = 0.f;
    for (int g2 = 0; g2 < n; ++g2) {
      const float w = sM[g2] == -INFINITY ? 0.f : fast_exp2(sM[g2] - mx);
      num += w * sO[g2][tid];
      dsum += w * sL[g2];
    }
    const __bf16 r = (__bf16)(num / dsum);
    o[(size_t)blockIdx.x * kHeadDim + tid] = __builtin_bit_cast(uint16_t, r);
  }
}

// ---------------------------------------------------------------- launcher
int cu_count() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n < 1)
      n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// Workgroups per kv-head group: about one per CU in all (each holds 157 KB of
// LDS), never more than one sequence's steps.  Slots: one per (workgroup,
// sequence) pair of the list (SplitRange), w + b < n_wg + B.
constexpr int kDecMaxWg = 256;  // CUs of the GPU: workspaces are sized for as many
static_assert(kDecMaxWg <= kRedGroups * kRedMaxPer, "the reduce reads every slot of one sequence");
static void decode_geometry(int n_cu, int B, int Hkv, int max_len, int* n_wg, int* n_slots) {
  const int hg = (Hkv + kDecHeads - 1) / kDecHeads;
  const long long steps = ((long long)max_len + kDecTile - 1) / kDecTile;
  long long n = n_cu / hg;
  if (B == 1 && n > steps) n = steps;
  if (n < 1) n = 1;
  *n_wg = (int)n;
  *n_slots = (int)(n + B - 1);
}

// Bytes of the states and, for a batch, the ends of its sequences
static size_t slot_bytes(long long n_slots, int B, int Hq) {
  return (size_t)n_slots * Hq * kStateFloats * sizeof(float) + (B > 1 ? 2 * (size_t)B * sizeof(int) : 0);
}

// The slots per head that a workspace holds at least: fewer than
// decode_geometry's for few sequences of few keys, for up to 4 kv heads and
// beyond 64 sequences.  A call with less than decode_workspace_bytes takes
// fewer workgroups or several launches (fit_workspace).
static long long state_slots(int B, int Hkv, int max_len) {
  const long long groups = (long long)B * ((Hkv + kDecHeads - 1) / kDecHeads);
  const long long steps = ((long long)max_len + kDecTile - 1) / kDecTile;
  long long n = B <= 64 ? 128 : (256 + groups - 1) / groups;
  if (n > 128) n = 128;
  if (n > steps) n = steps;
  return n * B;
}

size_t decode_state_bytes(int B, int Hq, int Hkv, int max_len) {
  return (size_t)state_slots(B, Hkv, max_len) * Hq * kStateFloats * sizeof(float);
}

size_t decode_workspace_bytes(int B, int Hq, int Hkv, int max_len) {
  int n_wg, n_slots;
  decode_geometry(kDecMaxWg, B, Hkv, max_len, &n_wg, &n_slots);
  return std::max(slot_bytes(n_slots, B, Hq), decode_state_bytes(B, Hq, Hkv, max_len));
}

// What fits a workspace of at least decode_state_bytes: the sequences per
// launch (a call takes ceil(B / n_seq) of them, one after another in the same
// workspace), workgroups and slots.  The fewest launches that leave at least
// half of the workgroups; one sequence a launch fits always (state_slots is B
// at least, and its one slot is all a single workgroup needs).
struct DecodeFit {
  int n_seq, n_wg, n_slots;
};
static DecodeFit fit_workspace(int n_cu, int B, int Hq, int Hkv, int max_len, size_t ws_bytes) {
  DecodeFit f;
  for (int launches = 1;; ++launches) {
    f.n_seq = (B + launches - 1) / launches;
    decode_geometry(n_cu, f.n_seq, Hkv, max_len, &f.n_wg, &f.n_slots);
    if (slot_bytes(f.n_slots, f.n_seq, Hq) <= ws_bytes) return f;
    const size_t ends = slot_bytes(0, f.n_seq, Hq);
    const long long slots =
        ws_bytes > ends ? (long long)((ws_bytes - ends) / slot_bytes(1, 1, Hq)) : 0;
    const long long n = slots - (f.n_seq - 1);
    if (2 * n >= f.n_wg || f.n_seq == 1) {
      f.n_wg = (int)std::max(1LL, n);
      f.n_slots = f.n_wg + f.n_seq - 1;
      return f;
    }
  }
}

size_t decode_map_workspace_bytes(int B, int Hq, int Hkv, int max_len, bool /*freq*/) {
  return decode_workspace_bytes(B, Hq, Hkv, max_len);
}

// block_table == nullptr: dense caches [B][max_len][Hkv][128]; otherwise
// pools [n_pages][1 << page_shift][Hkv][128] and max_len = max_pages << page_shift.
hipError_t launch_decode(bool bifocal, const uint16_t* q, const uint16_t* kc, const uint16_t* vc,
                         const int32_t* kv_lens, int max_len, uint16_t* o, const float2* table,
                         int B, int Hq, int Hkv, int w_pre, int w0, float* ws,
                         hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1,
                         const int32_t* block_table, int max_pages, int n_pages, int page_shift,
                         const double* freq_og, size_t ws_bytes) {
  // freq_og: nullptr for the Eq. (3) map, else the frequency map's omega_i
  // (64) and ramp gamma_i (64).  ws holds the states of n_slots splits and,
  // for a batch, behind them two ints per sequence (split_ends).
  const DecodeFit fit =
      fit_workspace(std::min(cu_count(), kDecMaxWg), B, Hq, Hkv, max_len, ws_bytes);
  if (fit.n_seq < B) {
    const size_t row = (size_t)Hq * kHeadDim;
    const size_t cache = block_table != nullptr ? 0 : (size_t)max_len * Hkv * kHeadDim;
    for (int b = 0; b < B; b += fit.n_seq) {
      const int n = std::min(fit.n_seq, B - b);
      const hipError_t e = launch_decode(
          bifocal, q + b * row, kc + b * cache, vc + b * cache, kv_lens + b, max_len, o + b * row,
          table, n, Hq, Hkv, w_pre, w0, ws, stream, b == 0 ? ev0 : nullptr,
          b + n == B ? ev1 : nullptr,
          block_table != nullptr ? block_table + (size_t)b * max_pages : nullptr, max_pages,
          n_pages, page_shift, freq_og, ws_bytes);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  DecodeArgs a = {};
  a.q = q;
  a.kc = kc;
  a.vc = vc;
  a.kv_lens = kv_lens;
  a.ws = ws;
  a.table = table;
  a.B = B;
  a.Hq = Hq;
  a.Hkv = Hkv;
  a.g = Hq / Hkv;
  a.max_len = max_len;
  a.block_table = block_table;
  a.max_pages = max_pages;
  a.n_pages = n_pages;
  a.page_shift = page_shift;
  a.n_hgroups = (Hkv + kDecHeads - 1) / kDecHeads;
  a.n_wg = fit.n_wg;
  a.n_slots = fit.n_slots;
  a.w_pre = w_pre;
  a.w0 = w0;
  a.q_scale = 1.4426950408889634f / sqrtf((float)kHeadDim);
  const long long nwg = (long long)a.n_wg * a.n_hgroups;
  if (nwg > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  hipError_t e = hipSuccess;
  const bool freq = bifocal && freq_og != nullptr;
  FreqRamp ramp;
  if (freq) {
    for (int i = 0; i < kHalf; ++i) {
      ramp.omega[i] = freq_og[i];
      ramp.gamma[i] = freq_og[kHalf + i];
    }
  }
  // ev0 / ev1 (optional) are recorded on the stream around the split kernel
  if (ev0 != nullptr && (e = hipEventRecord(ev0, stream)) != hipSuccess) return e;
  const dim3 grid((unsigned)nwg), block(kDecThreads);
  const bool paged = block_table != nullptr;
  if (freq && paged)
    hipLaunchKernelGGL((decode_split_kernel<2, true>), grid, block, 0, stream, a, ramp);
  else if (freq)
    hipLaunchKernelGGL((decode_split_kernel<2, false>), grid, block, 0, stream, a, ramp);
  else if (bifocal && paged)
    hipLaunchKernelGGL((decode_split_kernel<1, true>), grid, block, 0, stream, a, NoRamp{});
  else if (bifocal)
    hipLaunchKernelGGL((decode_split_kernel<1, false>), grid, block, 0, stream, a, NoRamp{});
  else if (paged)
    hipLaunchKernelGGL((decode_split_kernel<0, true>), grid, block, 0, stream, a, NoRamp{});
  else
    hipLaunchKernelGGL((decode_split_kernel<0, false>), grid, block, 0, stream, a, NoRamp{});
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (ev1 != nullptr && (e = hipEventRecord(ev1, stream)) != hipSuccess) return e;
  if (B > 1)
    hipLaunchKernelGGL(decode_reduce_batch_kernel, dim3((unsigned)B * Hq), dim3(256), 0, stream, a,
                       o);
  else if (a.n_wg <= 4 * kRedGroups)
    hipLaunchKernelGGL(decode_reduce_kernel<4>, dim3(Hq, 4), dim3(256), 0, stream, a, o);
  else
    hipLaunchKernelGGL(decode_reduce_kernel<kRedMaxPer>, dim3(Hq, 4), dim3(256), 0, stream, a, o);
  return hipGetLastError();
}

// ------------------------------------- fixed device scratch (no allocation)
// For callers that cannot allocate device memory (code under graph capture,
// tight serving loops): one file-scope array per device holds the fp32
// cos/sin table of positions [0, kNoAllocMaxLen) and the split states.  The
// array lives as long as the process.  Calls on one device share it, and each
// keeps the last call's contents (the table stays, the states are rewritten
// in full by every call), so calls that overlap on one device race.
constexpr int kNoAllocMaxLen = 1 << 17;
constexpr size_t kNoAllocTableBytes = (size_t)kNoAllocMaxLen * kHalf * sizeof(float2);  // 64 MiB
// A call is accepted by its count of split states per sequence
// (decode_state_bytes); the slots that a batch needs beyond that count
// (decode_workspace_bytes) are at most n_wg per query head, i.e. 256 x 32
// heads of 528 bytes, and the ends of its sequences.
constexpr size_t kNoAllocStateBytes = (size_t)24 << 20;
constexpr size_t kNoAllocSlackBytes = (size_t)5 << 20;
static __device__ __align__(256) unsigned char
    scratch[kNoAllocTableBytes + kNoAllocStateBytes + kNoAllocSlackBytes];

hipError_t launch_build_table(float2* table, uint32_t* table16, int n_pos, const double* omega,
                              hipStream_t stream);

int noalloc_decode_max_len() { return kNoAllocMaxLen; }
size_t noalloc_decode_state_bytes() { return kNoAllocStateBytes; }
size_t noalloc_decode_slot_bytes() { return kNoAllocStateBytes + kNoAllocSlackBytes; }

namespace {
struct NoAllocDevice {
  unsigned char* ptr = nullptr;  // this device's copy of `scratch`
  double theta = 0.0;            // rope_theta of the table it holds (0: none yet)
};
std::mutex g_noalloc_mu;
NoAllocDevice g_noalloc[64];
}  // namespace

// The current device's table and state regions.  The first call on a device
// looks the array's address up (with that device current); the first call
// for a new theta builds the table from omega and waits for it, so that a
// call on any stream may read it afterwards.
hipError_t noalloc_decode_buffers(double theta, const double* omega, hipStream_t stream,
                                  const float2** table, float** states) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  NoAllocDevice& d = g_noalloc[dev];
  if (d.ptr == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    d.ptr = (unsigned char*)p;
  }
  if (d.theta != theta) {
    d.theta = 0.0;
    e = launch_build_table((float2*)d.ptr, nullptr, kNoAllocMaxLen, omega, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return e;
    d.theta = theta;
  }
  *table = (const float2*)d.ptr;
  *states = (float*)(d.ptr + kNoAllocTableBytes);
  return hipSuccess;
}

}  // namespace jl
