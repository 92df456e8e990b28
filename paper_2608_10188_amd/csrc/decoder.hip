// Device decoder of the AXP1 absolute-offset LZ77 block format for gfx950.
//
// Three kernels per window of blocks (the paper's ANS / parse / copy split,
// Table 2):
//   k_ans    one wave64 per (block, stream): order-0 rANS of the literal,
//            length, offset and command streams with the slot table in LDS;
//            renormalisation words are handed to the lanes that need them by
//            ballot + prefix count over a register window of the word stream.
//   k_parse  one workgroup per block: commands are parsed 256 to 1024 at a time by
//            block-wide prefix scans (positions, literal positions, value
//            indices; DPP moves inside the wave) and an associative scan of
//            the four-entry distance history (each command is a map on
//            history tuples); literal runs leave as whole 16-byte groups of
//            the output, zeros where matches will be; matches become tokens
//            (src, dst, len).
//   match layer: every token (src, dst, len) is a periodic fill
//            out[dst+k] = out[src + k mod dist] (periodic-fill section).  Two
//            schedules:
//   - roots (the default): no token waits for another.  k_roots follows each
//     piece of a match's source to the literal bytes it comes from, which are
//     final after the parse; the bytes of long chains, and every byte of
//     archives taken to be deep (k_mark), become entries of a jump array that
//     k_sweep and k_finish resolve.
//   - rounds (once one of their knobs is set, and for the serial ablation):
//     the tokens whose destinations meet a token's source bytes form one
//     contiguous index range (tokens are stored in output order), found once
//     by binary search; a token is ready when those are done.  k_round0 (a
//     workgroup per block, fills gathered in an LDS tile of the block's chunks
//     that receive match bytes) and k_round run level-synchronous rounds (the
//     dependency levels of the paper's wavefront decoder) with plain cached
//     accesses, the kernel boundary being the only synchronisation.  The last
//     round's leftovers are finished by pointer jumping over window positions
//     (k_jmarklong ... k_jgather), or marked in a bitmap that k_pcount /
//     k_pscatter compact into an ascending list for k_tail, one persistent
//     launch whose waves take 64-token chunks from a ticket counter and publish
//     through agent-coherent stores.
//
// Times that a comment sets against each other are whole decodes unless it says
// otherwise, of two builds in one session on the code of their day; what else
// changed since moves both sides.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "aceapex.h"
#include "ax_common.h"
#include "engine.h"

namespace {

// Device pointers that kernels load from memory (job tables) or select at run
// time lose their address space; accesses through generic pointers become
// flat instructions, which also count against the LDS wait counter.  Kernels
// convert them to global pointers explicitly.
#define AX_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ inline AX_GLOBAL T* gp(T* p) {
  return (AX_GLOBAL T*)p;
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_u __attribute__((aligned(1)));  // 16 bytes at any byte address (one dwordx4 load)
typedef u32x4 u32x4_w __attribute__((aligned(4)));  // four words at any word address
typedef uint32_t u32_u __attribute__((aligned(1)));
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kMaxB = 16384;           // largest block the device path decodes
constexpr uint32_t kParseThreads = 256;
// Windows of few blocks parse them with more threads, so in fewer chunks: a
// chunk is a chain of block-wide steps whose latency hardly grows with it.
// Whole decodes with 256, 512 and 1024 threads, in us: 4 blocks of DNA 75, 65,
// 62; 192 of text 83, 78, 76; 256 of DNA 102, 89, 86; 384 of text 100, 94, 97;
// 512 of DNA 116, 106, 110; 768 of DNA 150, 137, 151, of text 140, 136, 148;
// 1024 of DNA 153, 142, 166 but of text 165, 168, 181, of reads 173, 180, 192 and
// of 4 KiB blocks 65, 69, 85; 2048 of reads 224, 233, 264; 15500 of DNA 685,
// 732, 1043.  Of 4 KiB blocks (about a hundred commands of DNA) 64, 256 of DNA 57,
// 55, 49 and 60, 59, 52, of text 64, 62, 60; with 256 and 512 threads 512 of DNA
// 65, 62, 768 of DNA 71, 71, of text 78, 83.  A compute unit each is the line for
// 1024, three blocks for 512.
constexpr uint32_t kParseWide = 1024, kParseMid = 512;
constexpr uint32_t kParseWideBlocks = 256, kParseMidBlocks = 768;
constexpr uint32_t kOffStage = 3072;        // offset-stream bytes staged in LDS by k_parse
constexpr uint32_t kLenStage = 256;         // length-stream bytes staged in LDS by k_parse
constexpr uint32_t kLenBpt = 1, kOffBpt = 2;  // LEB bytes per thread per pass: length / offset streams
constexpr uint32_t kCopyThreads = 256;      // match-layer workgroup
constexpr uint8_t kPending = 0xFF;          // done[] value of a token not yet copied
constexpr uint32_t kSub = 64;               // pending-list sublists (one counter each, 256 B apart)
constexpr uint32_t kCounterStride = 64;     // u32 between two sublist counters
constexpr uint32_t kMaxRoundGrid = 4096;    // workgroups of a round launch
// Counters of the match bytes of a window's open blocks (one takes 6 ns an
// addition: 4096 blocks' parse 34, with it 59 us).
constexpr uint32_t kCopiedShards = 8;
// A block counts if one byte in so many is copied, repeats of its own bytes not
// counted: a walk through such a repeat ends at once, and the tile repeats the
// rest.  Blocks that repeat their first byte, 64 MiB / 1 GiB, marked 369 / 5550 us,
// walked 253 / 2810.
constexpr uint32_t kOwnShare = 32;
// last round: list the leftovers (persistent launch) or mark them for
// pointer jumping (first entries and leftover-map bits)
constexpr int kMarkList = 1, kMarkJump = 2;

struct DevStatus {
  int32_t err;
  uint32_t pad0;
  unsigned long long bad_block;
  uint32_t ticket;
  uint32_t long_count;
  uint32_t n_pending;  // tokens the bulk rounds left (the deep remainder); roots: whether a sweep has work
  uint32_t pad2;
  uint32_t jump_used;    // jump passes that found active entries (0: all of them did)
  uint32_t n_jwords;     // leftover-map words with bits set (the jump kernels' work list)
  uint32_t pend0;        // tokens round 0 left to the later rounds (reported when asked)
  uint32_t marked;       // roots, windows with open blocks: the first blocks that k_settle marks
  uint32_t pad1[52];
};
static_assert(sizeof(DevStatus) == 256, "status block is 256 bytes");

// One archive of a plan (a whole-archive decode, one archive of a batch, or
// the source closure of a range): where it is, and where its bytes go.
struct JobDev {
  const uint8_t* arc;   // device archive
  uint8_t* out;         // decoded bytes: at the archive's absolute positions, or by slot (below)
  uint64_t payload_at;  // header + index bytes
  uint64_t n_bytes, nb;
  uint32_t B, mm;
  // a range decode's compact scratch: block b's bytes at out + slot[b] * B;
  // a slot of `junk` or more means the junk block (blocks the plan does not
  // decode; only bytes nobody needs are read from it).  null: absolute.
  uint32_t* slot;
  uint32_t junk;
};

// One block of a window.  A window holds the blocks of its jobs job by job
// (in the plan's window order of jobs), ascending within a job, and the
// window's tokens are stored block after block in that order.
struct WinBlock {
  uint64_t b;       // block index in its archive
  uint32_t job;
  uint32_t tok;     // window index of the block's first token
  uint32_t first;   // window index of this job's first block in the window
  uint32_t count;   // blocks of this job in the window
};

// Where the bytes of archive position p of a job's output live.  OutDirect:
// the output holds the archive at its absolute positions (whole-archive and
// batch decodes).  OutMapped: a range decode's compact scratch, the bytes of
// block b at slot[b] * B (the slot table is set for the blocks the plan
// decodes; any other block maps to the junk block, whatever its entry holds,
// so a stale entry can never send an access outside the scratch).  Copy
// kernels are instantiated for each; the whole-archive path compiles to the
// plain pointer arithmetic.
typedef AX_GLOBAL uint8_t* gbytes;
struct OutDirect {
  gbytes base;
  __device__ explicit OutDirect(const JobDev& j) : base(gp(j.out)) {}
  __device__ OutDirect with_base(gbytes b) const { OutDirect o = *this; o.base = b; return o; }
  __device__ gbytes at(uint64_t p) const { return base + p; }
  __device__ bool contiguous(uint64_t, uint32_t) const { return true; }  // n bytes from p in one piece
};
struct OutMapped {
  gbytes base;
  const AX_GLOBAL uint32_t* slot;
  uint32_t lb, junk;
  __device__ explicit OutMapped(const JobDev& j)
      : base(gp(j.out)), slot(gp(j.slot)), lb(uint32_t(__builtin_ctz(j.B))), junk(j.junk) {}
  __device__ OutMapped with_base(gbytes b) const { OutMapped o = *this; o.base = b; return o; }
  __device__ gbytes at(uint64_t p) const {
    uint32_t x = slot[p >> lb];
    if (x >= junk) x = junk;
    return base + (uint64_t(x) << lb) + (p & ((1u << lb) - 1u));
  }
  __device__ bool contiguous(uint64_t p, uint32_t n) const { return (p & ((1u << lb) - 1u)) + n <= (1u << lb); }
};

__device__ inline uint32_t job_off_cap(const JobDev& j) { return (10u * (j.B / j.mm + 1) + 15u) & ~15u; }
__device__ inline uint32_t job_len_cap(const JobDev& j) { return 3u * j.B; }

__device__ inline void report(DevStatus* st, int code, uint64_t block) {
  if (atomicCAS(&st->err, 0, code) == 0) atomicExch(&st->bad_block, (unsigned long long)block);
}

__device__ inline uint32_t lane_id() { return __lane_id(); }
// Fourth word of a raw buffer descriptor on gfx9-family parts (32-bit data
// format; untyped byte stores ignore it)
constexpr int kBufferWord3 = 0x00020000;

__device__ inline uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0u));
}

__device__ inline uint32_t ld32(const uint8_t* p) { return *reinterpret_cast<const uint32_t*>(p); }

// ------------------------------------------------------------------ k_ans --

struct AnsArgs {
  const JobDev* jobs;
  const WinBlock* wbl;       // this window's blocks
  uint32_t n_items;          // blocks in this window
  uint32_t slot_b;           // scratch slot stride of the literal and command streams
  uint8_t* lit;              // scratch, slot_b per slot
  uint8_t* cmd;              // scratch, slot_b per slot
  uint8_t* off;              // scratch, off_cap per slot
  uint8_t* len;              // scratch, len_cap per slot
  uint32_t off_cap, len_cap;
  uint32_t* nsym;            // 4 per slot
  DevStatus* st;
};

// Wave-level exclusive prefix sum of a u32.
__device__ inline uint32_t wave_excl_sum(uint32_t v, uint32_t* total) {
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o, 64);
    if (lane_id() >= (uint32_t)o) x += y;
  }
  *total = __shfl(x, 63, 64);
  return x - v;
}

// Wave-level moves for the scans (DPP): row_shr:k moves each lane's value k
// lanes up inside its row of 16; row_bcast:15 / :31 hand lane 15 / 31 to the
// rows selected by the row mask.  Lanes without a source, or in unselected
// rows, receive `id`.
constexpr int kDppRowShr = 0x110, kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143, kDppWaveShr1 = 0x138;
template <int CTRL, int ROWS>
__device__ inline uint32_t dpp_move(uint32_t id, uint32_t x) {
  return uint32_t(__builtin_amdgcn_update_dpp(int(id), int(x), CTRL, ROWS, 0xF, false));
}

// Inclusive wave scan of a u32 (sum): 1, 2, 4, 8 inside the rows, then the
// row totals across rows.
__device__ inline uint32_t wave_incl_sum32(uint32_t x) {
  x += dpp_move<kDppRowShr + 1, 0xF>(0, x);
  x += dpp_move<kDppRowShr + 2, 0xF>(0, x);
  x += dpp_move<kDppRowShr + 4, 0xF>(0, x);
  x += dpp_move<kDppRowShr + 8, 0xF>(0, x);
  x += dpp_move<kDppRowBcast15, 0xA>(0, x);
  x += dpp_move<kDppRowBcast31, 0xC>(0, x);
  return x;
}

// The decode loop is a chain of three LDS reads per symbol and is bound by
// instruction issue when the device is full, by that chain when it is not.
// Tables go by a symbol's rank among the present ones: the slot table is then
// a prefix sum over start marks, four slots a word, instead of a loop over the
// slots and the symbol list.
//
// kWide, for windows of at most kWideBlocks blocks: the chain is what counts
// and LDS is free, so every slot gets its whole entry (16 KiB, seven waves a
// compute unit) and a step's chain is two reads.  64 KiB of DNA 76.7 -> 75.1 us,
// 4 MiB 104.5 -> 102.0, a 16 KiB range 95.5 -> 92.5; 80 MiB of text and other
// long literal alphabets are the same.  With more blocks the waves that fit
// count: 2048 blocks of reads 226 -> 246 us, 4096 of DNA 155 -> 199, 15500 of
// DNA 686 -> 941 (whole decodes); at a line of 1100 a batch of 32 ranges lost 8 to
// 12 of 350 us.
constexpr uint32_t kWideBlocks = 512;
template <bool kWide>
__global__ __launch_bounds__(64) void k_ans(AnsArgs a) {
  __shared__ uint32_t wide[kWide ? ax::kProbScale : 1];  // slot -> f | (slot - cum) << 12 | symbol << 24
  // slot -> rank, or 4 * rank (the entry's place in bytes) where that fits
  __shared__ __attribute__((aligned(16))) uint8_t ranktab[ax::kProbScale];
  __shared__ uint32_t fctab[256];  // by rank: f | cum << 12 | symbol << 24

  const uint32_t item = blockIdx.x % a.n_items;
  const uint32_t stream = blockIdx.x / a.n_items;  // 0 LIT, 1 LEN, 2 OFF, 3 CMD
  const WinBlock wb = a.wbl[item];
  const JobDev& J = a.jobs[wb.job];
  const uint64_t b = wb.b;
  const uint32_t lane = lane_id();
  uint8_t* const outs[4] = {a.lit + uint64_t(item) * a.slot_b, a.len + uint64_t(item) * a.len_cap,
                            a.off + uint64_t(item) * a.off_cap, a.cmd + uint64_t(item) * a.slot_b};
  const uint32_t caps[4] = {J.B, job_len_cap(J), job_off_cap(J), J.B};
  AX_GLOBAL uint8_t* const out = gp(outs[stream]);
  const uint32_t cap = caps[stream];
  uint32_t* nsym = a.nsym + 4 * item + stream;

  const uint64_t* idx = reinterpret_cast<const uint64_t*>(J.arc + 64);
  const uint64_t o0 = idx[b], o1 = idx[b + 1];
  const uint8_t* blk = J.arc + J.payload_at + o0;
  const uint64_t blen = o1 - o0;  // validated on the host: >= 16, 16-aligned
  uint64_t at = 16;
  for (uint32_t k = 0; k < stream; ++k) at += ld32(blk + 4 * k);
  const uint32_t rlen = ld32(blk + 4 * stream);
  if (at + rlen > blen || rlen < 8 || (rlen & 3)) {
    if (lane == 0) { report(a.st, AX_E_CORRUPT, b); *nsym = 0; }
    return;
  }
  const uint8_t* rec = blk + at;
  const uint32_t n = ld32(rec), mode = rec[4], pa = rec[5], pb = rec[6];
  if (n > cap) {
    if (lane == 0) { report(a.st, AX_E_CORRUPT, b); *nsym = 0; }
    return;
  }
  if (mode == 0) {  // raw: copy 4 bytes per lane per step
    if (8 + uint64_t(n) > rlen) {
      if (lane == 0) { report(a.st, AX_E_CORRUPT, b); *nsym = 0; }
      return;
    }
    const uint32_t words = (n + 3) / 4;
    for (uint32_t w = lane; w < words; w += 64)
      reinterpret_cast<AX_GLOBAL uint32_t*>(out)[w] = gp(reinterpret_cast<const uint32_t*>(rec + 8))[w];
    if (lane == 0) *nsym = n;
    return;
  }
  if (mode == 1) {  // constant
    const uint32_t v = pa * 0x01010101u, words = (n + 3) / 4;
    for (uint32_t w = lane; w < words; w += 64) reinterpret_cast<AX_GLOBAL uint32_t*>(out)[w] = v;
    if (lane == 0) *nsym = n;
    return;
  }
  bool bad = mode != 2 || pa > ax::kMaxLanesLog2 || rlen < 12;
  const uint32_t K = 1u << (pa & 7), present = pb + 1;
  bad |= present < 2;
  uint64_t p = 12;
  const uint32_t nw = bad ? 0 : ld32(rec + 8);
  const uint64_t states_at = p;
  p += 4ull * K;
  const uint64_t words_at = p;
  p = (p + 2ull * nw + 3) & ~3ull;
  const uint64_t set_at = p;
  p += present <= 32 ? present : 32;
  p = (p + 1) & ~1ull;
  const uint64_t freq_at = p;
  p = (p + 2ull * present + 3) & ~3ull;
  bad |= p != rlen;
  if (bad) {
    if (lane == 0) { report(a.st, AX_E_CORRUPT, b); *nsym = 0; }
    return;
  }
  // the states and the first words, on their way while the tables are built
  // (254 MB of DNA 686 -> 681 us, 16 MiB in 4 KiB blocks 153.6 -> 151.0)
  const AX_GLOBAL uint16_t* words = gp(reinterpret_cast<const uint16_t*>(rec + words_at));
  uint32_t x = lane < K ? ld32(rec + states_at + 4 * lane) : ax::kRansLow;
  const uint32_t wlast = nw ? nw - 1 : 0;
  auto fetch = [&](uint32_t i) -> uint32_t { return uint32_t(words[i < wlast ? i : wlast]); };
  const uint32_t P0 = fetch(lane), P1 = fetch(64 + lane);
  uint32_t N = fetch(128 + lane);
  // --- tables: lane l holds up to four present symbols in ascending order.
  uint32_t sym0 = 4 * lane, bits = 0;  // its symbols: sym0 + j where bit j is set
  if (present <= 32) {
    if (lane < present) sym0 = rec[set_at + lane], bits = 1;
  } else {
    bits = (rec[set_at + (lane >> 1)] >> ((lane & 1) * 4)) & 15u;
  }
  const uint32_t cnt = __popc(bits), ranks = wave_incl_sum32(cnt), rank0 = ranks - cnt;
  bad = uint32_t(__builtin_amdgcn_readlane(ranks, 63)) != present;
  uint32_t myf[4], fsum = 0;
#pragma unroll
  for (uint32_t j = 0, r = rank0; j < 4; ++j) {
    myf[j] = 0;
    if (!((bits >> j) & 1)) continue;
    if (r < present) myf[j] = *reinterpret_cast<const uint16_t*>(rec + freq_at + 2 * r);
    bad |= myf[j] < 1 || myf[j] >= ax::kProbScale;
    fsum += myf[j];
    ++r;
  }
  if (present <= 32 && cnt && lane > 0) bad |= rec[set_at + lane - 1] >= sym0;  // strictly ascending
  const uint32_t fincl = wave_incl_sum32(fsum);
  bad |= uint32_t(__builtin_amdgcn_readlane(fincl, 63)) != ax::kProbScale;
  const u32x4 zero = {0, 0, 0, 0};
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) *reinterpret_cast<u32x4*>(ranktab + 64 * lane + 16 * q) = zero;
  if (__ballot(bad)) {
    if (lane == 0) { report(a.st, AX_E_CORRUPT, b); *nsym = 0; }
    return;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t j = 0, r = rank0, cum = fincl - fsum; j < 4; ++j) {  // cum < 4096: every f is at least 1
    if (!((bits >> j) & 1)) continue;
    fctab[r] = myf[j] | (cum << 12) | ((sym0 + j) << 24);
    if (r) ranktab[cum] = !kWide && present <= 64 ? 4 : 1;
    cum += myf[j];
    ++r;
  }
  __syncthreads();
  {  // marks -> ranks: lane l sums its slots [64l, 64l+64), byte-wise four a word
    u32x4 v[4];
    uint32_t run = 0;  // the sum so far, in every byte
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      v[q] = *reinterpret_cast<const u32x4*>(ranktab + 64 * lane + 16 * q);
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) {
        uint32_t x = v[q][e];
        x += x << 8;
        x += x << 16;
        v[q][e] = x + run;
        run = __builtin_amdgcn_perm(0u, v[q][e], 0x03030303u);
      }
    }
    const uint32_t mine = run & 0xFFu, base = (wave_incl_sum32(mine) - mine) * 0x01010101u;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) *reinterpret_cast<u32x4*>(ranktab + 64 * lane + 16 * q) = v[q] + base;
  }
  __syncthreads();
  if (kWide) {
#pragma unroll 8
    for (uint32_t slot = lane; slot < ax::kProbScale; slot += 64) {
      const uint32_t fc = fctab[ranktab[slot]];
      wide[slot] = (fc & 0xFF000FFFu) | ((slot - ((fc >> 12) & 0xFFFu)) << 12);
    }
    __syncthreads();
  }
  // --- decode: lane j owns symbols j, j+K, ...
  // The renormalisation words of a step are taken in lane order from a
  // window: lane l's register P holds word base+l in its low half and word
  // base+64+l in its high half, N holds word base+128+l (in flight while the
  // window is used).  A step's words lie in [ptr, ptr+64) with ptr-base < 64,
  // so one permute of P from lane (ptr-base+below) mod 64 and a byte select
  // of the half give each lane its word.  Once ptr-base reaches 64 the window
  // moves by 64: P takes its high half and N's word, and N is reloaded.  Loads
  // are unconditional, the index clamped to the last word (inside the record;
  // a valid stream never consumes a word past nw)
  bad = x < ax::kRansLow;
  uint32_t base = 0;
  uint32_t P = P0 | (P1 << 16);
  uint32_t ptr = 0;
  const uint32_t steps = (n + K - 1) / K;
  // one step for the lanes in `need` (a subset of the decoding lanes):
  // returns the new state of a lane from its decoded xn
  auto renorm = [&](uint64_t m, uint32_t xn, bool need) -> uint32_t {
    const uint32_t q = __builtin_amdgcn_mbcnt_hi(
        uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), ptr - base));  // < 128; the permute takes the lane mod 64
    const uint32_t v = __builtin_amdgcn_ds_bpermute(int(q << 2), int(P));
    // (xn << 16) | the word: xn's two low bytes above v's low or high half
    const uint32_t xr = __builtin_amdgcn_perm(xn, v, q < 64 ? 0x05040100u : 0x05040302u);
    ptr += __popcll(m);
    if (ptr - base >= 64) {
      base += 64;
      P = __builtin_amdgcn_perm(N, P, 0x05040302u);
      N = fetch(base + 128 + lane);
    }
    return need ? xr : xn;
  };
  // Steps with all K lanes decoding: no per-lane bounds (a lane beyond K
  // decodes its own state and stores past the buffer's end, which drops it;
  // with K = 64 not even the ballot needs a mask).  Four steps' symbols are
  // gathered in a register, transposed in groups of four lanes, and leave as
  // one word per lane: a byte store for each step kept the store path busy for
  // three quarters of the kernel's time (254 MB DNA: 173 us, now 162; with the
  // slot table filled slot by slot 181)
  const uint32_t full = n / K;
  const uint64_t kmask = K == 64 ? ~0ull : ((1ull << K) - 1ull);
  const __amdgpu_buffer_rsrc_t orsrc = __builtin_amdgcn_make_buffer_rsrc(outs[stream], 0, int(n), kBufferWord3);
  const uint32_t beyond = lane < K ? 0u : 0x40000000u;
  // the entry of x's slot, and the state after its symbol
  auto entry = [&](auto small_tag, uint32_t& xn) -> uint32_t {
    const uint32_t slot = x & (ax::kProbScale - 1);
    uint32_t fc;
    if (kWide) {
      fc = wide[slot];
      xn = (fc & 0xFFFu) * (x >> ax::kProbBits) + ((fc >> 12) & 0xFFFu);
      return fc;
    }
    const uint32_t r = ranktab[slot];
    if (decltype(small_tag)::value) fc = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(fctab) + r);
    else fc = fctab[r];
    xn = (fc & 0xFFFu) * (x >> ax::kProbBits) + slot - ((fc >> 12) & 0xFFFu);
    return fc;
  };
  auto full_steps = [&](auto all_tag, auto small_tag) {
    constexpr bool kAll = decltype(all_tag)::value;
    auto step = [&]() -> uint32_t {
      uint32_t xn;
      const uint32_t fc = entry(small_tag, xn);
      const bool need = xn < ax::kRansLow;
      uint64_t m = __builtin_amdgcn_ballot_w64(need);
      if (!kAll) m &= kmask;
      x = renorm(m, xn, need);
      return fc;
    };
    uint32_t t = 0;
    if (kAll || K >= 4) {
      // lane 4 q + i takes step i's symbols of lanes 4 q .. 4 q + 3
      const uint32_t sel1 = lane & 1 ? 0x03070105u : 0x06020400u, sel2 = lane & 2 ? 0x03020706u : 0x05040100u;
      const int at = int(((lane & 3u) * K + (lane & ~3u)) | beyond);
      for (; t + 4 <= full; t += 4) {
        uint32_t v = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) v = __builtin_amdgcn_perm(step(), v, 0x07030201u);  // symbols are the top bytes
        v = __builtin_amdgcn_perm(dpp_move<0xB1, 0xF>(0, v), v, sel1);  // with lane ^ 1
        v = __builtin_amdgcn_perm(dpp_move<0x4E, 0xF>(0, v), v, sel2);  // with lane ^ 2
        __builtin_amdgcn_raw_buffer_store_b32(v, orsrc, at, int(t * K), 0);
      }
    }
    for (; t < full; ++t) {
      const uint32_t fc = step();
      __builtin_amdgcn_raw_buffer_store_b8(uint8_t(fc >> 24), orsrc, int(lane | beyond), int(t * K), 0);
    }
  };
  const bool small = !kWide && present <= 64;
  if (K == 64 && small) full_steps(std::true_type{}, std::true_type{});
  else if (K == 64) full_steps(std::true_type{}, std::false_type{});
  else if (small) full_steps(std::false_type{}, std::true_type{});
  else full_steps(std::false_type{}, std::false_type{});
  uint32_t i = full * K + lane;
  for (uint32_t t = full; t < steps; ++t, i += K) {
    const bool act = lane < K && i < n;
    uint32_t xn;
    const uint32_t fc = small ? entry(std::true_type{}, xn) : entry(std::false_type{}, xn);
    const bool need = act && xn < ax::kRansLow;
    const uint32_t xr = renorm(__ballot(need), xn, need);
    if (act) {
      x = xr;
      out[i] = uint8_t(fc >> 24);
    }
  }
  bad |= lane < K && x != ax::kRansLow;
  bad |= ptr != nw;
  if (__ballot(bad)) {
    if (lane == 0) report(a.st, AX_E_CORRUPT, b);
  }
  if (lane == 0) *nsym = n;
}

// ---------------------------------------------------------------- k_parse --

// What the match layer looks source positions up in (kRecs), one record per
// 32 positions of a block: x = match coverage, y = token starts, z = the
// window's tokens starting before these positions, w = the next 32 positions'
// coverage, so one 16-byte load answers a lookup.  A block's records take the
// first half of its own command slot, dead when its parse ends.
__device__ inline AX_GLOBAL u32x4* block_recs(uint8_t* cmd, uint32_t slot_b, uint32_t item) {
  return reinterpret_cast<AX_GLOBAL u32x4*>(gp(cmd + uint64_t(item) * slot_b));
}

struct ParseArgs {
  const JobDev* jobs;
  const WinBlock* wbl;
  uint32_t n_items;
  uint32_t n_tok;            // tokens in the window
  uint32_t slot_b;
  const uint8_t* lit;
  uint8_t* cmd;              // the commands; then the records (kRecs)
  const uint8_t *off, *len;
  uint32_t off_cap, len_cap;
  const uint32_t* nsym;
  uint64_t* tok;             // 2 u64 per token: src, dst | (len-1) << 48
  uint32_t* tblk;            // per token: its window block (null: the match layer needs neither this nor done)
  uint8_t* done;             // per token: kPending until the match layer copies it
  DevStatus* st;
  int write_out;             // 0: tokens only (the token-index build), no output bytes
  uint32_t open0, open1;     // the window's blocks whose match bytes are counted (Win::open)
  uint32_t* copied;          // their counters
};

// History maps.  A command acts on the four-entry distance history as a map
// from the history before it to the history after it; a run of commands
// composes these maps.  Each of the four output slots names where its
// distance comes from: an input slot j, or the explicit match at chunk
// position c (its distance is cdist[c]).  A map is two words: the slot bytes
// (j or c) and the tag bytes (0xFF: the slot byte is an input slot, 0x00: a
// chunk position).  Composing two maps is a byte gather, two v_perm_b32.
struct HMap {
  uint32_t v, t;
};
constexpr HMap kMapId{0x03020100u, 0xFFFFFFFFu};

// (later g) after (earlier f): slot i takes f's slot j where g's slot i reads
// input j (selector byte j: f's bytes are the permute's low four), else keeps
// g's own slot i (selector byte 4 + i).
__device__ inline HMap map_after(HMap g, HMap f) {
  const uint32_t sel = (g.v & g.t) | (0x07060504u & ~g.t);
  return HMap{__builtin_amdgcn_perm(g.v, f.v, sel), __builtin_amdgcn_perm(g.t, f.t, sel)};
}
__device__ inline uint64_t pick4(const uint64_t h[4], uint64_t j) {
  return j == 0 ? h[0] : j == 1 ? h[1] : j == 2 ? h[2] : h[3];
}

// Of more than 256 chunk positions a byte names only the lane; the tag byte of
// a position is then its wave (below 16, an input slot keeps 0xFF).
__device__ inline HMap map_of_wave(HMap m, uint32_t wv) { return HMap{m.v, m.t | (~m.t & (wv * 0x01010101u))}; }
__device__ inline HMap map_after_waves(HMap g, HMap f) {
  const uint32_t hi = g.t & 0x80808080u, in = (hi - (hi >> 7)) | hi;  // 0xFF where an input slot
  const uint32_t sel = (g.v & in) | (0x07060504u & ~in);
  return HMap{__builtin_amdgcn_perm(g.v, f.v, sel), __builtin_amdgcn_perm(g.t, f.t, sel)};
}

template <uint32_t kT>
struct ParseShared {
  static constexpr uint32_t kWaves = kT / 64;
  static_assert(kWaves == 4 || kWaves == 8 || kWaves == 16, "a row of 16 lanes scans the waves");
  // the literal bytes of the 16-byte group a chunk leaves open, by chunk
  // parity (a chunk reads its predecessor's while it may write its own)
  u32x4 gcarry[2];
  uint64_t covw[kMaxB / 64];      // match coverage of the block's output positions (kRecs)
  uint64_t startw[kMaxB / 64];    // token starts among them (kRecs)
  uint64_t runbits[kMaxB / 64];   // starts of the chunk's literal runs, in the block's output positions
  uint16_t runpre[kMaxB / 64];    // run starts in earlier words
  uint16_t rundelta[kT];  // per run: output position - literal index
  uint16_t runbeg[kT];    // per run: first output position
  uint16_t runend[kT];    // per run: one past its last output position
  u32x4 below[17];                // below[k]: sixteen bytes, the first k of them 0xFF
  // the block's decoded offset and length streams, when they fit, and where
  // each of their values ends (one past its last byte)
  __attribute__((aligned(16))) uint8_t offb[kOffStage + 16];
  __attribute__((aligned(16))) uint8_t lenb[kLenStage + 16];
  uint16_t offend[kOffStage];
  uint16_t lenend[kLenStage];
  uint64_t offval[kT];
  uint64_t wsum[kWaves][2];
  HMap wmap[kWaves];
  uint64_t cdist[kT];  // distance of the explicit match at each chunk position
  uint64_t last4[4];              // the chunk's last explicit-match distances, newest first
  uint32_t wterm[kWaves];
  int32_t wlast[kWaves];
  uint32_t leb_found, leb_cursor;
  // coverage bits of the 16-byte group a chunk leaves open, by chunk parity
  // (a chunk reads its predecessor's while it may write its own)
  uint32_t mcarry[2];
  int bad;
  alignas(4) uint8_t anyb[2][kWaves];  // block_any: one byte per wave, two call sites
};

// Block-wide "any thread's p": a ballot per wave, one LDS byte
// per wave, one barrier.  Slot k's bytes are rewritten only after a later
// barrier, so every thread has read them.
template <class S>
__device__ inline bool block_any(bool p, S& sh, int k) {
  const bool w = __ballot(p) != 0;
  if (lane_id() == 0) sh.anyb[k][threadIdx.x >> 6] = uint8_t(w);
  __syncthreads();
  uint32_t any = 0;
#pragma unroll
  for (uint32_t q = 0; q < S::kWaves / 4; ++q) any |= reinterpret_cast<const uint32_t*>(sh.anyb[k])[q];
  return any != 0;
}

// Block-wide exclusive scan of a u64 holding two u32 sums (the halves are
// scanned separately: no half may carry).  One barrier: a slot is written again
// only after a later one.  Of more than four waves, each wave scans the sums in
// its first row of lanes.
__device__ inline uint32_t row_incl_sum32(uint32_t x) {
  x += dpp_move<kDppRowShr + 1, 0xF>(0, x);
  x += dpp_move<kDppRowShr + 2, 0xF>(0, x);
  x += dpp_move<kDppRowShr + 4, 0xF>(0, x);
  x += dpp_move<kDppRowShr + 8, 0xF>(0, x);
  return x;
}
template <class S>
__device__ inline uint64_t block_excl_sum64(uint64_t v, uint64_t* total, S& sh, int slotk) {
  const uint32_t lane = lane_id(), wv = threadIdx.x >> 6;
  const uint64_t x = wave_incl_sum32(uint32_t(v)) | (uint64_t(wave_incl_sum32(uint32_t(v >> 32))) << 32);
  if (lane == 63) sh.wsum[wv][slotk] = x;
  __syncthreads();
  if constexpr (S::kWaves > 4) {
    const uint64_t w = lane < S::kWaves ? sh.wsum[lane][slotk] : 0;
    const uint32_t lo = row_incl_sum32(uint32_t(w)), hi = row_incl_sum32(uint32_t(w >> 32));
    auto upto = [&](uint32_t k) {  // the sum of waves 0 to k
      return uint64_t(uint32_t(__builtin_amdgcn_readlane(lo, k))) | (uint64_t(uint32_t(__builtin_amdgcn_readlane(hi, k))) << 32);
    };
    *total = upto(S::kWaves - 1);
    const uint32_t u = __builtin_amdgcn_readfirstlane(wv);
    return (u ? upto(u - 1) : 0) + x - v;
  }
  uint64_t pre = 0, tot = 0;
  for (uint32_t k = 0; k < 4; ++k) {
    const uint64_t t = sh.wsum[k][slotk];
    if (k < wv) pre += t;
    tot += t;
  }
  *total = tot;
  return pre + x - v;
}

// Block-wide exclusive scan of history maps; returns the map before this
// command and the chunk's total map.
template <int CTRL, int ROWS>
__device__ inline HMap map_dpp(HMap m) {
  return HMap{dpp_move<CTRL, ROWS>(kMapId.v, m.v), dpp_move<CTRL, ROWS>(kMapId.t, m.t)};
}
template <class S>
__device__ inline HMap block_excl_map(HMap m, HMap* total, S& sh) {
  const uint32_t lane = lane_id(), wv = threadIdx.x >> 6;
  HMap x = m;  // inclusive wave scan, earlier lanes' maps applied first (the identity fills gaps)
  x = map_after(x, map_dpp<kDppRowShr + 1, 0xF>(x));
  x = map_after(x, map_dpp<kDppRowShr + 2, 0xF>(x));
  x = map_after(x, map_dpp<kDppRowShr + 4, 0xF>(x));
  x = map_after(x, map_dpp<kDppRowShr + 8, 0xF>(x));
  x = map_after(x, map_dpp<kDppRowBcast15, 0xA>(x));
  x = map_after(x, map_dpp<kDppRowBcast31, 0xC>(x));
  if constexpr (S::kWaves > 4) x = map_of_wave(x, wv);
  if (lane == 63) sh.wmap[wv] = x;
  __syncthreads();
  HMap pre = kMapId, tot = kMapId;
  if constexpr (S::kWaves > 4) {
    HMap w = lane < S::kWaves ? sh.wmap[lane] : kMapId;
    w = map_after_waves(w, map_dpp<kDppRowShr + 1, 0xF>(w));
    w = map_after_waves(w, map_dpp<kDppRowShr + 2, 0xF>(w));
    w = map_after_waves(w, map_dpp<kDppRowShr + 4, 0xF>(w));
    w = map_after_waves(w, map_dpp<kDppRowShr + 8, 0xF>(w));
    auto upto = [&](uint32_t k) {
      return HMap{uint32_t(__builtin_amdgcn_readlane(w.v, k)), uint32_t(__builtin_amdgcn_readlane(w.t, k))};
    };
    *total = upto(S::kWaves - 1);
    const uint32_t u = __builtin_amdgcn_readfirstlane(wv);
    if (u) pre = upto(u - 1);
    return map_after_waves(map_dpp<kDppWaveShr1, 0xF>(x), pre);
  }
  for (uint32_t k = 0; k < 4; ++k) {
    if (k < wv) pre = map_after(sh.wmap[k], pre);
    tot = map_after(sh.wmap[k], tot);
  }
  *total = tot;
  return map_after(map_dpp<kDppWaveShr1, 0xF>(x), pre);  // inclusive of the previous lane
}

// Distance named by slot k of a map: an input slot of hist, or an explicit
// match of the chunk.
template <class S>
__device__ inline uint64_t map_value(HMap m, uint32_t k, const uint64_t hist[4], const S& sh) {
  const uint32_t g = (m.v >> (8 * k)) & 0xFFu;
  if constexpr (S::kWaves > 4) {
    const uint32_t w = (m.t >> (8 * k)) & 0xFFu;
    return (w >> 7) ? pick4(hist, g & 3) : sh.cdist[64 * w + g];
  }
  return ((m.t >> (8 * k)) & 1u) ? pick4(hist, g & 3) : sh.cdist[g];
}

// Decode `count` consecutive LEB128 values starting at byte *cursor of
// src[0..n) into dst (u64) — all threads, BPT bytes each per window.  A byte below 0x80 ends a value; terminators are counted by a block
// scan, and each terminator's thread assembles its value from the bytes after
// the previous terminator.  Returns false on a malformed or missing value.
// *cursor advances past the last value.
template <uint32_t BPT, class Src, class S>
__device__ bool leb_values(Src src, uint32_t n, uint32_t* cursor, uint32_t count, uint64_t* dst, S& sh) {
  const uint32_t t = threadIdx.x, lane = lane_id(), wv = t >> 6;
  const uint32_t first = *cursor;
  uint32_t found = 0;
  uint32_t win = first & ~(BPT - 1);
  uint32_t value_start = first;  // start of the value that is open at the window start
  bool ok = true;
  while (found < count) {
    if (win >= n) { ok = false; break; }
    const uint32_t p0 = win + BPT * t;
    uint32_t tm = 0;  // terminators among this thread's bytes
#pragma unroll
    for (uint32_t q = 0; q < BPT; ++q) {
      const uint32_t pos = p0 + q;
      if (pos >= first && pos < n && src[pos] < 0x80) tm |= 1u << q;
    }
    const uint32_t c = __popc(tm);
    const uint32_t incl = wave_incl_sum32(c);
    const int32_t mylast = tm ? int32_t(p0 + 31 - __clz(tm)) : -1;
    const uint64_t hm = __ballot(tm != 0);
    if (lane == 63) sh.wterm[wv] = incl;
    if (hm == 0 ? lane == 0 : lane == uint32_t(63 - __clzll(hm))) sh.wlast[wv] = mylast;
    __syncthreads();
    uint32_t before = incl - c, all = 0;
    for (uint32_t k = 0; k < S::kWaves; ++k) {
      if (k < wv) before += sh.wterm[k];
      all += sh.wterm[k];
    }
    // the last terminator before this thread's bytes
    const uint64_t lower = hm & ((1ull << lane) - 1ull);
    const int32_t from_lane = __shfl(mylast, lower ? 63 - __clzll(lower) : 0, 64);
    int32_t prev = lower ? from_lane : -1;
    if (prev < 0)
      for (int32_t k = int32_t(wv) - 1; k >= 0; --k)
        if (sh.wlast[k] >= 0) { prev = sh.wlast[k]; break; }
    uint32_t vi = found + before;
    uint32_t start = prev >= 0 ? uint32_t(prev) + 1 : value_start;
    for (uint32_t q = 0; q < BPT; ++q) {
      if (!((tm >> q) & 1)) continue;
      const uint32_t pos = p0 + q;
      if (vi < count) {
        if (pos + 1 - start > 10) {
          ok = false;
        } else {
          uint64_t v = 0;
          for (uint32_t r = start; r <= pos; ++r) v |= uint64_t(src[r] & 0x7F) << (7 * (r - start));
          if (pos - start == 9 && src[pos] > 1) ok = false;
          dst[vi] = v;
          if (vi == count - 1) sh.leb_cursor = pos + 1;
        }
      }
      ++vi;
      start = pos + 1;
    }
    // the value still open at the end of this window starts after its last terminator
    int32_t last = -1;
    for (int32_t k = int32_t(S::kWaves) - 1; k >= 0; --k)
      if (sh.wlast[k] >= 0) { last = sh.wlast[k]; break; }
    if (last >= 0) value_start = uint32_t(last) + 1;
    if (win + BPT * 64 * S::kWaves - value_start > 10 && found + all < count) ok = false;  // a value longer than 10 bytes
    found += all;
    win += BPT * 64 * S::kWaves;
    __syncthreads();
  }
  if (block_any(!ok, sh, 0)) return false;
  if (count) *cursor = sh.leb_cursor;
  __syncthreads();
  return true;
}

// The terminators (bytes below 0x80) among the first n bytes of v, one bit per byte.
__device__ inline uint32_t leb_ends(u32x4 v, uint32_t n) {
  auto four = [](uint32_t w) {
    w = (~w >> 7) & 0x01010101u;
    return (w | (w >> 7) | (w >> 14) | (w >> 21)) & 0xFu;
  };
  const uint32_t m = four(v.x) | (four(v.y) << 4) | (four(v.z) << 8) | (four(v.w) << 12);
  return n >= 16 ? m : m & ((1u << n) - 1u);
}

// Value k of a staged stream: its bytes are src[end[k - 1], end[k]).  False on
// a value longer than ten bytes or beyond 64 bits.  (The bytes behind a value
// may be read and are masked off: the stages are padded.)
__device__ inline bool leb_staged(const uint8_t* src, const uint16_t* end, uint32_t k, uint64_t& v) {
  const uint32_t b = k ? end[k - 1] : 0u, n = end[k] - b;
  const uint32_t* const w = reinterpret_cast<const uint32_t*>(src) + (b >> 2);
  const uint32_t w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
  uint64_t x = __builtin_amdgcn_alignbyte(w1, w0, b) | (uint64_t(__builtin_amdgcn_alignbyte(w2, w1, b)) << 32);
  const uint32_t hi = n > 8 ? __builtin_amdgcn_alignbyte(w3, w2, b) : 0u;  // bytes 8 and 9
  if (n < 8) x &= (1ull << (8 * n)) - 1;
  // seven bits of each of eight bytes, in pairs, fours, then all
  x = (x & 0x007F007F007F007Full) | ((x & 0x7F007F007F007F00ull) >> 1);
  x = (x & 0x00003FFF00003FFFull) | ((x & 0x3FFF00003FFF0000ull) >> 2);
  v = (x & 0x0FFFFFFFull) | ((x >> 32) << 28) | (uint64_t(hi & 0x7Fu) << 56);
  if (n <= 9) return true;
  v |= uint64_t((hi >> 8) & 1u) << 63;
  return n == 10 && (hi & 0xFF00u) <= 0x100u;
}

// Of 256 threads seven waves per SIMD (at most 72 VGPRs), as many as the LDS
// allows (six: 254 MB DNA 741 instead of 728 us, eight: 768).
//
// A chunk, a command per thread, is a chain of block-wide steps: with few blocks in
// flight its latency counts, with many the instructions issued.  The values
// of the offset and length streams are therefore found once per block (one
// scan over the staged bytes lists where every value ends) and read by the
// command that needs them, instead of a scan over a window of the stream for
// every chunk: 64 KiB of DNA parse in 42 -> 29 us, 254 MB in 253 -> 208 us.
//
// kRecs: 0 no records, 1 records for the match layer, 2 also count the match
// bytes of open blocks (as a branch of 1 it costs the smallest decodes 0.2 us).
template <class O, int kRecs, uint32_t kT>
__global__ __launch_bounds__(kT, kT == kParseThreads ? 7 : 4) void k_parse(ParseArgs a) {
  __shared__ ParseShared<kT> sh;
  const uint32_t item = blockIdx.x, t = threadIdx.x;
  const uint8_t* cmd = a.cmd + uint64_t(item) * a.slot_b;
  const AX_GLOBAL uint8_t* const litg = gp(a.lit + uint64_t(item) * a.slot_b);
  const uint8_t* offs = a.off + uint64_t(item) * a.off_cap;
  const uint8_t* lens = a.len + uint64_t(item) * a.len_cap;
  // loads that need only the block's place in the window come first: the
  // chunk's command bytes (inside the slot whatever the count) and one 16-byte piece per thread of the offset and length
  // streams, staged in LDS if the stream fits the stage (the slots are
  // 16-aligned and their capacities multiples of 16, so the loads stay in this
  // block's slots)
  static_assert(kOffStage <= 16 * kT && kLenStage <= 16 * kT, "one piece per thread");
  uint32_t cnext = t < a.slot_b ? gp(cmd)[t] : 0u;
  u32x4 po = {0, 0, 0, 0}, pl = {0, 0, 0, 0};
  if (16 * t < min(kOffStage, a.off_cap)) po = *reinterpret_cast<const AX_GLOBAL u32x4*>(gp(offs) + 16 * t);
  if (16 * t < min(kLenStage, a.len_cap)) pl = *reinterpret_cast<const AX_GLOBAL u32x4*>(gp(lens) + 16 * t);
  const WinBlock wb = a.wbl[item];
  const uint64_t tok_lo = wb.tok, tok_n = (item + 1 < a.n_items ? a.wbl[item + 1].tok : a.n_tok) - wb.tok;
  const uint32_t n_lit = a.nsym[4 * item + 0], n_len = a.nsym[4 * item + 1];
  const uint32_t n_off = a.nsym[4 * item + 2], n_cmd = a.nsym[4 * item + 3];
  const JobDev& J = a.jobs[wb.job];
  const uint64_t b = wb.b;
  const uint32_t B = J.B, mm = J.mm;
  const uint64_t bs = b * B;
  const uint32_t blen = uint32_t(min<uint64_t>(B, J.n_bytes - bs));
  // the archive's own match count, checked at the end
  const uint64_t* mpre = reinterpret_cast<const uint64_t*>(J.arc + 64) + J.nb + 1;
  const uint64_t arc_n = mpre[b + 1] - mpre[b];

  if (t == 0)
    sh.bad = (n_lit > B || n_cmd > B || n_len > job_len_cap(J) || n_off > job_off_cap(J)) ? 1 : 0;
  if (kRecs && t < kMaxB / 64) sh.covw[t] = 0, sh.startw[t] = 0;
  static_assert(kMaxB / 64 <= kT, "one map word per thread");
  // the block's output bytes (contiguous); groups below `full` are whole
  AX_GLOBAL uint8_t* const o = a.write_out ? O(J).at(bs) : nullptr;
  const uint32_t full = blen & ~15u;
  const bool off_lds = n_off <= kOffStage, len_lds = n_len <= kLenStage;
  uint32_t oe = 0, le = 0;
  if (off_lds && 16 * t < n_off) {
    *reinterpret_cast<u32x4*>(sh.offb + 16 * t) = po;
    oe = leb_ends(po, n_off - 16 * t);
  }
  if (len_lds && 16 * t < n_len) {
    *reinterpret_cast<u32x4*>(sh.lenb + 16 * t) = pl;
    le = leb_ends(pl, n_len - 16 * t);
  }
  if (t < 17) {
    const uint64_t lo = t < 8 ? (1ull << (8 * t)) - 1 : ~0ull;
    const uint64_t hi = t <= 8 ? 0 : t < 16 ? (1ull << (8 * (t - 8))) - 1 : ~0ull;
    sh.below[t] = u32x4{uint32_t(lo), uint32_t(lo >> 32), uint32_t(hi), uint32_t(hi >> 32)};
  }
  if (t < kMaxB / 64) sh.runbits[t] = 0;
  // where the streams' values end; off_n and len_n count them
  uint64_t ends;
  const uint64_t eex = block_excl_sum64(uint64_t(__popc(oe)) | (uint64_t(__popc(le)) << 32), &ends, sh, 1);
  const uint32_t off_n = uint32_t(ends), len_n = uint32_t(ends >> 32);
  for (uint32_t k = uint32_t(eex); oe; oe &= oe - 1, ++k) sh.offend[k] = uint16_t(16 * t + __builtin_ctz(oe) + 1);
  for (uint32_t k = uint32_t(eex >> 32); le; le &= le - 1, ++k) sh.lenend[k] = uint16_t(16 * t + __builtin_ctz(le) + 1);
  bool failed = sh.bad != 0;
  // streams too long for their stage are read from global memory, a chunk's values at a time
  const AX_GLOBAL uint8_t* const offg = gp(offs);
  const AX_GLOBAL uint8_t* const leng = gp(lens);

  uint32_t dst = 0, litp = 0, offc = 0, lenc = 0;  // offc, lenc: staged, values taken; else bytes
  uint64_t ntok = 0;
  uint64_t hist[4] = {1, 2, 3, 4};
  for (uint32_t c0 = 0; c0 < n_cmd && !failed; c0 += kT) {
    const uint32_t i = c0 + t;
    const bool valid = i < n_cmd;
    const uint32_t c = valid ? cnext : 0u;
    cnext = i + kT < n_cmd ? cmd[i + kT] : 0u;  // the next chunk's, in flight meanwhile
    const uint32_t kind = c & 3;
    bool bad = valid && kind == 3;
    const uint32_t v = kind == 2 ? (c >> 4) : (c >> 2);
    const bool esc = valid && !bad && v == (kind == 2 ? 15u : 63u);
    const bool is0 = valid && kind == 0, is1 = valid && kind == 1, is2 = valid && kind == 2;
    const uint64_t packed = uint64_t(esc) | (uint64_t(is1) << 16) | (uint64_t(is0) << 32) | (uint64_t(is1 || is2) << 48);
    uint64_t ctot;
    const uint64_t cex = block_excl_sum64(packed, &ctot, sh, 0);
    const uint32_t esc_i = uint32_t(cex & 0xFFFF), k1_i = uint32_t((cex >> 16) & 0xFFFF);
    const uint32_t run_i = uint32_t((cex >> 32) & 0xFFFF), tok_i = uint32_t(cex >> 48);
    const uint32_t n_esc = uint32_t(ctot & 0xFFFF), n_k1 = uint32_t((ctot >> 16) & 0xFFFF);
    const uint32_t n_tokc = uint32_t(ctot >> 48);
    // length and offset values of this chunk
    uint32_t ext = 0;
    if (len_lds) {
      if (esc) {
        uint64_t e = 0;
        if (lenc + esc_i < len_n && leb_staged(sh.lenb, sh.lenend, lenc + esc_i, e) && e <= B) ext = uint32_t(e);
        else bad = true;
      }
      lenc += n_esc;
    } else if (n_esc) {  // n_esc is the same for the whole block
      if (!leb_values<kLenBpt>(leng, n_len, &lenc, n_esc, sh.offval, sh)) {
        failed = true;
        break;
      }
      if (esc) {
        const uint64_t e = sh.offval[esc_i];
        ext = uint32_t(e);
        bad |= e > B;
      }
      __syncthreads();
    }
    uint64_t off = 0;  // an explicit match's source
    if (off_lds) {
      if (is1) bad |= offc + k1_i >= off_n || !leb_staged(sh.offb, sh.offend, offc + k1_i, off);
      offc += n_k1;
    } else {
      if (!leb_values<kOffBpt>(offg, n_off, &offc, n_k1, sh.offval, sh)) {
        failed = true;
        break;
      }
      if (is1) off = sh.offval[k1_i];
    }
    uint32_t len = 0;
    if (valid && !bad) len = v + (kind == 0 ? 1u : mm) + ext;
    const uint64_t lp = uint64_t(len) | (uint64_t(is0 ? len : 0u) << 32);
    uint64_t ptot;
    const uint64_t pex = block_excl_sum64(lp, &ptot, sh, 1);
    const uint32_t cdst = dst + uint32_t(pex & 0xFFFFFFFFu), clit = litp + uint32_t(pex >> 32);
    const uint32_t chunk_lit = uint32_t(ptot >> 32);
    if (valid && uint64_t(cdst) + len > blen) bad = true;
    if (is0 && uint64_t(clit) + len > n_lit) bad = true;
    const uint64_t absdst = bs + cdst;
    uint64_t src = 0;
    if (is1) {
      src = off;
      if (src >= absdst) bad = true;
      else sh.cdist[t] = absdst - src;
    }
    const uint32_t n_rep = n_tokc - n_k1;
    uint64_t nh[4];
    if (n_rep) {  // repeat matches read the history: scan the command maps
      HMap mine = kMapId;
      if (is1) {
        mine = HMap{(kT == 256 ? t : t & 63u) | 0x02010000u, 0xFFFFFF00u};
      } else if (is2) {
        const uint32_t r = (c >> 2) & 3;
        mine = HMap{r | ((r >= 1 ? 0u : 1u) << 8) | ((r >= 2 ? 1u : 2u) << 16) | ((r >= 3 ? 2u : 3u) << 24),
                    0xFFFFFFFFu};
      }
      HMap mtot;
      const HMap before = block_excl_map(mine, &mtot, sh);  // also orders the cdist writes
      if (is2) {
        const uint64_t d = map_value(before, (c >> 2) & 3, hist, sh);
        if (d > absdst) bad = true;
        else src = absdst - d;
      }
      for (uint32_t k = 0; k < 4; ++k) nh[k] = map_value(mtot, k, hist, sh);
    } else {  // explicit matches only: the history takes their last distances
      if (is1 && !bad && k1_i + 4 >= n_k1) sh.last4[n_k1 - 1 - k1_i] = absdst - src;
      __syncthreads();
      const uint32_t m4 = min(n_k1, 4u);
      for (uint32_t k = 0; k < 4; ++k) nh[k] = k < m4 ? sh.last4[k] : pick4(hist, k - m4);
    }
    if ((is1 || is2) && !bad) {
      const uint64_t gi = ntok + tok_i;
      if (gi < tok_n) {
        uint64_t* tk = a.tok + 2 * (tok_lo + gi);
        tk[0] = src;
        tk[1] = absdst | (uint64_t(len - 1) << 48);
        if (a.tblk) {
          a.tblk[tok_lo + gi] = item;
          a.done[tok_lo + gi] = kPending;
        }
        if (kRecs) atomicOr(reinterpret_cast<uint32_t*>(sh.startw) + (cdst >> 5), 1u << (cdst & 31));
      } else {
        bad = true;
      }
    }
    // literal runs: starts in the block's output positions
    if (is0 && !bad && len) {
      atomicOr(reinterpret_cast<uint32_t*>(sh.runbits) + (cdst >> 5), 1u << (cdst & 31));
      sh.rundelta[run_i] = uint16_t(cdst - clit);
      sh.runbeg[run_i] = uint16_t(cdst);
      sh.runend[run_i] = uint16_t(cdst + len);
    }
    if (block_any(bad, sh, 1)) { failed = true; break; }
    const uint32_t n_runs = uint32_t((ctot >> 32) & 0xFFFF);
    {  // run starts before each word of the output positions (B / 64 <= 256 words)
      const uint32_t c = t < B / 64 ? __popcll(sh.runbits[t]) : 0;
      uint64_t rt;
      const uint64_t pre = block_excl_sum64(c, &rt, sh, 0);
      if (t < B / 64) sh.runpre[t] = uint16_t(pre);
    }
    __syncthreads();
    // place the chunk's literal bytes by aligned 16-byte output groups: each
    // literal run meeting a group supplies the 16 literal bytes lined up with
    // the group under the group's byte mask, and the group leaves with one
    // 16-byte store (zeros where matches will be).  The group the chunk ends
    // in is carried to the next chunk, which begins in it
    const uint32_t dend = dst + uint32_t(ptot & 0xFFFFFFFFu);
    for (uint32_t c = (dst >> 4) + t; 16 * c < dend; c += kT) {
      const uint32_t d0 = max(16 * c, dst), d1 = min(16 * c + 16, dend), w = d0 >> 6;
      int32_t r = int32_t(sh.runpre[w] + __popcll(sh.runbits[w] & (~0ull >> (63 - (d0 & 63))))) - 1;
      if (r < 0 || d0 >= sh.runend[r]) ++r;  // the run holding d0, else the next one
      u32x4 val = {0, 0, 0, 0};
      uint32_t lit16 = 0;  // the group's literal bytes in this chunk
      for (; r < int32_t(n_runs) && sh.runbeg[r] < d1; ++r) {
        const uint32_t x0 = max(d0, uint32_t(sh.runbeg[r])), x1 = min(d1, uint32_t(sh.runend[r]));
        const int32_t l0 = int32_t(16 * c) - int32_t(sh.rundelta[r]);  // literal index of the group's byte 0
        // the 16 literal bytes lined up with the group: one unaligned load
        // (l0 may be as low as -15, and the load may run past the stream:
        // still inside the workspace)
        const u32x4 e = *reinterpret_cast<const AX_GLOBAL u32x4_u*>(litg + l0);
        const uint32_t m16 = ((1u << (x1 - 16 * c)) - 1u) & ~((1u << (x0 - 16 * c)) - 1u);
        val |= e & sh.below[x1 - 16 * c] & ~sh.below[x0 - 16 * c];
        lit16 |= m16;
        if (sh.runend[r] >= d1) break;
      }
      const uint32_t par = (c0 / kT) & 1;
      const bool head = d0 > 16 * c, open = d1 < 16 * c + 16 && d1 < blen;  // begun in / goes on in another chunk
      if (kRecs) {  // match coverage of the group: its bytes in this chunk that no literal fills
        uint32_t m = ((1u << (d1 - 16 * c)) - 1u) & ~((1u << (d0 - 16 * c)) - 1u) & ~lit16;
        if (head) m |= sh.mcarry[par ^ 1];
        if (open) sh.mcarry[par] = m;
        else reinterpret_cast<uint16_t*>(sh.covw)[c] = uint16_t(m);
      }
      if (head) val |= sh.gcarry[par ^ 1];
      if (open) {
        sh.gcarry[par] = val;
      } else if (a.write_out) {
        if (16 * c < full) {
          *reinterpret_cast<AX_GLOBAL u32x4*>(o + 16 * c) = val;
        } else {
          for (uint32_t i = 16 * c; i < blen; ++i) o[i] = uint8_t(val[(i >> 2) & 3] >> (8 * (i & 3)));
        }
      }
    }
    __syncthreads();
    if (t < kMaxB / 64) sh.runbits[t] = 0;  // the next chunk's bits are set several barriers on
    dst += uint32_t(ptot & 0xFFFFFFFFu);
    litp += chunk_lit;
    ntok += n_tokc;
    for (int k = 0; k < 4; ++k) hist[k] = nh[k];
  }
  // bytes taken of a staged stream
  if (off_lds) offc = offc <= off_n ? (offc ? sh.offend[offc - 1] : 0u) : ~0u;
  if (len_lds) lenc = lenc <= len_n ? (lenc ? sh.lenend[lenc - 1] : 0u) : ~0u;
  if (!failed && (dst != blen || litp != n_lit || lenc != n_len || offc != n_off || ntok != tok_n || arc_n != tok_n))
    failed = true;
  if (failed) {
    if (t == 0) report(a.st, AX_E_CORRUPT, b);
    return;
  }
  if (!kRecs) return;
  if (kRecs == 2 && item >= a.open0 && item < a.open1 && t < 64) {
    // not those of a block that does little but repeat its own bytes: walks end there at once
    uint32_t from = 0;
    if (t < tok_n) {
      const u64x2 tk = reinterpret_cast<const AX_GLOBAL u64x2*>(gp(a.tok))[tok_lo + t];
      const uint64_t dist = (tk.y & ((1ull << 48) - 1)) - tk.x;
      from = uint32_t(tk.y >> 48) + 1;
      if (tk.x >= bs && dist < from) from = uint32_t(dist);
    }
    const uint32_t walked = __builtin_amdgcn_readlane(wave_incl_sum32(from), 63);
    if (t == 0 && (tok_n > 64 || kOwnShare * walked >= blen))
      atomicAdd(a.copied + (item % kCopiedShards) * kCounterStride, blen - n_lit);
  }
  // the records the match layer looks sources up in: two per thread
  const uint64_t cw = t < kMaxB / 64 ? sh.covw[t] : 0, sw = t < kMaxB / 64 ? sh.startw[t] : 0;
  uint64_t all;
  const uint32_t pre = uint32_t(tok_lo) + uint32_t(block_excl_sum64(uint64_t(__popcll(sw)), &all, sh, 0));
  if (t < B / 64) {
    const uint32_t cn = t + 1 < B / 64 ? uint32_t(sh.covw[t + 1]) : 0u;
    AX_GLOBAL u32x4* const r = block_recs(a.cmd, a.slot_b, item) + 2 * t;
    r[0] = u32x4{uint32_t(cw), uint32_t(sw), pre, uint32_t(cw >> 32)};
    r[1] = u32x4{uint32_t(cw >> 32), uint32_t(sw >> 32), pre + uint32_t(__popc(uint32_t(sw))), cn};
  }
}

// ------------------------------------------------------------ match layer --

struct CopyArgs {
  const JobDev* jobs;
  const WinBlock* wbl;
  uint32_t n_items;
  const uint64_t* tok;       // window tokens in (job, output) order
  const uint32_t* tblk;      // per token: its window block
  uint32_t n_tok;
  uint32_t* cov;             // per token: first covering token, count
  uint8_t* done;             // per token: round that copied it, or kPending
  const uint32_t* list_in;   // pending tokens of the previous round: kSub sublists of sub_cap
  uint32_t* list_out;
  const uint32_t* cnt_in;    // kSub counters, kCounterStride apart
  uint32_t* cnt_out;
  uint32_t* cnt_clear;       // the counters the next round writes
  uint32_t sub_cap;
  uint32_t* long_list;       // round 0: ready tokens of at least kSplitToken bytes
  uint32_t* long_cnt;
  uint32_t round;
  DevStatus* st;
  uint32_t* pbits;           // the last round's leftovers, one bit per token
  const uint32_t* plist;     // the same tokens, ascending (the persistent finish's work)
  int mark;                  // this round is the last: 0 no, else kMarkList or kMarkJump
  uint64_t spin_limit;
  int serial;
  int fill_round, fill_tail;  // later rounds / persistent launch: kFillLaneWave or kFillSegmented
  uint32_t tail_chunks;       // consecutive 64-token chunks per persistent-launch ticket
  uint32_t* J;                // pointer jumping: one entry per window position
  uint64_t* lmap;             // pointer jumping: leftover map
  uint32_t S;                 // position stride of a window block
  uint8_t* cmd;              // command slots holding the parse's records (null: round 0 finds every cover)
  uint32_t one_job;           // 1: the plan has one job, so every token's output is jobs[0]'s
};

__device__ inline void token_at(const uint64_t* tok, uint64_t t, uint64_t& src, uint64_t& dst, uint32_t& len) {
  src = tok[2 * t];
  const uint64_t w = tok[2 * t + 1];
  dst = w & ((1ull << 48) - 1);
  len = uint32_t(w >> 48) + 1;
}

// Tokens [lo, lo+cnt) are those whose destinations meet [s0, s1) of the
// job of window block wb.  Tokens are disjoint and sorted by destination
// within a job, and a job's window blocks are contiguous and ascending, so
// the search runs over the job's window blocks, then inside the block that
// holds s0.  Source bytes outside every window block of the job were
// written by an earlier window or are not decoded by this plan (a range
// decode reads only bytes whose blocks it holds), so nothing waits on them.
__device__ inline void find_cover(const CopyArgs& a, const WinBlock& wb, uint32_t B, uint64_t s0, uint64_t s1,
                                  uint32_t& lo, uint32_t& cnt) {
  const uint64_t sb = s0 / B;
  const uint32_t job_end = wb.first + wb.count;
  uint32_t x = wb.first, y = job_end;
  const uint64_t b0 = a.wbl[wb.first].b;
  if (sb >= b0 && sb - b0 < wb.count && a.wbl[wb.first + uint32_t(sb - b0)].b == sb) {
    x = wb.first + uint32_t(sb - b0);  // the job's blocks are consecutive up to sb (whole-archive windows)
  } else {
    while (x < y) {  // first window block of the job with b >= sb
      const uint32_t mid = (x + y) >> 1;
      if (a.wbl[mid].b < sb) x = mid + 1; else y = mid;
    }
  }
  const uint32_t end_tok = job_end < a.n_items ? a.wbl[job_end].tok : a.n_tok;
  uint32_t p = x < job_end ? a.wbl[x].tok : end_tok;
  if (x < job_end && a.wbl[x].b == sb) {  // first token of block x ending after s0
    uint32_t q = x + 1 < a.n_items ? a.wbl[x + 1].tok : a.n_tok;
    while (p < q) {
      const uint32_t mid = (p + q) >> 1;
      const uint64_t w = a.tok[2 * uint64_t(mid) + 1];
      if ((w & ((1ull << 48) - 1)) + (w >> 48) + 1 <= s0) p = mid + 1; else q = mid;
    }
  }
  lo = p;
  cnt = 0;
  while (p + cnt < end_tok && (a.tok[2 * uint64_t(p + cnt) + 1] & ((1ull << 48) - 1)) < s1) ++cnt;
}

// Round 0 leaves the cover of its pending tokens to the round that first
// needs it (the covers of its ready tokens are never needed).
constexpr uint32_t kCovLazy = 0xFFFFFFFFu;
__device__ inline void cover_of(const CopyArgs& a, uint32_t t, uint64_t src, uint64_t dst, uint32_t len,
                                uint32_t& lo, uint32_t& cnt) {
  lo = a.cov[2 * t];
  cnt = a.cov[2 * t + 1];
  if (cnt != kCovLazy) return;
  const WinBlock wb = a.wbl[a.tblk[t]];
  const uint64_t dist = dst - src;
  find_cover(a, wb, a.jobs[wb.job].B, src, src + (dist < len ? dist : len), lo, cnt);
  a.cov[2 * t] = lo;
  a.cov[2 * t + 1] = cnt;
}

// The output of token t's archive.
template <class O>
__device__ inline O token_out(const CopyArgs& a, uint32_t t) { return O(a.jobs[a.wbl[a.tblk[t]].job]); }

template <bool COH>
__device__ inline uint8_t ldb(const AX_GLOBAL uint8_t* p) {
  if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}
template <bool COH>
__device__ inline void stb(gbytes p, uint8_t v) {
  if constexpr (COH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

// The serial ablation: one lane, byte after byte, reading the bytes it may
// itself have just written (a self-overlapping match is a dependency chain).
template <bool COH, class O>
__device__ inline void fill_serial(const O& out, uint64_t dst, uint64_t src, uint32_t len) {
  for (uint32_t k = 0; k < len; ++k) {
    stb<COH>(out.at(dst + k), ldb<COH>(out.at(src + k)));
    __builtin_amdgcn_s_waitcnt(0x0F70);  // the next load may read this byte
  }
}

// One lane fills a token as a periodic fill: sixteen source loads in flight,
// then sixteen stores.  The source index runs over the period dist (for
// dist >= len it never wraps and the fill is a plain copy).
template <bool COH, class O>
__device__ inline void fill_lane(const O& out, uint64_t dst, uint64_t src, uint32_t len) {
  const uint64_t dist = dst - src;
  uint64_t j = 0;
  for (uint32_t k0 = 0; k0 < len; k0 += 16) {
    uint64_t idx[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      idx[q] = j;
      if (++j == dist) j = 0;
    }
    uint8_t v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = (k0 + q < len) ? ldb<COH>(out.at(src + idx[q])) : uint8_t(0);
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (k0 + q < len) stb<COH>(out.at(dst + k0 + q), v[q]);
  }
}

// The whole wave fills one long token: eight bytes per lane in flight.
template <bool COH, class O>
__device__ inline void fill_wave(const O& out, uint64_t dst, uint64_t src, uint32_t len, uint32_t lane) {
  const uint64_t dist = dst - src;
  const uint64_t step = dist > 64 ? 64 : 64 % uint32_t(dist);  // no 64-bit division
  uint64_t j = dist > lane ? lane : lane % uint32_t(dist);
  for (uint32_t k0 = lane; k0 < len; k0 += 512) {
    uint64_t idx[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      idx[q] = j;
      j += step;
      if (j >= dist) j -= dist;
    }
    uint8_t v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = (k0 + 64 * q < len) ? ldb<COH>(out.at(src + idx[q])) : uint8_t(0);
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (k0 + 64 * q < len) stb<COH>(out.at(dst + k0 + 64 * q), v[q]);
  }
}

constexpr uint32_t kLongToken = 64;     // lane/wave fill: tokens at least this long use the whole wave
constexpr uint32_t kSplitToken = 1024;  // round 0: tokens at least this long get a workgroup each

// Per-wave staging of the ready tokens for the segmented fill.
struct FillStage {
  uint32_t end[64];   // inclusive prefix of lengths (0 for tokens not copied)
  uint32_t len[64];
  uint64_t dst[64];
  uint64_t src[64];
  gbytes out[64];
};

constexpr uint32_t kFillBytes = 8;  // consecutive bytes per lane per pass
enum { kFillLaneWave = 0, kFillSegmented = 1 };

// Segmented periodic fill of this wave's ready tokens: their bytes are laid
// end to end and every lane takes kFillBytes consecutive ones per pass, so a
// pass issues 64 * kFillBytes independent source loads before its stores,
// whatever the mix of short and long tokens.  Byte k of a token comes from
// src + (k mod dist) (dist >= len: a plain copy).
template <bool COH, class O>
__device__ inline void fill_ready(const O& out, bool ready, uint64_t dst, uint64_t src, uint32_t len, int serial,
                                  int fill_mode, FillStage& fs) {
  const uint32_t lane = lane_id();
  if (serial) {
    if (ready) fill_serial<COH>(out, dst, src, len);
    return;
  }
  if (fill_mode == kFillLaneWave) {  // short tokens lane by lane, long ones by the whole wave
    const bool lng = ready && len >= kLongToken;
    if (ready && !lng) fill_lane<COH>(out, dst, src, len);
    uint64_t lm = __ballot(lng);
    while (lm) {
      const int l = __builtin_ctzll(lm);
      lm &= lm - 1;
      const O o = out.with_base(
          reinterpret_cast<gbytes>(__shfl((unsigned long long)reinterpret_cast<uintptr_t>(out.base), l, 64)));
      fill_wave<COH>(o, __shfl((unsigned long long)dst, l, 64), __shfl((unsigned long long)src, l, 64),
                     __shfl(len, l, 64), lane);
    }
    return;
  }
  const uint32_t mine = ready ? len : 0u;
  uint32_t total;
  const uint32_t excl = wave_excl_sum(mine, &total);
  fs.end[lane] = excl + mine;
  fs.len[lane] = mine;
  fs.dst[lane] = dst;
  fs.src[lane] = src;
  fs.out[lane] = out.base;
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  for (uint32_t base = 0; base < total; base += 64 * kFillBytes) {
    const uint32_t f0 = base + lane * kFillBytes;
    uint64_t at[kFillBytes];
    uint64_t to[kFillBytes];
    uint8_t v[kFillBytes];
    if (f0 < total) {
      uint32_t l = 0;  // first token whose end exceeds f0
#pragma unroll
      for (uint32_t step = 32; step; step >>= 1)
        if (fs.end[l + step - 1] <= f0) l += step;
      uint32_t e = fs.end[l], start = e - fs.len[l];
      uint64_t d = fs.dst[l], sr = fs.src[l], dist = d - sr;
      O o = out.with_base(fs.out[l]);
      uint64_t k = f0 - start;  // < 2^16: a token lies inside one block
      uint64_t j = dist > k ? k : uint64_t(uint32_t(k) % uint32_t(dist));
#pragma unroll
      for (uint32_t q = 0; q < kFillBytes; ++q) {
        const uint32_t f = f0 + q;
        if (f < total && f >= e) {  // next token with bytes
          do { ++l; } while (fs.len[l] == 0);
          e = fs.end[l];
          start = e - fs.len[l];
          d = fs.dst[l], sr = fs.src[l], dist = d - sr;
          o = out.with_base(fs.out[l]);
          k = 0, j = 0;
        }
        at[q] = reinterpret_cast<uint64_t>(o.at(sr + j));
        to[q] = f < total ? reinterpret_cast<uint64_t>(o.at(d + k)) : ~0ull;
        ++k;
        if (++j == dist) j = 0;
      }
#pragma unroll
      for (uint32_t q = 0; q < kFillBytes; ++q)
        v[q] = to[q] != ~0ull ? ldb<COH>(reinterpret_cast<const AX_GLOBAL uint8_t*>(at[q])) : uint8_t(0);
#pragma unroll
      for (uint32_t q = 0; q < kFillBytes; ++q)
        if (to[q] != ~0ull) stb<COH>(reinterpret_cast<gbytes>(to[q]), v[q]);
    }
  }
  __builtin_amdgcn_wave_barrier();
}

// Workgroup g of a grid of n is dispatched to XCD g mod 8 (round-robin);
// this gives every XCD a contiguous run of items instead, so neighbouring
// blocks share an L2 (a block's match sources are mostly just behind it).
__device__ inline uint32_t xcd_item(uint32_t g, uint32_t n) {
  const uint32_t x = g & 7u, slot = g >> 3, q = n >> 3, r = n & 7u;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + slot;
}

// ------------------------------------------------ marking for pointer jumping --
//
// In the last bulk round, the tokens still pending (the deep remainder) are
// marked for pointer jumping (see the jump kernels below): every byte of a
// pending token gets its first entry in the jump array — its source position
// src + (k mod dist) by window position (byte o of window block x is
// x * S + o), or the source's value when the source's block is not in the
// window (the byte is final) — and its bit in the leftover map.  A wave lays
// its lanes' pending tokens end to end and takes eight bytes per lane.
constexpr uint32_t kJRes = 0x80000000u;  // entry holds a final byte value (low 8 bits)
constexpr uint32_t kJMarkBytes = 8;
constexpr uint32_t kJLongMark = 256;     // pending tokens at least this long are marked by a workgroup each

struct MarkStage {
  uint32_t end[64];  // inclusive prefix of pending lengths
  uint32_t item[64];
  uint64_t src[64], dst[64];
};

// Window position of the first byte of archive block qb of the job of
// window block wb, or false when that block is not in this window (its bytes
// are final: an earlier window wrote them, or the plan does not decode
// them).
__device__ inline bool window_block(const WinBlock* wbl, uint32_t S, const WinBlock& wb, uint64_t qb, uint32_t& wq) {
  const uint64_t b0 = wbl[wb.first].b;
  uint32_t x;
  if (qb >= b0 && qb - b0 < wb.count && wbl[wb.first + uint32_t(qb - b0)].b == qb) {
    x = wb.first + uint32_t(qb - b0);  // the job's blocks are consecutive up to qb (whole-archive windows)
  } else {
    uint32_t lo = wb.first, hi = wb.first + wb.count;
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (wbl[mid].b < qb) lo = mid + 1; else hi = mid;
    }
    if (lo == wb.first + wb.count || wbl[lo].b != qb) return false;
    x = lo;
  }
  wq = x * S;
  return true;
}

// Whether no match of this window writes a byte of [s0, s1) of the job of
// window block wb (block `item`, whose bytes start at archive position bs):
// those bytes are literals or final, so a token reading them is ready in
// round 0.  Read from the match coverage the parse wrote; bytes of blocks
// outside the window are final or not needed (as for find_cover).
__device__ inline bool sources_literal(const CopyArgs& a, const WinBlock& wb, uint32_t item, uint64_t bs, uint32_t B,
                                       uint64_t s0, uint64_t s1) {
  const uint32_t lb = __builtin_ctz(B);
  while (s0 < s1) {
    const uint64_t qb = s0 >> lb, e = min(s1, (qb + 1) << lb);
    uint32_t wq = item * a.S;
    if (qb == (bs >> lb) || window_block(a.wbl, a.S, wb, qb, wq)) {
      const AX_GLOBAL u32x4* const rec = block_recs(a.cmd, a.S, wq / a.S);
      const uint32_t p0 = uint32_t(s0 & (B - 1)), p1 = p0 + uint32_t(e - s0);  // block positions
      for (uint32_t w = p0 >> 5; w <= (p1 - 1) >> 5; ++w) {
        const uint32_t lo = w == (p0 >> 5) ? (p0 & 31) : 0, hi = w == ((p1 - 1) >> 5) ? ((p1 - 1) & 31) : 31;
        if (rec[w].x & (~0u >> (31 - hi)) & (~0u << lo)) return false;
      }
    }
    s0 = e;
  }
  return true;
}

// Mark this wave's pending tokens (one per lane: `pend`, token t).  `row`:
// when not null, every token lies in window block `row_item` and its bits go
// to that block's LDS row (32-bit words); else to the leftover map with
// global atomics.
template <class O>
__device__ void mark_wave(const CopyArgs& a, bool pend, uint32_t t, MarkStage& ms, uint32_t* row,
                          uint32_t row_item) {
  const uint32_t lane = lane_id();
  uint64_t src = 0, dst = 0;
  uint32_t len = 0;
  if (pend) token_at(a.tok, t, src, dst, len);
  // long tokens of a round over the leftover list are marked by a wave each
  // (k_jmarklong): one wave laying out several would hold up the whole
  // launch (a round-0 workgroup marks at most its own block).  They go to the round's
  // output sublists, which the last round does not otherwise use: token t to
  // sublist (t / 64) mod kSub, so a sublist holds at most ceil(T / 64 / kSub)
  // * 64 of them, and its counter is one of kSub addresses 256 B apart
  const bool lng = pend && len >= kJLongMark && !row;  // a block's own row bounds its work
  if (lng) {
    const uint32_t sub = (t >> 6) % kSub;
    const uint32_t at = atomicAdd(a.cnt_out + sub * kCounterStride, 1u);
    a.list_out[uint64_t(sub) * a.sub_cap + at] = t;
  }
  if (!pend || lng) len = 0;
  uint32_t total;
  const uint32_t ex = wave_excl_sum(len, &total);
  if (!total) return;
  ms.end[lane] = ex + len;
  ms.item[lane] = pend ? a.tblk[t] : 0u;
  ms.src[lane] = src;
  ms.dst[lane] = dst;
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  AX_GLOBAL uint32_t* const J = gp(a.J);
  uint32_t* const lm32 = reinterpret_cast<uint32_t*>(a.lmap);
  for (uint32_t f0 = lane * kJMarkBytes; f0 < total; f0 += 64 * kJMarkBytes) {
    uint32_t l = 0;  // first token whose prefix end exceeds f0
#pragma unroll
    for (uint32_t step = 32; step; step >>= 1)
      if (ms.end[l + step - 1] <= f0) l += step;
    uint32_t e = ms.end[l], item = ms.item[l];
    WinBlock wb = a.wbl[item];
    JobDev jd = a.jobs[wb.job];
    uint64_t bs = wb.b * jd.B;
    uint32_t lb = __builtin_ctz(jd.B);  // block sizes are powers of two
    src = ms.src[l], dst = ms.dst[l];
    uint32_t k = f0 - (l ? ms.end[l - 1] : 0u);
    uint64_t dist = dst - src, j = dist > k ? k : uint64_t(k % uint32_t(dist));
    // window position of the source block last looked up (sources of a run
    // of bytes are consecutive: one lookup per block)
    uint64_t cb = wb.b;
    uint32_t cbase = item * a.S;
    bool cin = true;
    uint32_t mw = ~0u, mbits = 0;  // leftover-map word being gathered and its bits
    for (uint32_t q = 0; q < kJMarkBytes && f0 + q < total; ++q) {
      if (f0 + q >= e) {  // the next pending token
        do { ++l; } while (ms.end[l] == e);
        e = ms.end[l];
        src = ms.src[l], dst = ms.dst[l];
        if (ms.item[l] != item) {
          item = ms.item[l];
          wb = a.wbl[item];
          jd = a.jobs[wb.job];
          bs = wb.b * jd.B;
          lb = __builtin_ctz(jd.B);
        }
        k = 0, j = 0, dist = dst - src;
        cb = wb.b, cbase = item * a.S, cin = true;
      }
      const uint64_t sp = src + j;  // source position
      const uint64_t sb = sp >> lb;
      if (sb != cb) {
        cb = sb;
        cin = window_block(a.wbl, a.S, wb, sb, cbase);
      }
      const uint32_t v = cin ? cbase + uint32_t(sp & (jd.B - 1)) : kJRes | *O(jd).at(sp);
      const uint32_t d = item * a.S + uint32_t(dst - bs) + k;  // this byte's window position
      J[d] = v;
      if ((d >> 5) != mw) {
        if (mbits) {
          if (row) atomicOr(&row[mw - row_item * (a.S / 32)], mbits);
          else atomicOr(&lm32[mw], mbits);
        }
        mw = d >> 5, mbits = 0;
      }
      mbits |= 1u << (d & 31);
      ++k;
      if (++j == dist) j = 0;
    }
    if (mbits) {
      if (row) atomicOr(&row[mw - row_item * (a.S / 32)], mbits);
      else atomicOr(&lm32[mw], mbits);
    }
  }
  __builtin_amdgcn_wave_barrier();  // the stage is read before the caller's next use
}

// Level-synchronous rounds.  A token copied in round r marks done = r; a
// token is ready in round r only if its covering tokens are marked < r, i.e.
// were copied by an earlier launch, so no access within a round races.
//
// Round 0 runs one workgroup per window block, in four passes.  (1) Each
// token's covering range is found; ready tokens (sources all literal bytes,
// or before the window) are noted in LDS with the 16-byte chunks of the block
// they will write, leftovers go to the next round's lists.  (2) Those chunks
// of the block's output (the literals the parse placed) are loaded into an
// LDS tile.  (3) The ready tokens are filled into the tile, sources read from
// global memory where they are final.  (4) The chunks are written back with
// 16-byte stores: the match bytes reach memory as whole chunks instead of
// byte-granular scattered writes, and chunks without match bytes are neither
// read nor written.  Tokens of at least kSplitToken bytes go to k_long.
// Leftovers go to sublist (t / 64) mod kSub, so a sublist holds at most
// ceil(T / 64 / kSub) * 64 tokens.
template <class O, bool kCovMap>
__global__ __launch_bounds__(kCopyThreads) void k_round0(CopyArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t tile[kMaxB];
  __shared__ uint32_t dirty[kMaxB / 16 / 32];  // chunks of the tile that receive match bytes
  __shared__ uint32_t rdy[kMaxB / 32];         // the block's tokens filled here (min_match >= 1)
  // the block's tokens left pending, marked for jumping when round 0 is the
  // only round (the coverage-map instantiation; the other one keeps its LDS
  // for one more resident workgroup)
  __shared__ uint32_t lft[kCovMap ? kMaxB / 32 : 1];
  const uint32_t lane = lane_id(), item = xcd_item(blockIdx.x, gridDim.x);
  const WinBlock wb = a.wbl[item];
  const JobDev& J = a.jobs[wb.job];
  const O out(J);
  const uint32_t B = J.B;
  const uint64_t bs = wb.b * B;
  const gbytes ob = out.at(bs);  // this block's bytes (contiguous)
  const uint32_t blen = uint32_t(min<uint64_t>(B, J.n_bytes - bs));
  const uint32_t nchunk = (blen + 15) / 16;
  const uint32_t t1 = item + 1 < a.n_items ? a.wbl[item + 1].tok : a.n_tok;
  const uint32_t ntb = t1 - wb.tok;  // <= blen: tokens are at least a byte long
  // the status is checked once the block's own loads are in flight
  if (__hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  if (blockIdx.x == 0 && threadIdx.x < kSub) a.cnt_clear[threadIdx.x * kCounterStride] = 0;
  // the serial ablation reads in-block sources back from the tile: load all of it
  for (uint32_t k = threadIdx.x; k < kMaxB / 16 / 32; k += kCopyThreads) dirty[k] = a.serial ? ~0u : 0u;
  for (uint32_t k = threadIdx.x; k < (ntb + 31) / 32; k += kCopyThreads) {
    rdy[k] = 0;
    if (kCovMap) lft[k] = 0;
  }
  __syncthreads();
  for (uint32_t base = wb.tok; base < t1; base += kCopyThreads) {
    const uint32_t t = base + threadIdx.x;
    const bool act = t < t1;
    uint64_t src = 0, dst = 0;
    uint32_t len = 0;
    bool ready = false;
    if (act) {
      token_at(a.tok, t, src, dst, len);
      const uint64_t dist = dst - src, s1 = src + (dist < len ? dist : len);
      if (kCovMap) {  // the only round: readiness from the coverage map, covers when first needed
        ready = sources_literal(a, wb, item, bs, B, src, s1);
        if (!ready) a.cov[2 * t + 1] = kCovLazy;
      } else {
        uint32_t lo, cnt;
        find_cover(a, wb, B, src, s1, lo, cnt);
        a.cov[2 * t] = lo;
        a.cov[2 * t + 1] = cnt;
        ready = cnt == 0;
      }
    }
    const bool split = ready && !a.serial && len >= kSplitToken;
    const uint64_t sm = __ballot(split);
    if (sm) {
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(a.long_cnt, uint32_t(__popcll(sm)));
      at = __shfl(at, 0, 64);
      if (split) a.long_list[at + lanes_below(sm)] = t;
    }
    if (ready && !split) {
      a.done[t] = 0;
      const uint32_t r = t - wb.tok, drel = uint32_t(dst - bs);
      atomicOr(&rdy[r >> 5], 1u << (r & 31));
      const uint32_t c0 = drel >> 4, c1 = (drel + len - 1) >> 4;  // len < kSplitToken: a few words
      for (uint32_t w = c0 >> 5; w <= c1 >> 5; ++w) {
        const uint32_t lo_b = w == (c0 >> 5) ? (c0 & 31) : 0, hi_b = w == (c1 >> 5) ? (c1 & 31) : 31;
        atomicOr(&dirty[w], (hi_b == 31 ? ~0u : (2u << hi_b) - 1) & ~((1u << lo_b) - 1));
      }
    }
    const bool left = act && !ready;
    if (a.mark) {  // the only round: leftovers stay pending (listed, or marked after the fills)
      if (left && a.mark == kMarkList) atomicOr(a.pbits + (t >> 5), 1u << (t & 31));
      if (kCovMap && left && a.mark == kMarkJump) atomicOr(&lft[(t - wb.tok) >> 5], 1u << ((t - wb.tok) & 31));
      continue;
    }
    // a wave's tokens fall in at most two 64-token groups, hence two
    // sublists: the first lane of each group reserves its group's places, both
    // in one atomic instruction
    const uint32_t g0 = (base + (threadIdx.x & ~63u)) >> 6;
    const bool in0 = left && (t >> 6) == g0, in1 = left && (t >> 6) == g0 + 1;
    const uint64_t m0 = __ballot(in0), m1 = __ballot(in1);
    if (m0 | m1) {
      const uint32_t f0 = m0 ? uint32_t(__builtin_ctzll(m0)) : 64u, f1 = m1 ? uint32_t(__builtin_ctzll(m1)) : 64u;
      const uint32_t sub0 = g0 % kSub, sub1 = (g0 + 1) % kSub;
      uint32_t at = 0;
      if (lane == f0 || lane == f1) {  // a lane is in at most one group
        const bool h = lane == f1;
        at = atomicAdd(a.cnt_out + (h ? sub1 : sub0) * kCounterStride, uint32_t(__popcll(h ? m1 : m0)));
      }
      const uint32_t at0 = __shfl(at, int(f0 & 63u), 64), at1 = __shfl(at, int(f1 & 63u), 64);
      if (in0) a.list_out[uint64_t(sub0) * a.sub_cap + at0 + lanes_below(m0)] = t;
      if (in1) a.list_out[uint64_t(sub1) * a.sub_cap + at1 + lanes_below(m1)] = t;
    }
  }
  __syncthreads();
  const uint32_t full = blen / 16;
  for (uint32_t k = threadIdx.x; k < nchunk; k += kCopyThreads) {
    if (!((dirty[k >> 5] >> (k & 31)) & 1)) continue;
    if (k < full) {
      *reinterpret_cast<u32x4*>(tile + 16 * k) = *reinterpret_cast<const AX_GLOBAL u32x4*>(ob + 16 * k);
    } else {
      for (uint32_t i = 16 * k; i < blen; ++i) tile[i] = ob[i];
    }
  }
  __syncthreads();
  for (uint32_t base = wb.tok; base < t1; base += kCopyThreads) {
    const uint32_t t = base + threadIdx.x;
    const uint32_t r = t - wb.tok;
    const bool ready = t < t1 && ((rdy[r >> 5] >> (r & 31)) & 1);
    if (!__ballot(ready)) continue;
    uint64_t src = 0, dst = 0;
    uint32_t len = 0;
    if (ready) token_at(a.tok, t, src, dst, len);
    // tile fill: out[dst + k] = out[src + (k mod dist)], destination in the tile
    const bool mine = ready && (a.serial || len < kLongToken);
    const uint32_t drel = uint32_t(dst - bs);
    if (mine && a.serial) {  // the ablation: byte after byte, in-block sources read back from the tile
      for (uint32_t k = 0; k < len; ++k) {
        const uint64_t p = src + k;
        tile[drel + k] = p < bs ? *out.at(p) : tile[p - bs];
      }
    } else if (mine) {
      const uint64_t dist = dst - src;
      uint64_t j = 0;
      for (uint32_t k0 = 0; k0 < len; k0 += 16) {
        if (src + k0 + 16 <= dst && out.contiguous(src + k0, 16)) {  // 16 source bytes before the destination: one unaligned load
          const u32x4 v = *reinterpret_cast<const AX_GLOBAL u32x4_u*>(out.at(src + k0));
#pragma unroll
          for (uint32_t q = 0; q < 16; ++q)
            if (k0 + q < len) tile[drel + k0 + q] = uint8_t(v[q >> 2] >> (8 * (q & 3)));
          j = k0 + 16 == dist ? 0 : k0 + 16;  // dist >= k0 + 16: the periodic index of the next byte
          continue;
        }
        uint64_t idx[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          idx[q] = j;
          if (++j == dist) j = 0;
        }
        uint8_t v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = (k0 + q < len) ? *out.at(src + idx[q]) : uint8_t(0);
#pragma unroll
        for (int q = 0; q < 16; ++q)
          if (k0 + q < len) tile[drel + k0 + q] = v[q];
      }
    }
    uint64_t wm = __ballot(ready && !mine);  // medium tokens: the whole wave each
    while (wm) {
      const int l = __builtin_ctzll(wm);
      wm &= wm - 1;
      const uint64_t s0 = __shfl((unsigned long long)src, l, 64);
      const uint32_t d0 = __shfl(drel, l, 64), n0 = __shfl(len, l, 64);
      const uint64_t dist = bs + d0 - s0;
      const uint32_t dd = dist < n0 ? uint32_t(dist) : n0;  // the period (n0 when it never wraps)
      const uint32_t step = 64 % dd;
      uint32_t j = lane % dd;
      for (uint32_t k0 = lane; k0 < n0; k0 += 512) {  // eight source loads in flight per lane
        uint32_t jj[8];
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
          jj[q] = j;
          j += step;
          if (j >= dd) j -= dd;
        }
        uint8_t v[8];
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) v[q] = k0 + 64 * q < n0 ? *out.at(s0 + jj[q]) : uint8_t(0);
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q)
          if (k0 + 64 * q < n0) tile[d0 + k0 + 64 * q] = v[q];
      }
    }
  }
  __syncthreads();
  for (uint32_t k = threadIdx.x; k < nchunk; k += kCopyThreads) {
    if (!((dirty[k >> 5] >> (k & 31)) & 1)) continue;
    if (k < full) {
      *reinterpret_cast<AX_GLOBAL u32x4*>(ob + 16 * k) = *reinterpret_cast<const u32x4*>(tile + 16 * k);
    } else {
      for (uint32_t i = 16 * k; i < blen; ++i) ob[i] = tile[i];
    }
  }
  if (!kCovMap || a.mark != kMarkJump) return;
  // the block's pending tokens, marked for pointer jumping: the tile's bytes
  // now hold the block's leftover-map row and the waves' stages
  __syncthreads();
  uint32_t* const row = reinterpret_cast<uint32_t*>(tile);
  MarkStage* const mst = reinterpret_cast<MarkStage*>(tile + kMaxB / 8);
  static_assert(kMaxB / 8 + (kCopyThreads / 64) * sizeof(MarkStage) <= kMaxB, "marking fits the tile");
  for (uint32_t k = threadIdx.x; k < a.S / 32; k += kCopyThreads) row[k] = 0;
  __syncthreads();
  for (uint32_t base = wb.tok; base < t1; base += kCopyThreads) {
    const uint32_t t = base + threadIdx.x, r = t - wb.tok;
    const bool pend = t < t1 && ((lft[r >> 5] >> (r & 31)) & 1);
    mark_wave<O>(a, pend, t, mst[threadIdx.x >> 6], row, item);
  }
  __syncthreads();
  uint32_t* const lm = reinterpret_cast<uint32_t*>(a.lmap) + uint64_t(item) * (a.S / 32);
  for (uint32_t k = threadIdx.x; k < a.S / 32; k += kCopyThreads) lm[k] = row[k];
}

// Round 0 as a flat grid over the window's tokens (the alternative
// schedule): 64 consecutive tokens per wave, fills written straight to
// global memory by the wave (short tokens a lane each, long ones the wave,
// or all laid end to end over the lanes).  Same results and lists as
// k_round0; the leftovers of a wave (64-aligned tokens) fall in one 64-token
// group and so in one sublist.
template <class O>
__global__ __launch_bounds__(kCopyThreads) void k_round0_waves(CopyArgs a) {
  __shared__ FillStage stage[kCopyThreads / 64];
  __shared__ MarkStage mstage[kCopyThreads / 64];
  if (__hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  const uint32_t lane = lane_id();
  FillStage& fs = stage[threadIdx.x >> 6];
  if (blockIdx.x == 0 && threadIdx.x < kSub) a.cnt_clear[threadIdx.x * kCounterStride] = 0;
  for (uint64_t base = uint64_t(blockIdx.x) * kCopyThreads; base < a.n_tok; base += uint64_t(gridDim.x) * kCopyThreads) {
    const uint32_t t = uint32_t(base + threadIdx.x);
    const bool act = t < a.n_tok;
    uint64_t src = 0, dst = 0;
    uint32_t len = 0, lo = 0, cnt = 0;
    O out(a.jobs[0]);
    if (act) {
      token_at(a.tok, t, src, dst, len);
      const WinBlock wb = a.wbl[a.tblk[t]];
      const JobDev& J = a.jobs[wb.job];
      out = O(J);
      const uint64_t dist = dst - src;
      find_cover(a, wb, J.B, src, src + (dist < len ? dist : len), lo, cnt);
      a.cov[2 * t] = lo;
      a.cov[2 * t + 1] = cnt;
    }
    const bool ready = act && cnt == 0;
    const bool split = ready && !a.serial && len >= kSplitToken;
    const uint64_t sm = __ballot(split);
    if (sm) {
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(a.long_cnt, uint32_t(__popcll(sm)));
      at = __shfl(at, 0, 64);
      if (split) a.long_list[at + lanes_below(sm)] = t;
    }
    fill_ready<false>(out, ready && !split, dst, src, len, a.serial, a.fill_round, fs);
    if (ready && !split) a.done[t] = 0;
    const bool left = act && !ready;
    if (a.mark) {
      if (left && a.mark == kMarkList) atomicOr(a.pbits + (t >> 5), 1u << (t & 31));
      if (a.mark == kMarkJump) mark_wave<O>(a, left, t, mstage[threadIdx.x >> 6], nullptr, 0);
      continue;
    }
    const uint64_t m = __ballot(left);
    if (m) {
      const uint32_t sub = (t >> 6) % kSub;  // the same for the whole wave
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(a.cnt_out + sub * kCounterStride, uint32_t(__popcll(m)));
      at = __shfl(at, 0, 64);
      if (left) a.list_out[uint64_t(sub) * a.sub_cap + at + lanes_below(m)] = t;
    }
  }
}

// Later rounds visit the previous round's leftovers.  Leftovers go to this
// workgroup's sublist (counters spread over kSub addresses), or, in the last
// round, to the bitmap of the persistent launch.
template <class O>
__global__ __launch_bounds__(kCopyThreads) void k_round(CopyArgs a) {
  __shared__ FillStage stage[kCopyThreads / 64];
  __shared__ MarkStage mstage[kCopyThreads / 64];
  __shared__ uint32_t sub_end[kSub];  // inclusive prefix of the input sublist lengths
  const uint32_t lane = lane_id();
  FillStage& fs = stage[threadIdx.x >> 6];
  // the status is checked once the counters' loads are in flight
  const uint32_t c_in = threadIdx.x < 64 ? a.cnt_in[threadIdx.x * kCounterStride] : 0u;
  if (__hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  if (blockIdx.x == 0 && threadIdx.x < kSub) a.cnt_clear[threadIdx.x * kCounterStride] = 0;
  if (threadIdx.x < 64) {
    uint32_t tot;
    sub_end[threadIdx.x] = wave_excl_sum(c_in, &tot) + c_in;
  }
  __syncthreads();
  const uint32_t n_items = sub_end[kSub - 1];
  const uint32_t my_sub = blockIdx.x % kSub;
  for (uint64_t base = uint64_t(blockIdx.x) * kCopyThreads; base < n_items; base += uint64_t(gridDim.x) * kCopyThreads) {
    const uint64_t item = base + threadIdx.x;
    const bool act = item < n_items;
    uint32_t t = 0;
    if (act) {  // sublist holding item
      uint32_t sl = 0;
#pragma unroll
      for (uint32_t step = 32; step; step >>= 1)
        if (sub_end[sl + step - 1] <= item) sl += step;
      const uint32_t start = sub_end[sl] - (sl ? sub_end[sl] - sub_end[sl - 1] : sub_end[0]);
      t = a.list_in[uint64_t(sl) * a.sub_cap + (item - start)];
    }
    uint64_t src = 0, dst = 0;
    uint32_t len = 0, lo = 0, cnt = 0;
    O out(a.jobs[0]);
    if (act) {
      token_at(a.tok, t, src, dst, len);
      if (!a.one_job) out = token_out<O>(a, t);
      cover_of(a, t, src, dst, len, lo, cnt);
    }
    // the covering tokens' done flags, four loads in flight at a time
    bool ready = act;
    for (uint32_t i0 = 0; i0 < cnt && ready; i0 += 4) {
      uint8_t f[4];
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) f[q] = i0 + q < cnt ? a.done[lo + i0 + q] : uint8_t(0);
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) ready = ready && f[q] < a.round;
    }
    fill_ready<false>(out, ready, dst, src, len, a.serial, a.fill_round, fs);
    if (ready) a.done[t] = uint8_t(a.round);
    const bool left = act && !ready;
    if (a.mark) {
      if (left && a.mark == kMarkList) atomicOr(a.pbits + (t >> 5), 1u << (t & 31));
      if (a.mark == kMarkJump) mark_wave<O>(a, left, t, mstage[threadIdx.x >> 6], nullptr, 0);
      continue;
    }
    const uint64_t m = __ballot(left);
    if (m) {
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(a.cnt_out + my_sub * kCounterStride, uint32_t(__popcll(m)));
      at = __shfl(at, 0, 64);
      if (left) a.list_out[uint64_t(my_sub) * a.sub_cap + at + lanes_below(m)] = t;
    }
  }
}

// Round 0's long tokens: one workgroup per token, sixteen bytes per thread
// in flight; the token is marked done (round 0) once the whole group is
// through.
template <class O>
__global__ __launch_bounds__(kCopyThreads) void k_long(CopyArgs a) {
  if (__hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  const uint32_t n = *a.long_cnt;
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const uint32_t t = a.long_list[i];
    uint64_t src, dst;
    uint32_t len;
    token_at(a.tok, t, src, dst, len);
    const O out = token_out<O>(a, t);
    const uint64_t dist = dst - src;
    const uint64_t step = dist > kCopyThreads ? kCopyThreads : kCopyThreads % uint32_t(dist);
    uint64_t j = dist > threadIdx.x ? threadIdx.x : threadIdx.x % uint32_t(dist);
    for (uint32_t k0 = threadIdx.x; k0 < len; k0 += 16 * kCopyThreads) {
      uint64_t idx[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        idx[q] = j;
        j += step;
        if (j >= dist) j -= dist;
      }
      uint8_t v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = (k0 + kCopyThreads * q < len) ? *out.at(src + idx[q]) : uint8_t(0);
#pragma unroll
      for (int q = 0; q < 16; ++q)
        if (k0 + kCopyThreads * q < len) *out.at(dst + k0 + kCopyThreads * q) = v[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) a.done[t] = 0;
  }
}

// Compaction of the last round's leftovers into an ascending list: per
// workgroup of 1024 bitmap words, a population count, then the scatter.
constexpr uint32_t kPackWords = 4 * kCopyThreads;

__device__ inline uint32_t block_sum_u32(uint32_t v, uint32_t* red) {
  uint32_t tot;
  const uint32_t ex = wave_excl_sum(v, &tot);
  (void)ex;
  if (lane_id() == 0) red[threadIdx.x >> 6] = tot;
  __syncthreads();
  uint32_t s = 0;
  for (uint32_t k = 0; k < kCopyThreads / 64; ++k) s += red[k];
  __syncthreads();
  return s;
}

__global__ __launch_bounds__(kCopyThreads) void k_pcount(const uint32_t* pbits, uint32_t n_words, uint32_t* pcnt) {
  __shared__ uint32_t red[kCopyThreads / 64];
  uint32_t c = 0;
  for (uint32_t k = 0; k < 4; ++k) {
    const uint32_t w = blockIdx.x * kPackWords + k * kCopyThreads + threadIdx.x;
    if (w < n_words) c += __popc(pbits[w]);
  }
  const uint32_t s = block_sum_u32(c, red);
  if (threadIdx.x == 0) pcnt[blockIdx.x] = s;
}

__global__ __launch_bounds__(kCopyThreads) void k_pscatter(const uint32_t* pbits, uint32_t n_words,
                                                           const uint32_t* pcnt, uint32_t* plist, DevStatus* st) {
  __shared__ uint32_t red[kCopyThreads / 64];
  uint32_t before = 0;
  for (uint32_t g = threadIdx.x; g < blockIdx.x; g += kCopyThreads) before += pcnt[g];
  const uint32_t base = block_sum_u32(before, red);
  // thread i takes words 4i..4i+3 of the workgroup's range (consecutive)
  uint32_t wv[4], c = 0;
  const uint32_t w0 = blockIdx.x * kPackWords + 4 * threadIdx.x;
  for (uint32_t k = 0; k < 4; ++k) {
    wv[k] = w0 + k < n_words ? pbits[w0 + k] : 0u;
    c += __popc(wv[k]);
  }
  uint32_t wtot;
  const uint32_t wex = wave_excl_sum(c, &wtot);
  if (lane_id() == 0) red[threadIdx.x >> 6] = wtot;
  __syncthreads();
  uint32_t at = base + wex;
  for (uint32_t k = 0; k < (threadIdx.x >> 6); ++k) at += red[k];
  for (uint32_t k = 0; k < 4; ++k) {
    uint32_t bits = wv[k];
    while (bits) {
      const uint32_t j = __builtin_ctz(bits);
      bits &= bits - 1;
      plist[at++] = (w0 + k) * 32 + j;
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kCopyThreads - 1) st->n_pending = at;
}

// Persistent finish over the compacted leftovers: 64-token chunks of the
// ascending list by ticket; each wave polls its unfinished tokens' covering
// tokens and copies a token once they are all done.  Output bytes and done
// flags use agent-coherent accesses and a store-completion wait precedes
// each done flag, so a flag seen by another XCD implies its bytes are visible
// there.  A token waits only on lower-indexed tokens, which are done or sit
// in lower chunks whose tickets running waves hold, so every wait ends.
template <class O>
__global__ __launch_bounds__(kCopyThreads) void k_tail(CopyArgs a) {
  __shared__ FillStage stage[kCopyThreads / 64];
  const uint32_t lane = lane_id();
  FillStage& fs = stage[threadIdx.x >> 6];
  if (__hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  const uint32_t per = a.tail_chunks;  // consecutive chunks per ticket
  const uint32_t n_pend = a.st->n_pending;
  const uint32_t n_chunks = (n_pend + 63) / 64;
  const uint32_t n_tickets = (n_chunks + per - 1) / per;
  for (;;) {
    uint32_t tk = 0;
    if (lane == 0) tk = atomicAdd(&a.st->ticket, 1u);
    tk = __shfl(tk, 0, 64);
    if (tk >= n_tickets) return;
    for (uint32_t chunk = tk * per; chunk < min(tk * per + per, n_chunks); ++chunk) {
      const uint32_t li = chunk * 64 + lane;
      const uint32_t t = li < n_pend ? a.plist[li] : 0u;
      bool pending = li < n_pend;
      if (!__ballot(pending)) continue;
      uint64_t src = 0, dst = 0;
      uint32_t len = 0, lo = 0, cnt = 0;
      O out(a.jobs[0]);
      if (pending) {
        token_at(a.tok, t, src, dst, len);
        out = token_out<O>(a, t);
        cover_of(a, t, src, dst, len, lo, cnt);
      }
      uint64_t spins = 0;
      while (__ballot(pending)) {
        // flags are read relaxed; an agent-scope acquire fence after a flag
        // that reads a producer's store synchronises with the producer's
        // agent-scope release fence before that store, so the bytes it
        // filled are visible to the loads after the fence, on any XCD
        bool ready = pending;
        for (uint32_t i = 0; i < cnt && ready; ++i)
          ready = __hip_atomic_load(a.done + lo + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != kPending;
        if (__ballot(ready)) {
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          fill_ready<true>(out, ready, dst, src, len, a.serial, a.fill_tail, fs);
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
          if (ready) __hip_atomic_store(a.done + t, uint8_t(a.round), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          pending = pending && !ready;
        } else {
          __builtin_amdgcn_s_sleep(1);
          if (++spins > a.spin_limit ||
              ((spins & 63) == 0 && __hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
            if (lane == 0 && spins > a.spin_limit) report(a.st, AX_E_DEVICE, ~0ull);
            return;
          }
        }
      }
    }
  }
}

// ------------------------------------------- deep remainder: pointer jumping --
//
// The tokens the bulk rounds leave pending (the deep remainder) are resolved
// by pointer jumping over their bytes rather than by a chase of one
// dependency hop at a time.  Positions are window-relative: byte o of window
// block x is x * S + o (S = the largest block size of the plan), so every
// byte of every archive block the window holds has a place in one array of
// 32-bit entries (the jump array) and one bit in each of two bitmaps: the
// leftover map (bytes written by pending tokens) and the active map
// (leftover bytes whose value is not known yet).  An entry holds either the
// window position its value comes from or, with kJRes set, the final byte
// value.  Byte k of a pending token (dst, src, len) takes its value from
// position src + (k mod dist), which lies below dst: a final byte (a
// literal, a token a round copied, a byte of an earlier window or of a block
// the plan does not decode) or a byte of another, earlier pending token.
// Entries therefore form a forest rooted at final values.  A pass replaces
// each active entry by the entry its entry names, twice over (three times
// the hops per pass), so about log3(chain length) passes resolve every
// chain; a gather then writes the leftover bytes as whole 16-byte chunks.
// Updating entries in place is safe in any order: an entry always names a
// byte holding the same value, and every read returns some complete entry.
constexpr uint32_t kJPasses = 32;        // pass-flag slots
constexpr uint32_t kJShards = 16;        // flag words per pass (workgroup g writes g mod 16)
constexpr uint32_t kJFlagStride = 16;    // u32 between two flag words
constexpr uint32_t kJMaxGrid = 8192;     // workgroups of a position-driven launch
constexpr uint32_t kJChaseLimit = 1u << 24;  // hops the gather follows before it reports a device error

struct JumpArgs {
  const JobDev* jobs;
  const WinBlock* wbl;
  uint32_t n_items;    // window blocks
  uint32_t n_tok;      // window tokens
  uint32_t S;          // position stride of a window block
  const uint64_t* tok;
  const uint32_t* tblk;
  const uint8_t* done;
  uint32_t* J;         // one entry per window position
  uint64_t* lmap;      // leftover map, one bit per window position
  uint64_t* amap;      // active map
  uint32_t* flags;     // kJPasses x kJShards words, kJFlagStride apart
  uint8_t** ibase;     // per window block: where its output bytes start
  uint32_t s_log2;     // log2 S
  const uint32_t* llist;  // long pending tokens: kSub sublists of sub_cap
  const uint32_t* lcnt;   // their counters, kCounterStride apart
  uint32_t sub_cap;
  uint32_t* wlist;     // leftover-map words with bits set
  DevStatus* st;
  uint32_t pass;
};

__device__ inline bool jump_failed(const DevStatus* st) {
  return __hip_atomic_load(&st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// An entry naming no leftover byte (cannot happen for entries the init
// wrote): the decode reports a device error instead of following it.
// `where` (recorded as the failing block, with the top bit set) names the
// check: 1 settling the first entries, 2 a pass, 3 the gather.
__device__ inline uint32_t jump_broken(DevStatus* st, uint32_t where) {
  report(st, AX_E_DEVICE, (1ull << 63) | where);
  return kJRes;
}

// Long pending tokens: one workgroup per token, byte k of the token on lane
// k mod 256 (first entries as in the marking of a round, bits by global
// atomics).
template <class O>
__global__ __launch_bounds__(kCopyThreads) void k_jmarklong(JumpArgs a) {
  __shared__ uint32_t sub_end[kSub];  // inclusive prefix of the sublist lengths
  if (jump_failed(a.st)) return;
  if (threadIdx.x < 64) {
    uint32_t tot;
    const uint32_t c = a.lcnt[threadIdx.x * kCounterStride];
    sub_end[threadIdx.x] = wave_excl_sum(c, &tot) + c;
  }
  __syncthreads();
  const uint32_t n = sub_end[kSub - 1], lane = threadIdx.x;  // the workgroup's lanes share a token
  AX_GLOBAL uint32_t* const J = gp(a.J);
  uint32_t* const lm32 = reinterpret_cast<uint32_t*>(a.lmap);
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    uint32_t sl = 0;  // sublist holding item i
#pragma unroll
    for (uint32_t step = 32; step; step >>= 1)
      if (sub_end[sl + step - 1] <= i) sl += step;
    const uint32_t start = sl ? sub_end[sl - 1] : 0u;
    const uint32_t t = a.llist[uint64_t(sl) * a.sub_cap + (i - start)];
    uint64_t src, dst;
    uint32_t len;
    token_at(a.tok, t, src, dst, len);
    const uint32_t item = a.tblk[t];
    const WinBlock wb = a.wbl[item];
    const JobDev jd = a.jobs[wb.job];
    const uint32_t lb = __builtin_ctz(jd.B);
    const uint64_t bs = wb.b << lb, dist = dst - src;
    uint64_t cb = ~0ull;  // the source block last looked up, kept over the lane's passes
    uint32_t cbase = 0;
    bool cin = false;
    // byte k of the token goes to lane k mod 256, so each wave store covers
    // 64 consecutive entries; a wave's 64 positions meet at most three words
    // of the leftover map, set by three lanes from the wave's ballot
    const uint32_t d0 = item * a.S + uint32_t(dst - bs);  // window position of the token's first byte
    const bool wrap = dist < len;                          // a periodic fill: sources repeat every dist bytes
    const uint32_t per = wrap ? uint32_t(dist) : 0u;
    const uint32_t jstep = wrap ? kCopyThreads % per : kCopyThreads;
    uint32_t j = wrap ? lane % per : lane;  // source index of byte k
    const uint32_t wl = lane & 63u, wofs = lane & ~63u;
    for (uint32_t kb = 0; kb < len; kb += kCopyThreads) {
      const uint32_t k = kb + lane;
      const bool valid = k < len;
      if (valid) {
        const uint64_t sp = src + j, sb = sp >> lb;
        if (sb != cb) cb = sb, cin = window_block(a.wbl, a.S, wb, sb, cbase);
        J[d0 + k] = cin ? cbase + uint32_t(sp & (jd.B - 1)) : kJRes | *O(jd).at(sp);
      }
      const uint64_t m = __ballot(valid);
      if (m && wl < 3) {
        const uint32_t p0 = d0 + kb + wofs, off = p0 & 31u;  // the wave's first position
        uint32_t bits;
        if (wl == 0) bits = uint32_t(m << off);
        else if (wl == 1) bits = off ? uint32_t(m >> (32 - off)) : uint32_t(m >> 32);
        else bits = off ? uint32_t(m >> (64 - off)) : 0u;
        if (bits) atomicOr(&lm32[(p0 >> 5) + wl], bits);
      }
      j += jstep;
      if (wrap && j >= per) j -= per;
    }
  }
}

// The work list: the leftover-map words with bits set, in one pass (each
// workgroup takes kJListWords words, finds its busy ones and appends them at
// a place reserved with one atomic add; the list is in no particular order,
// which the walks below do not need).  When more than a quarter of the map's words are busy
// the kernels below walk the whole map instead (dense).
constexpr uint32_t kJListWords = 16 * kCopyThreads;
__device__ inline bool jump_dense(const JumpArgs& a, uint32_t n_words) {
  return uint64_t(n_words) * 4 > uint64_t(a.n_items) * (a.S / 64);
}

__global__ __launch_bounds__(kCopyThreads) void k_jlist(JumpArgs a) {
  __shared__ uint32_t wtot[kCopyThreads / 64];
  __shared__ uint32_t base;
  if (jump_failed(a.st)) return;
  const uint64_t words = uint64_t(a.n_items) * (a.S / 64), w0 = uint64_t(blockIdx.x) * kJListWords;
  constexpr uint32_t kPer = kJListWords / kCopyThreads;  // words per thread, kCopyThreads apart (coalesced reads)
  uint32_t bits = 0, c = 0;
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint64_t g = w0 + q * kCopyThreads + threadIdx.x;
    if (g < words && a.lmap[g] != 0) bits |= 1u << q, ++c;
  }
  uint32_t tot;
  const uint32_t ex = wave_excl_sum(c, &tot);
  if (lane_id() == 0) wtot[threadIdx.x >> 6] = tot;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t all = 0;
    for (uint32_t k = 0; k < kCopyThreads / 64; ++k) all += wtot[k];
    base = all ? atomicAdd(&a.st->n_jwords, all) : 0u;
  }
  __syncthreads();
  uint32_t at = base + ex;
  for (uint32_t k = 0; k < (threadIdx.x >> 6); ++k) at += wtot[k];
  while (bits) {
    const uint32_t q = __builtin_ctz(bits);
    bits &= bits - 1;
    a.wlist[at++] = uint32_t(w0 + q * kCopyThreads + threadIdx.x);
  }
}

// The position-driven kernels below visit the leftover-map words with bits
// set, eight at a time, one position per lane, so the map's rows are read
// and written as coalesced 256-byte rows.  Two walks, chosen per window by
// the list build: when more than a quarter of the map's words are busy, a
// wave reads 64 map words per step (four 16-word chunks a grid apart, so a
// dense region spreads over many waves) and takes the busy ones eight at a
// time; otherwise the work list is walked eight words per step (the next
// step's words in flight), so a sparse map costs no empty reads.
constexpr uint32_t kJStepWords = 8;
constexpr uint32_t kJChunk = 16;

// A group of up to kJStepWords busy map words: their indices and bits
// (wave-uniform, held in scalar registers; bits 0 marks an unused slot).
struct WordGroup {
  uint32_t g[kJStepWords];
  uint64_t wv[kJStepWords];
};

// (the builtin returns int: widen through uint32_t, not by sign extension)
__device__ inline uint64_t uniform64(uint64_t v) {
  return uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v))))) |
         (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v >> 32))))) << 32);
}

// Call f(group) for groups of up to kJStepWords busy words of `map` (the
// leftover or the active map).
template <class F>
__device__ inline void walk_words(const JumpArgs& a, const uint64_t* map, F&& f) {
  const uint32_t lane = lane_id();
  const uint64_t waves = uint64_t(gridDim.x) * (kCopyThreads / 64);
  const uint64_t wave = uint64_t(blockIdx.x) * (kCopyThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t n = a.st->n_jwords;
  WordGroup w;
  if (jump_dense(a, n)) {
    const uint64_t words = uint64_t(a.n_items) * (a.S / 64);
    const uint64_t steps = (words + kJChunk * 4 * waves - 1) / (kJChunk * 4 * waves);
    for (uint64_t i = 0; i < steps; ++i) {
      // lane l reads word l mod 16 of chunk (4 i + l / 16) * waves + wave
      const uint64_t mine = ((i * 4 + (lane >> 4)) * waves + wave) * kJChunk + (lane & 15u);
      const uint64_t mw = mine < words ? map[mine] : 0ull;
      uint64_t nz = uniform64(__ballot(mw != 0));
      while (nz) {
#pragma unroll
        for (uint32_t u = 0; u < kJStepWords; ++u) {
          w.g[u] = 0;
          w.wv[u] = 0;
          if (nz) {
            const uint32_t wi = uint32_t(__builtin_ctzll(nz));
            nz &= nz - 1;
            w.wv[u] = uniform64(__shfl((unsigned long long)mw, int(wi), 64));
            w.g[u] = uint32_t(((i * 4 + (wi >> 4)) * waves + wave) * kJChunk + (wi & 15u));
          }
        }
        f(w);
      }
    }
    return;
  }
  for (uint64_t i0 = wave * kJStepWords; i0 < n; i0 += waves * kJStepWords) {
#pragma unroll
    for (uint32_t u = 0; u < kJStepWords; ++u) {
      w.g[u] = i0 + u < n ? a.wlist[i0 + u] : 0u;
      w.wv[u] = i0 + u < n ? map[w.g[u]] : 0ull;
    }
    f(w);
  }
}

// Value of the byte at window position v (a final byte).
__device__ inline uint32_t jbyte(const JumpArgs& a, uint32_t v) {
  return gp(a.ibase[v >> a.s_log2])[v & ((1u << a.s_log2) - 1u)];
}

// First entries, settled: an entry naming a position outside the leftover
// map (a final byte) takes that byte's value; the rest stay active.
__global__ __launch_bounds__(kCopyThreads) void k_jinit(JumpArgs a) {
  if (jump_failed(a.st)) return;
  const uint32_t lane = lane_id(), limit = a.n_items * a.S;
  AX_GLOBAL uint32_t* const J = gp(a.J);
  walk_words(a, a.lmap, [&](const WordGroup& w) __attribute__((always_inline)) {
    const uint32_t* const g = w.g;
    const uint64_t* const wv = w.wv;
    uint32_t v[kJStepWords];
#pragma unroll
    for (uint32_t u = 0; u < kJStepWords; ++u) v[u] = ((wv[u] >> lane) & 1) ? J[g[u] * 64 + lane] : kJRes;
    bool leftover[kJStepWords];
#pragma unroll
    for (uint32_t u = 0; u < kJStepWords; ++u) {
      leftover[u] = true;
      if (!(v[u] & kJRes)) {
        if (v[u] >= limit) v[u] = jump_broken(a.st, 1);
        else leftover[u] = (a.lmap[v[u] >> 6] >> (v[u] & 63)) & 1;
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < kJStepWords; ++u)
      if (!leftover[u]) v[u] = kJRes | jbyte(a, v[u]);
#pragma unroll
    for (uint32_t u = 0; u < kJStepWords; ++u) {
      if (!wv[u]) continue;
      const bool act = (wv[u] >> lane) & 1;
      if (act && !leftover[u]) J[g[u] * 64 + lane] = v[u];
      const uint64_t still = __ballot(act && !(v[u] & kJRes));
      if (lane == 0) a.amap[g[u]] = still;
    }
  });
  // the dense walk visits only busy words: the others' active bits are zero
  if (jump_dense(a, a.st->n_jwords)) {
    const uint64_t words = uint64_t(a.n_items) * (a.S / 64);
    for (uint64_t w = uint64_t(blockIdx.x) * kCopyThreads + threadIdx.x; w < words;
         w += uint64_t(gridDim.x) * kCopyThreads)
      if (!a.lmap[w]) a.amap[w] = 0;
  }
}

// One jump pass: every active entry takes the entry two steps along its
// chain.  A pass whose predecessor left nothing active exits at once (and
// the first such pass records how many passes did work).
__global__ __launch_bounds__(kCopyThreads) void k_jpass(JumpArgs a) {
  if (jump_failed(a.st)) return;
  if (a.pass > 0) {
    const uint32_t* pf = a.flags + (a.pass - 1) * kJShards * kJFlagStride;
    const uint32_t f = threadIdx.x < kJShards ? pf[threadIdx.x * kJFlagStride] : 0u;
    if (!__syncthreads_or(int(f))) {
      if (blockIdx.x == 0 && threadIdx.x == 0 && a.st->jump_used == 0) a.st->jump_used = a.pass;
      return;
    }
  }
  const uint32_t lane = lane_id(), limit = a.n_items * a.S;
  AX_GLOBAL uint32_t* const J = gp(a.J);
  bool any = false;
  walk_words(a, a.amap, [&](const WordGroup& w) __attribute__((always_inline)) {
    const uint32_t* const g = w.g;
    const uint64_t* const wv = w.wv;
    uint32_t v[kJStepWords];
#pragma unroll
    for (uint32_t u = 0; u < kJStepWords; ++u) v[u] = ((wv[u] >> lane) & 1) ? J[g[u] * 64 + lane] : kJRes;
#pragma unroll
    for (uint32_t u = 0; u < kJStepWords; ++u)
      if (!(v[u] & kJRes)) v[u] = v[u] < limit ? J[v[u]] : jump_broken(a.st, 2);
#pragma unroll
    for (uint32_t u = 0; u < kJStepWords; ++u)
      if (!(v[u] & kJRes)) v[u] = v[u] < limit ? J[v[u]] : jump_broken(a.st, 2);
#pragma unroll
    for (uint32_t u = 0; u < kJStepWords; ++u) {
      if (!wv[u]) continue;
      const bool act = (wv[u] >> lane) & 1;
      if (act) J[g[u] * 64 + lane] = v[u];
      const uint64_t still = __ballot(act && !(v[u] & kJRes));
      if (lane == 0 && still != wv[u]) a.amap[g[u]] = still;
      any |= still != 0;
    }
  });
  if (__syncthreads_or(int(any)) && threadIdx.x == 0)
    a.flags[(a.pass * kJShards + blockIdx.x % kJShards) * kJFlagStride] = 1;
}

// Output: every leftover byte takes its entry's value (following any entry
// the passes left unfinished).  Of a group of eight busy words, a lane owns
// four consecutive positions of one word in each half: one 16-byte entry
// load, then one 32-bit store when all four are leftover (byte stores
// otherwise: the other bytes keep their value).
__global__ __launch_bounds__(kCopyThreads) void k_jgather(JumpArgs a) {
  if (jump_failed(a.st)) return;
  const uint32_t lane = lane_id(), limit = a.n_items * a.S, omask = (1u << a.s_log2) - 1u;
  const AX_GLOBAL uint32_t* const J = gp(a.J);
  const uint32_t sub = lane >> 4, q4 = 4 * (lane & 15u);
  static_assert(kJStepWords == 8, "the gather takes a group's words as two halves of four");
  walk_words(a, a.lmap, [&](const WordGroup& w) __attribute__((always_inline)) {
#pragma unroll
    for (uint32_t h = 0; h < 2; ++h) {
      // this lane's word of the half: word 4 h + (lane / 16) (a select: it varies by lane)
      const uint32_t g0 = w.g[4 * h], g1 = w.g[4 * h + 1], g2 = w.g[4 * h + 2], g3 = w.g[4 * h + 3];
      const uint64_t w0 = w.wv[4 * h], w1 = w.wv[4 * h + 1], w2 = w.wv[4 * h + 2], w3 = w.wv[4 * h + 3];
      const uint32_t gk = sub < 2 ? (sub == 0 ? g0 : g1) : (sub == 2 ? g2 : g3);
      const uint64_t wk = sub < 2 ? (sub == 0 ? w0 : w1) : (sub == 2 ? w2 : w3);
      const uint32_t bits4 = uint32_t(wk >> q4) & 0xFu;
      if (!bits4) continue;
      const uint32_t p = gk * 64 + q4;
      u32x4 e = *reinterpret_cast<const AX_GLOBAL u32x4*>(J + p);
      uint32_t x0 = (bits4 & 1) ? e.x : kJRes, x1 = (bits4 & 2) ? e.y : kJRes;
      uint32_t x2 = (bits4 & 4) ? e.z : kJRes, x3 = (bits4 & 8) ? e.w : kJRes;
      if (!(x0 & x1 & x2 & x3 & kJRes)) {  // an entry the passes did not finish: follow it
        for (uint32_t hop = 0; !(x0 & kJRes); ++hop) x0 = x0 < limit && hop < kJChaseLimit ? J[x0] : jump_broken(a.st, 3);
        for (uint32_t hop = 0; !(x1 & kJRes); ++hop) x1 = x1 < limit && hop < kJChaseLimit ? J[x1] : jump_broken(a.st, 3);
        for (uint32_t hop = 0; !(x2 & kJRes); ++hop) x2 = x2 < limit && hop < kJChaseLimit ? J[x2] : jump_broken(a.st, 3);
        for (uint32_t hop = 0; !(x3 & kJRes); ++hop) x3 = x3 < limit && hop < kJChaseLimit ? J[x3] : jump_broken(a.st, 3);
      }
      AX_GLOBAL uint8_t* const o = gp(a.ibase[p >> a.s_log2]) + (p & omask);
      if (bits4 == 0xFu) {
        *reinterpret_cast<AX_GLOBAL uint32_t*>(o) = (x0 & 0xFFu) | ((x1 & 0xFFu) << 8) | ((x2 & 0xFFu) << 16) | ((x3 & 0xFFu) << 24);
      } else {
        if (bits4 & 1) o[0] = uint8_t(x0);
        if (bits4 & 2) o[1] = uint8_t(x1);
        if (bits4 & 4) o[2] = uint8_t(x2);
        if (bits4 & 8) o[3] = uint8_t(x3);
      }
    }
  });
}

// ------------------------------------------------------ match layer: roots --
//
// The match layer of the default schedule.  Every output byte of a match
// comes, over a chain of matches, from a literal byte (or from a byte of an
// earlier window), and literal bytes are final once the parse is through.  So
// a match needs no other match to be written first: k_roots follows each
// piece of a match's source to the literals behind it and copies those, all
// blocks at once.  A step of such a walk looks up one of the parse's records:
// a position is either a literal, then the bytes up to the next match are
// taken, or the byte of a match, found by its rank, and the walk goes on at
// that match's source.  A step is two loads of 16 bytes at unrelated
// addresses, the record and then either the bytes or the match: what bounds
// the kernel is the latency of these two loads times a wave's longest walk,
// and how many such gathers a compute unit serves (one address per cycle), so
// both cases share one load instruction (separate loads, the bytes always
// among them: 382 us for the 254 MB DNA archive's matches, this form 220 us).
//
// A walk ends after kRootSteps steps: its bytes are marked as pending in a
// bitmap, each with the window position it was followed to (the jump array),
// and k_sweep and k_finish resolve them.  Walking on instead keeps a block's
// whole workgroup for one lane.  In blocks of archives taken to be deep nearly
// every walk would end so, and all bytes are marked at once (k_mark).
//
// Against the rounds schedule (same data, whole match layer): 254 MB DNA
// 512 -> 330 us, 80 MiB text 1632 -> 565 us, 64 KiB DNA 122 -> 22 us.
//
// A block's window position o of window block x is x * S + o, as for the
// pointer-jumping remainder of the rounds schedule, whose jump array (kJRes
// marks a final byte) and leftover map these kernels use.

constexpr uint32_t kRootItem = 16;   // bytes per work item: one 16-byte source load
// Steps before a walk's bytes are left pending (against nine, 254 MB of DNA / 32
// MiB of reads take with 3, 4, 6 and 12 steps 1.13 / 1.04, 1.07 / 1.01, 1.02 / 1.00
// and 1.04 / 1.07 times as long).
constexpr uint32_t kRootSteps = 9;

// The window's first blocks are marked, the others walked: those of archives
// taken to be deep, then (open) those of archives that are if enough of their
// bytes are copies, which their parse has counted by then.
struct DeepBlocks {
  uint32_t sure, open;     // blocks
  uint32_t copied_from;    // match bytes from which the open ones are marked
  const uint32_t* copied;  // their counters
  __device__ uint32_t marked() const {
    if (open == 0) return sure;
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < kCopiedShards; ++k) sum += copied[k * kCounterStride];
    return sum >= copied_from ? sure + open : sure;
  }
  // what k_settle found
  __device__ uint32_t marked(const DevStatus* st) const { return open == 0 ? sure : st->marked; }
};

struct RootArgs {
  const JobDev* jobs;
  const WinBlock* wbl;
  uint32_t n_items;
  uint32_t n_tok;
  uint32_t s_log2;        // log2 S
  const uint64_t* tok;    // window tokens in (job, output) order
  uint8_t* cmd;           // command slots: the blocks' records
  uint32_t* J;            // jump array: one entry per window position
  uint64_t* lmap;         // pending bytes, one bit per window position
  DevStatus* st;
  DeepBlocks deep;
  uint32_t mark_log2;     // k_mark: log2 of the positions of a workgroup
};

// Where source positions of a window block's job lie in the window, and where
// their bytes are.  find() is false for positions of no block of the window:
// those are final (an earlier window wrote them) or, in a range decode, not
// needed by anybody.
struct RootDirect {  // the job's blocks are consecutive in the window
  gbytes out;
  uint64_t j0, n_bytes;
  uint32_t span, base, lb, sl;
  __device__ RootDirect(const RootArgs& a, const JobDev& J, const WinBlock& wb)
      : out(gp(J.out)), n_bytes(J.n_bytes), lb(uint32_t(__builtin_ctz(J.B))), sl(a.s_log2) {
    j0 = a.wbl[wb.first].b << lb;
    span = wb.count << lb;  // at most 2^31
    base = wb.first << sl;
  }
  __device__ bool find(uint64_t s, uint32_t& pos) const {
    const uint64_t rel = s - j0;
    if (rel >= span) return false;
    const uint32_t r = uint32_t(rel);
    pos = base + ((r >> lb) << sl) + (r & ((1u << lb) - 1u));
    return true;
  }
  // where the byte of s is; wide: 16 bytes may be read from there
  __device__ gbytes byte_at(uint64_t s, bool, uint32_t, bool& wide) const {
    wide = s + kRootItem <= n_bytes;
    return out + s;
  }
};
struct RootMapped {  // a range decode: slot x of the scratch is window block x (a stale entry names another block)
  gbytes out;
  const AX_GLOBAL uint32_t* slot;
  const WinBlock* wbl;
  uint32_t n_items, lb, junk;
  __device__ RootMapped(const RootArgs& a, const JobDev& J, const WinBlock&)
      : out(gp(J.out)), slot(gp(J.slot)), wbl(a.wbl), n_items(a.n_items), lb(uint32_t(__builtin_ctz(J.B))), junk(J.junk) {}
  __device__ bool find(uint64_t s, uint32_t& pos) const {
    const uint32_t x = slot[s >> lb];
    if (x >= n_items || wbl[x].b != s >> lb) return false;
    pos = (x << lb) + uint32_t(s & ((1u << lb) - 1u));
    return true;
  }
  // the scratch holds the junk block behind the window's: 16 bytes from any
  // window position, and for other positions bytes nobody needs
  __device__ gbytes byte_at(uint64_t, bool in, uint32_t pos, bool& wide) const {
    wide = true;
    return out + (in ? uint64_t(pos) : uint64_t(junk) << lb);
  }
};
template <class O> struct RootWin;
template <> struct RootWin<OutDirect> { typedef RootDirect type; };
template <> struct RootWin<OutMapped> { typedef RootMapped type; };

// Inclusive wave scan of a u32 (maximum).
__device__ inline uint32_t wave_incl_max32(uint32_t x) {
  x = max(x, dpp_move<kDppRowShr + 1, 0xF>(0, x));
  x = max(x, dpp_move<kDppRowShr + 2, 0xF>(0, x));
  x = max(x, dpp_move<kDppRowShr + 4, 0xF>(0, x));
  x = max(x, dpp_move<kDppRowShr + 8, 0xF>(0, x));
  x = max(x, dpp_move<kDppRowBcast15, 0xA>(0, x));
  x = max(x, dpp_move<kDppRowBcast31, 0xC>(0, x));
  return x;
}

// Sixteen bytes as two words, byte 0 lowest.
struct B16 {
  uint64_t lo, hi;
};
__device__ inline B16 b16_low(B16 v, uint32_t m) {  // the first m <= 16 bytes
  if (m < 8) return B16{v.lo & ((1ull << (8 * m)) - 1), 0};
  return B16{v.lo, m < 16 ? v.hi & ((1ull << (8 * (m - 8))) - 1) : v.hi};
}
__device__ inline B16 b16_up(B16 v, uint32_t n) {  // moved up by n < 16 bytes
  if (n >= 8) return B16{0, v.lo << (8 * (n - 8))};
  return B16{v.lo << (8 * n), n ? (v.hi << (8 * n)) | (v.lo >> (64 - 8 * n)) : v.hi};
}

// One item's walk: bytes [0, kend) of the item come from archive positions
// src0...; k of them are in acc.  s is where byte k's source was followed to,
// standing for run bytes.  A source inside a self-overlapping match repeats
// with its period: once a period of it is taken the rest is repeated from acc
// (rep: period | first byte not taken yet << 8 | end << 16).
struct Walk {
  uint64_t src0, s, next_s;  // next_s, next_run: where the bytes after this run go on (run 0: at src0 + k)
  uint32_t k, kend, run, next_run, rep;
  B16 acc;
  __device__ void go_on() {
    if (next_run) s = next_s, run = next_run;
    else s = src0 + k, run = kend - k;
    next_run = 0;
  }
};

// One step; false once the item is complete.
template <class W>
__device__ inline bool walk_step(Walk& x, const W& win, const RootArgs& a, uint32_t B) {
  uint32_t pos = 0, r, u = 0;
  const bool in = win.find(x.s, pos);
  if (in) {
    const uint32_t off = pos & ((1u << a.s_log2) - 1u), bit = off & 31u;
    const u32x4 q = block_recs(a.cmd, 1u << a.s_log2, pos >> a.s_log2)[off >> 5];
    const uint64_t cov = ((uint64_t(q.w) << 32) | q.x) >> bit;  // at least 33 positions: more than an item
    r = cov ? uint32_t(__builtin_ctzll(cov)) : 64u;
    r = min(r, B - off);
    u = q.z + uint32_t(__popc(q.y & (~0u >> (31 - bit)))) - 1;
  } else {  // final bytes, up to the end of their block
    r = B - uint32_t(x.s & (B - 1));
  }
  bool wide;
  const gbytes from = win.byte_at(x.s, in, pos, wide);
  const gbytes p = r ? from : reinterpret_cast<gbytes>(gp(const_cast<uint64_t*>(a.tok)) + 2 * uint64_t(u));
  u32x4 v = {0, 0, 0, 0};
  const uint32_t m = min(r, x.run);
  if (r == 0 || wide) {
    v = *reinterpret_cast<const AX_GLOBAL u32x4_u*>(p);
  } else {  // the output's last bytes
    for (uint32_t i = 0; i < m; ++i) v[(i >> 2) & 3] |= uint32_t(p[i]) << (8 * (i & 3));
  }
  const B16 b = {uint64_t(v.x) | (uint64_t(v.y) << 32), uint64_t(v.z) | (uint64_t(v.w) << 32)};
  if (r) {
    const B16 up = b16_up(b16_low(b, m), x.k);
    x.acc.lo |= up.lo, x.acc.hi |= up.hi;
    x.k += m;
    if (x.rep && x.k >= ((x.rep >> 8) & 0xFF)) {
      const uint32_t pe = x.rep >> 16;
      for (uint32_t span = x.rep & 0xFF; x.k < pe; span *= 2) {
        // bytes [k, k + span) repeat those span before them
        const uint32_t e = min(pe, x.k + span);
        const B16 up = b16_up(x.acc, span), t = b16_low(up, e), below = b16_low(up, x.k);
        x.acc.lo |= t.lo ^ below.lo, x.acc.hi |= t.hi ^ below.hi;
        x.k = e;
      }
      x.rep = 0;
      x.run = x.next_run = 0;
    } else {
      x.s += m, x.run -= m;
    }
    if (x.run == 0) x.go_on();
    return x.k < x.kend;
  }
  const uint64_t us = b.lo, ud = b.hi & ((1ull << 48) - 1), dist = ud - us;
  const uint32_t ulen = uint32_t(b.hi >> 48) + 1;
  const uint32_t per = dist < ulen ? uint32_t(dist) : ulen;
  uint32_t o = uint32_t(x.s - ud);
  const uint32_t all = min(x.run, ulen - o);
  if (all > per && !x.rep) x.rep = per | ((x.k + per) << 8) | ((x.k + all) << 16);
  if (o >= per) o %= per;
  const uint32_t run = min(all, per - o);
  if (run < x.run) x.next_s = x.s + run, x.next_run = x.run - run;
  x.run = run;
  x.s = us + o;
  return true;
}

// Jump-array entries of an item's bytes [k, kend), je = entry of its byte 0.
template <class W>
__device__ inline void mark_item(const Walk& x, const W& win, AX_GLOBAL uint32_t* je) {
  const uint64_t s2 = x.src0 + x.k + x.run;  // the source of the bytes after this run
  const uint32_t n2 = x.kend - x.k - x.run;
  uint32_t pa = 0, pb = 0, pz = 0;
  bool plain = win.find(x.s, pa) && win.find(x.s + x.run - 1, pz) && pz == pa + x.run - 1;
  if (n2) plain = plain && win.find(s2, pb) && win.find(s2 + n2 - 1, pz) && pz == pb + n2 - 1;
  if (plain) {  // both runs are consecutive window positions
    const uint32_t cut = x.k + x.run, ea = pa - x.k, eb = pb - cut;
#pragma unroll
    for (uint32_t g = 0; g < kRootItem; g += 4) {
      const u32x4 e = {(g < cut ? ea : eb) + g, (g + 1 < cut ? ea : eb) + g + 1, (g + 2 < cut ? ea : eb) + g + 2,
                       (g + 3 < cut ? ea : eb) + g + 3};
      if (x.k <= g && g + 4 <= x.kend) {
        *reinterpret_cast<AX_GLOBAL u32x4_w*>(je + g) = e;
      } else {
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
          if (g + q >= x.k && g + q < x.kend) je[g + q] = e[q];
      }
    }
    return;
  }
  for (uint32_t j = x.k; j < x.kend; ++j) {
    const uint64_t sp = j < x.k + x.run ? x.s + (j - x.k) : x.src0 + j;
    uint32_t p = 0;
    bool wide;
    const bool in = win.find(sp, p);
    je[j] = in ? p : kJRes | *win.byte_at(sp, false, 0, wide);
  }
}

// The first m (1..16) bytes of v into the zero-filled tile at byte at: word
// ORs, so items that share a word need no order.
__device__ inline void tile_or(uint32_t* tile, uint32_t at, B16 v) {
  // bytes moved up by at mod 4: selector 4 + i - shift picks from the word and the one before
  const uint32_t sel = 0x07060504u - (at & 3) * 0x01010101u;
  const uint32_t v0 = uint32_t(v.lo), v1 = uint32_t(v.lo >> 32), v2 = uint32_t(v.hi), v3 = uint32_t(v.hi >> 32);
  uint32_t* const t = tile + (at >> 2);
  const uint32_t w0 = __builtin_amdgcn_perm(v0, 0u, sel), w1 = __builtin_amdgcn_perm(v1, v0, sel),
                 w2 = __builtin_amdgcn_perm(v2, v1, sel), w3 = __builtin_amdgcn_perm(v3, v2, sel),
                 w4 = __builtin_amdgcn_perm(0u, v3, sel);
  if (w0) atomicOr(t, w0);
  if (w1) atomicOr(t + 1, w1);
  if (w2) atomicOr(t + 2, w2);
  if (w3) atomicOr(t + 3, w3);
  if (w4) atomicOr(t + 4, w4);
}

// One workgroup per window block.  A token's first min(len, dist) bytes are
// cut into items of kRootItem bytes, laid end to end over the wave's lanes;
// the rest of a self-overlapping token repeats them (periodic fill) from the
// tile.  (With five, six or eight waves a block the decode of 254 MB DNA takes
// 790 to 804 us instead of 724.)  The tile starts zeroed and the parse left
// zeros where matches go, so a 16-byte chunk of the block is finished by OR-ing
// the tile into it, and chunks without match bytes are not touched.
template <class O>
__device__ __forceinline__ void roots_block(const RootArgs& a, uint32_t first, uint32_t block, uint32_t blocks) {
  __shared__ __attribute__((aligned(16))) uint32_t tile[kMaxB / 4 + 4];  // the last item's fifth word
  __shared__ uint64_t row[kMaxB / 64];                                   // the block's pending bytes
  __shared__ uint32_t heads[kCopyThreads];                               // per wave: tokens starting at an item
  const uint32_t lane = lane_id(), item = first + xcd_item(block, blocks);
  const WinBlock wb = a.wbl[item];
  const uint32_t t1 = item + 1 < a.n_items ? a.wbl[item + 1].tok : a.n_tok;
  const AX_GLOBAL u64x2* const tok = reinterpret_cast<const AX_GLOBAL u64x2*>(gp(a.tok));
  // the block's tokens in as few passes as hold them, evenly over the waves of
  // each, so that a wave's items mostly fit its lanes; the first pass's are
  // loaded ahead
  constexpr uint32_t kWaves = kCopyThreads / 64;
  const uint32_t ntb = t1 - wb.tok, passes = (ntb + kCopyThreads - 1) / kCopyThreads;
  const uint32_t share = passes ? (ntb + kWaves * passes - 1) / (kWaves * passes) : 0u;  // <= 64
  const uint32_t base0 = wb.tok + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * share;
  u64x2 tk = {0, 0};
  if (lane < share && base0 + lane < t1) tk = tok[base0 + lane];
  const JobDev& J = a.jobs[wb.job];
  const typename RootWin<O>::type win(a, J, wb);
  const uint32_t B = J.B, sw = 1u << (a.s_log2 - 6);
  const uint64_t bs = wb.b * B;
  const gbytes ob = O(J).at(bs);
  const uint32_t blen = uint32_t(min<uint64_t>(B, J.n_bytes - bs));
  AX_GLOBAL uint32_t* const jarr = gp(a.J);
  uint8_t* const tile8 = reinterpret_cast<uint8_t*>(tile);
  uint32_t* const row32 = reinterpret_cast<uint32_t*>(row);
  uint32_t* const hd = heads + (threadIdx.x & ~63u);
  // the status is checked once the block's own loads are in flight
  if (__hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  for (uint32_t k = threadIdx.x; k < kMaxB / 16; k += kCopyThreads)
    *reinterpret_cast<u32x4*>(tile + 4 * k) = u32x4{0, 0, 0, 0};
  if (threadIdx.x < kMaxB / 64) row[threadIdx.x] = 0;
  __syncthreads();
  bool wpend = false;  // this wave left bytes pending
  const uint32_t jblk = item << a.s_log2;  // window position of the block's first byte
  for (uint32_t base = base0; base < t1; base += kWaves * share) {
    const bool have = lane < share && base + lane < t1;
    if (base != base0) {
      tk = u64x2{0, 0};
      if (have) tk = tok[base + lane];
    }
    const uint64_t tsrc = tk.x, dst = tk.y & ((1ull << 48) - 1), dist = dst - tsrc;
    const uint32_t tlen = have ? uint32_t(tk.y >> 48) + 1 : 0u, trel = uint32_t(dst - bs);
    const uint32_t tn = dist < tlen ? uint32_t(dist) : tlen;
    const uint32_t mine = (tn + kRootItem - 1) / kRootItem;
    const uint32_t incl = wave_incl_sum32(mine), start = incl - mine;
    const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
    for (uint32_t i0 = 0; i0 < total; i0 += 64) {
      // the token of item i0 + lane: the last one starting at or before it
      hd[lane] = 0;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (have && start >= i0 && start < i0 + 64) hd[start - i0] = lane;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const uint32_t first = uint32_t(__popcll(__ballot(have && start <= i0))) - 1;
      const int l = int(max(first, wave_incl_max32(hd[lane])));
      const uint32_t sub = i0 + lane - __shfl(start, l, 64);
      const uint32_t at = __shfl(trel, l, 64) + kRootItem * sub;  // block position
      Walk x;
      x.src0 = __shfl((unsigned long long)tsrc, l, 64) + kRootItem * sub;
      x.s = x.src0;
      x.kend = min(kRootItem, __shfl(trel, l, 64) + __shfl(tn, l, 64) - at);
      x.k = 0, x.run = x.kend, x.next_run = x.rep = 0, x.acc = B16{0, 0};
      bool act = i0 + lane < total;
      const uint32_t n0 = uint32_t(__popcll(__ballot(act)));
      bool deep = false;
      for (uint32_t step = 0; step < kRootSteps; ++step) {
        const uint32_t left = uint32_t(__popcll(__ballot(act)));
        if (!left) break;
        // most walks of a large wave still going: a deep archive
        deep = n0 >= 16 && step == 2 && 4 * left > 3 * n0;
        if (deep) break;
        if (act) act = walk_step(x, win, a, B);
      }
      if (i0 + lane < total && x.k) tile_or(tile, at, x.acc);
      if (__ballot(act)) {  // items left walking: their bytes are pending, named by where the walk stands
        wpend = true;
        if (act) {
          mark_item(x, win, jarr + jblk + at);
          const uint64_t m = uint64_t(((1u << x.kend) - 1u) & ~((1u << x.k) - 1u)) << (at & 31);
          atomicOr(&row32[at >> 5], uint32_t(m));
          if (m >> 32) atomicOr(&row32[(at >> 5) + 1], uint32_t(m >> 32));
        }
      }
    }
    // self-overlapping tokens: byte j >= dist repeats byte j mod dist of the token
    uint64_t rep = __ballot(tlen > tn);
    if (rep) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    while (rep) {
      const int l = __builtin_ctzll(rep);
      rep &= rep - 1;
      const uint32_t d0 = __builtin_amdgcn_readlane(trel, l), n = __builtin_amdgcn_readlane(tlen, l),
                     per = __builtin_amdgcn_readlane(tn, l);
      const uint32_t jstep = 64 % per;
      uint32_t j = lane % per;
      for (uint32_t k = per + lane; k < n; k += 64) {
        if (wpend && ((row32[(d0 + j) >> 5] >> ((d0 + j) & 31)) & 1)) {
          jarr[jblk + d0 + k] = jblk + d0 + j;
          atomicOr(&row32[(d0 + k) >> 5], 1u << ((d0 + k) & 31));
        } else {
          tile8[d0 + k] = tile8[d0 + j];
        }
        j += jstep;
        if (j >= per) j -= per;
      }
    }
  }
  const int any = __syncthreads_or(int(wpend));
  const uint32_t full = blen / 16;
  constexpr uint32_t kChunks = kMaxB / 16 / kCopyThreads;  // a thread's, their loads in flight together
  u32x4 add[kChunks], old[kChunks];
#pragma unroll
  for (uint32_t q = 0; q < kChunks; ++q) {
    const uint32_t c = q * kCopyThreads + threadIdx.x;
    add[q] = *reinterpret_cast<const u32x4*>(tile + 4 * c);
    if (c >= full) add[q] = u32x4{0, 0, 0, 0};
    old[q] = u32x4{0, 0, 0, 0};
    if (add[q].x | add[q].y | add[q].z | add[q].w) old[q] = *reinterpret_cast<const AX_GLOBAL u32x4*>(ob + 16 * c);
  }
#pragma unroll
  for (uint32_t q = 0; q < kChunks; ++q)
    if (add[q].x | add[q].y | add[q].z | add[q].w)
      *reinterpret_cast<AX_GLOBAL u32x4*>(ob + 16 * (q * kCopyThreads + threadIdx.x)) = old[q] | add[q];
  if (16 * full + threadIdx.x < blen) ob[16 * full + threadIdx.x] |= tile8[16 * full + threadIdx.x];  // the last bytes
  if (threadIdx.x < sw) gp(a.lmap)[uint64_t(item) * sw + threadIdx.x] = threadIdx.x < kMaxB / 64 ? row[threadIdx.x] : 0ull;
  if (any && threadIdx.x == 0) a.st->n_pending = 1;
}

// log2 of the positions a workgroup of k_mark takes: small in small windows,
// where a workgroup's chain of loads is what counts (1 MB of text 3 % faster
// with 1024 than with 4096), large in others (80 MiB of text 2 % faster with 4096)
constexpr uint32_t kMarkSmallLog2 = 10, kMarkLog2 = 12;

// Blocks of deep archives: walks would not end in a few steps, so every byte
// gets its jump-array entry at once, four consecutive positions a lane (the
// record shared by eight lanes, one 16-byte store each): a match byte names
// its source, any other holds its value.  The bitmap has every byte of the
// block.
template <class O>
__device__ __forceinline__ void mark_part(const RootArgs& a, uint32_t block, uint32_t blocks) {
  const uint32_t part = xcd_item(block, blocks), lp = a.s_log2 - a.mark_log2;  // parts per block: 2^lp
  const uint32_t item = part >> lp, p0 = (part & ((1u << lp) - 1u)) << a.mark_log2;
  const WinBlock wb = a.wbl[item];
  const JobDev& J = a.jobs[wb.job];
  const typename RootWin<O>::type win(a, J, wb);
  const uint32_t B = J.B, sw = 1u << (a.s_log2 - 6);
  const uint64_t bs = wb.b * B;
  const gbytes ob = O(J).at(bs);
  const uint32_t blen = uint32_t(min<uint64_t>(B, J.n_bytes - bs));
  const AX_GLOBAL u64x2* const tok = reinterpret_cast<const AX_GLOBAL u64x2*>(gp(a.tok));
  const AX_GLOBAL u32x4* const rec = block_recs(a.cmd, 1u << a.s_log2, item);
  AX_GLOBAL uint32_t* const je = gp(a.J) + (uint64_t(item) << a.s_log2);
  if (__hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  const uint32_t end = min(blen, p0 + (1u << a.mark_log2));
  // (two and four groups of four positions a thread with their loads in flight
  // together take registers from resident waves: 80 MiB text 676 -> 689, 723 us)
  for (uint32_t p = p0 + 4 * threadIdx.x; p < end; p += 4 * kCopyThreads) {
    const u32x4 q = rec[p >> 5];
    const uint32_t bit = p & 31u, cov = (q.x >> bit) & 0xFu, starts = q.y >> bit;
    uint32_t lit = 0;
    if (p + 4 <= blen) lit = *reinterpret_cast<const AX_GLOBAL uint32_t*>(ob + p);
    else
      for (uint32_t e = 0; p + e < blen; ++e) lit |= uint32_t(ob[p + e]) << (8 * e);
    // the match of byte 0, if it has one, and the next one to start, loaded together
    uint32_t u = q.z + uint32_t(__popc(q.y & (~0u >> (31 - bit)))) - 1;
    u64x2 t = {0, 0}, t2 = {0, 0};
    if (cov & 1u) t = tok[u];
    if (starts & 0xEu) t2 = tok[u + 1];
    u32x4 v;
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) {
      if (e && ((starts >> e) & 1u)) {
        t = t2;
        ++u;
        if (starts & (0xEu << e) & 0xFu) t2 = tok[u + 1];  // matches shorter than four bytes
      }
      uint32_t x = kJRes | ((lit >> (8 * e)) & 0xFFu);
      if ((cov >> e) & 1u) {
        const uint64_t ud = t.y & ((1ull << 48) - 1), dist = ud - t.x;
        uint32_t o = uint32_t(bs + p + e - ud);
        if (o >= dist) o %= uint32_t(dist);  // o < 2^16
        uint32_t pos = 0;
        const uint64_t s = t.x + o;
        if (win.find(s, pos)) {
          x = pos;
        } else {
          bool wide;
          x = kJRes | *win.byte_at(s, false, 0, wide);
        }
      }
      v[e] = x;
    }
    *reinterpret_cast<AX_GLOBAL u32x4*>(je + p) = v;
  }
  if (threadIdx.x < (1u << (a.mark_log2 - 6))) {
    const uint32_t w = p0 + 64 * threadIdx.x;
    gp(a.lmap)[uint64_t(item) * sw + (w >> 6)] = w + 64 <= blen ? ~0ull : w < blen ? (1ull << (blen - w)) - 1 : 0ull;
  }
  if (part == 0 && threadIdx.x == 0) a.st->n_pending = 1;
}

template <class O>
__global__ __launch_bounds__(kCopyThreads, 8) void k_roots(RootArgs a) {
  roots_block<O>(a, 0, blockIdx.x, gridDim.x);
}
template <class O>
__global__ __launch_bounds__(kCopyThreads) void k_mark(RootArgs a) {
  mark_part<O>(a, blockIdx.x, gridDim.x);
}
// A window of deep and other archives takes both at once (the first workgroups
// walk), and so its sweeps and finishes: neither kind waits for the
// other's last workgroups.  40 archives of 61 MiB in all, 16.4 of them deep, 443
// us with a launch per kind, 407 with one for both (deep ones first 412; half the
// sweep's workgroups for each kind 432, and with marking and walks apart 443).
// Seven waves a SIMD: the two bodies in one kernel spill with eight.  With open
// blocks the grid is that of all of them marked, and walks leave some idle.
template <class O>
__global__ __launch_bounds__(kCopyThreads, 7) void k_settle(RootArgs a) {
  const uint32_t marked = a.deep.marked(), walked = a.n_items - marked;
  if (blockIdx.x == 0 && threadIdx.x == 0) a.st->marked = marked;
  if (blockIdx.x < walked) {
    roots_block<O>(a, marked, blockIdx.x, walked);
  } else {
    const uint32_t part = blockIdx.x - walked, parts = marked << (a.s_log2 - a.mark_log2);
    if (part < parts) mark_part<O>(a, part, parts);
  }
}

// ---- pending bytes: sweep and finish
//
// The blocks are cut into eight runs, one per XCD (workgroup g of a launch
// goes to XCD g mod 8, whose L2 then holds the run's entries).
// k_sweep walks each run's pending bytes in ascending order, following a
// byte's entry to the first byte before the run or to a final byte, and
// writes what it found back (a pass of pointer jumping reads and writes every
// entry and only triples its reach: 80 MiB of text took five, 944 us, where
// the sweep takes 243 us).  Entries name lower positions, so a walk soon
// meets bytes that were swept before and carry their own walk's end; the bytes
// in flight write back where they stand every few hops (kSweepBack), so that
// they shorten each other's walks as well.
// (Stale entries, from another compute unit's cache, name the same value and
// only cost hops.)  After it, an entry holds its value or names a byte of an
// earlier run; k_finish writes the bytes, following those.
constexpr uint32_t kXcds = 8;
constexpr uint32_t kSweepSlots = 4;    // bytes a lane follows at a time
constexpr uint32_t kSweepRows = 8;     // map words a wave follows at a time where every byte has an entry
// Consecutive map words a wave takes at a time: rows of whole words where every
// byte has an entry (80 MiB of text with 4 / 2: 1.06 / 1.10 times as long), fewer
// where pending bytes come in clusters (with 4 / 2 / 1: 16 MiB of DNA in 4 KiB
// blocks 151 / 145 / 145 us, 32 MiB of reads 226 / 222 / 223, 254 MB of DNA 685 /
// 680 / 686).
constexpr uint32_t kAllChunk = 8, kFewChunk = 2;
constexpr uint32_t kSweepGrid = 2048;  // workgroups of a sweep or finish launch
// Map words a wave of k_finish has in flight (80 MiB text with 8: 701, not 677
// us), and takes at a time: dealing them out evenly counts for more than rows
// (with the sweep's eight: 80 MiB text 675, not 663 us, 1 MB 65.7, not 61.3).
constexpr uint32_t kFinishWords = 4;
// Hops after which a sweep writes back where its walks stand.  Other walks then
// skip what these have followed, so a chain of h bytes in flight at once takes
// about kSweepBack * log(h) / log(kSweepBack) hops, not h.  Matches that copy from
// just behind are such chains: rows of 16 bytes, each but four of them a copy of
// the row before, 4 and 32 MiB: 736 and 2202 us without writing back, 131 and
// 1149 every 16 hops, 116 and 975 every 8, 108 and 844 every 4.  Text, DNA and
// reads (chains of long hops) measure the same with all of them.
constexpr uint32_t kSweepBack = 4;
constexpr uint32_t kFinishLimit = 1u << 24;  // hops k_finish follows before it reports a device error
constexpr uint32_t kSweepLimit = 1u << 24;   // hops after which a sweep leaves the rest of its walks to k_finish

struct SweepArgs {
  uint32_t s_log2;
  uint32_t* J;
  const uint64_t* lmap;
  const JobDev* jobs;
  const WinBlock* wbl;
  uint32_t one_job;        // 1: the plan has one job, so window positions are contiguous in its output
  uint8_t* const* ibase;   // else per window block: where its output bytes start
  DevStatus* st;
  uint32_t n_items;
  DeepBlocks deep;
  uint32_t part;           // k_finish: this launch's eighth of the marked blocks, those before it final; kXcds: all at once
};

// Where the bytes of window positions are.
struct PosOut {
  gbytes lin;  // window position 0's byte, or null
  uint8_t* const* ibase;
  uint32_t sl;
  __device__ explicit PosOut(const SweepArgs& a) : lin(nullptr), ibase(a.ibase), sl(a.s_log2) {
    if (a.one_job) lin = gp(a.jobs->out) + (a.jobs->slot ? 0 : a.wbl->b << sl);
  }
  __device__ gbytes at(uint32_t v) const { return lin ? lin + v : gp(ibase[v >> sl]) + (v & ((1u << sl) - 1u)); }
};

// A wave's nonzero map words of 64: their indices and bits, in order.
struct WordQueue {
  uint64_t bits[64];
  uint32_t g[64];
};

// The map words [w0, w0 + n), `waves` waves taking kSweepChunk words each in turn:
// step i of wave `wave` reads its next 64 words (64 / kSweepChunk chunks).
template <uint32_t kSweepChunk>
__device__ inline uint32_t queue_words(const uint64_t* lmap, uint64_t w0, uint64_t n, uint64_t wave, uint64_t waves,
                                       uint64_t i, WordQueue& q) {
  const uint32_t lane = lane_id();
  const uint64_t m = ((i * (64 / kSweepChunk) + lane / kSweepChunk) * waves + wave) * kSweepChunk + lane % kSweepChunk;
  const uint64_t mw = m < n ? gp(lmap)[w0 + m] : 0ull;
  const uint64_t nz = __ballot(mw != 0);
  if (mw) {
    const uint32_t at = lanes_below(nz);
    q.bits[at] = mw;
    q.g[at] = uint32_t(w0 + m);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return uint32_t(__popcll(nz));
}

// kAll: every byte of the blocks has an entry (k_mark), so a hop is one load.
template <bool kAll>
__device__ __forceinline__ void sweep_run(const SweepArgs& a, uint32_t block, uint32_t blocks, WordQueue* queues) {
  if (a.st->n_pending == 0 || __hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  const uint32_t lane = lane_id(), g = block / kXcds;
  const uint32_t run = block % kXcds, marked = a.deep.marked(a.st);
  const uint32_t first = kAll ? 0u : marked;
  const uint64_t nb = kAll ? marked : a.n_items - marked;
  const uint32_t b0 = first + uint32_t(nb * run / kXcds), b1 = first + uint32_t(nb * (run + 1) / kXcds);
  const uint32_t lo = b0 << a.s_log2, wl = a.s_log2 - 6;
  AX_GLOBAL uint32_t* const J = gp(a.J);
  const AX_GLOBAL uint64_t* const lm = gp(a.lmap);
  WordQueue& q = queues[threadIdx.x >> 6];
  const PosOut po(a);
  const uint64_t wave = uint64_t(g) * (kCopyThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t waves = uint64_t(blocks / kXcds) * (kCopyThreads / 64);
  const uint64_t n = uint64_t(b1 - b0) << wl;
  for (uint64_t i = 0; i * 64 * waves < n; ++i) {
    const uint32_t cnt = queue_words<kAll ? kAllChunk : kFewChunk>(a.lmap, uint64_t(b0) << wl, n, wave, waves, i, q);
    if (kAll) {  // word by word: the bytes of a group of words leave as whole rows
      for (uint32_t c = 0; c < cnt; c += kSweepRows) {
        uint32_t v[kSweepRows], was[kSweepRows];
        uint32_t at[kSweepRows];  // kept: reading the queue again for every store costs 64 KiB of DNA 0.2 us
        bool in[kSweepRows];
#pragma unroll
        for (uint32_t u = 0; u < kSweepRows; ++u) {
          in[u] = c + u < cnt && ((q.bits[c + u < cnt ? c + u : 0] >> lane) & 1);
          at[u] = q.g[c + u < cnt ? c + u : 0] * 64 + lane;
          v[u] = in[u] ? J[at[u]] : kJRes;
          was[u] = v[u];
        }
        for (uint32_t hop = 1; hop < kSweepLimit; ++hop) {
          bool more = false;
#pragma unroll
          for (uint32_t u = 0; u < kSweepRows; ++u)
            if (!(v[u] & kJRes) && v[u] >= lo) v[u] = J[v[u]];
#pragma unroll
          for (uint32_t u = 0; u < kSweepRows; ++u) more |= !(v[u] & kJRes) && v[u] >= lo;
          if (!__ballot(more)) break;
          if (hop % kSweepBack) continue;
#pragma unroll
          for (uint32_t u = 0; u < kSweepRows; ++u)
            if (v[u] != was[u]) J[at[u]] = was[u] = v[u];
        }
#pragma unroll
        for (uint32_t u = 0; u < kSweepRows; ++u)
          if (v[u] != was[u]) J[at[u]] = v[u];
      }
      continue;
    }
    // every lane follows its bit of the queue's words, kSweepSlots words at a
    // time, each slot going on to its next word when its byte is done
    uint32_t p[kSweepSlots], v[kSweepSlots], nx[kSweepSlots];  // byte (or none), where its walk is, next word
#pragma unroll
    for (uint32_t u = 0; u < kSweepSlots; ++u) p[u] = ~0u, v[u] = 0, nx[u] = u;
    for (uint32_t hop = 1; hop < kSweepLimit; ++hop) {
      bool busy = false;
#pragma unroll
      for (uint32_t u = 0; u < kSweepSlots; ++u) {
        if (p[u] == ~0u && nx[u] < cnt) {
          if ((q.bits[nx[u]] >> lane) & 1) p[u] = v[u] = q.g[nx[u]] * 64 + lane;
          nx[u] += kSweepSlots;
        }
        busy |= p[u] != ~0u || nx[u] < cnt;
      }
      if (!__ballot(busy)) break;
      uint32_t jn[kSweepSlots];
      uint64_t w[kSweepSlots];
#pragma unroll
      for (uint32_t u = 0; u < kSweepSlots; ++u) {
        jn[u] = kJRes, w[u] = 0;
        if (p[u] != ~0u) w[u] = lm[v[u] >> 6], jn[u] = J[v[u]];
      }
#pragma unroll
      for (uint32_t u = 0; u < kSweepSlots; ++u) {
        if (p[u] == ~0u) continue;
        const bool pend = (w[u] >> (v[u] & 63)) & 1;
        v[u] = pend ? jn[u] : kJRes | *po.at(v[u]);
        if ((v[u] & kJRes) || v[u] < lo) {
          J[p[u]] = v[u];
          p[u] = ~0u;
        } else if (hop % kSweepBack == 0) {
          J[p[u]] = v[u];
        }
      }
    }
  }
}

// The pending bytes of the marked (kAll) or other blocks, four consecutive
// positions a lane: an entry holds the value or names an earlier byte.  In
// launches of an eighth each, in order, such a byte is final by then and read
// from the output; else the entries are followed to the value, over at most one
// entry per run.
template <bool kAll>
__device__ __forceinline__ void finish_part(const SweepArgs& a, uint32_t block, uint32_t blocks, WordQueue* queues) {
  if (a.st->n_pending == 0 || __hip_atomic_load(&a.st->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  const uint32_t marked = a.deep.marked(a.st);
  uint32_t b0 = kAll ? 0u : marked, b1 = kAll ? marked : a.n_items;
  if (kAll && a.part < kXcds) {
    b0 = uint32_t(uint64_t(marked) * a.part / kXcds);
    b1 = uint32_t(uint64_t(marked) * (a.part + 1) / kXcds);
  }
  const uint32_t lane = lane_id(), wl = a.s_log2 - 6, lo = kAll && a.part < kXcds ? b0 << a.s_log2 : 0u;
  const AX_GLOBAL uint32_t* const J = gp(a.J);
  const AX_GLOBAL uint64_t* const lm = gp(a.lmap);
  WordQueue& q = queues[threadIdx.x >> 6];
  const PosOut po(a);
  const uint64_t wave = uint64_t(block) * (kCopyThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t waves = uint64_t(blocks) * (kCopyThreads / 64);
  const uint64_t n = uint64_t(b1 - b0) << wl;
  const uint32_t sub = lane >> 4, q4 = 4 * (lane & 15u);
  for (uint64_t i = 0; i * 64 * waves < n; ++i) {
    const uint32_t cnt = queue_words<kFinishWords>(a.lmap, uint64_t(b0) << wl, n, wave, waves, i, q);
    for (uint32_t c = 0; c < cnt; c += kFinishWords) {
      constexpr uint32_t kRows = kFinishWords / 4;  // a lane's groups: word c + 4 h + lane / 16
      uint32_t bits[kRows], p[kRows];
      u32x4 x[kRows];
#pragma unroll
      for (uint32_t h = 0; h < kRows; ++h) {
        const uint32_t wi = c + 4 * h + sub;
        bits[h] = wi < cnt ? uint32_t(q.bits[wi] >> q4) & 0xFu : 0u;
        p[h] = (wi < cnt ? q.g[wi] * 64 : 0u) + q4;
        x[h] = u32x4{kJRes, kJRes, kJRes, kJRes};
        if (bits[h]) x[h] = *reinterpret_cast<const AX_GLOBAL u32x4*>(J + p[h]);
      }
#pragma unroll
      for (uint32_t h = 0; h < kRows; ++h)
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e)
          if (!((bits[h] >> e) & 1)) x[h][e] = kJRes;
      for (uint32_t hop = 0;; ++hop) {  // to the value, or to a settled byte
        bool more = false;
#pragma unroll
        for (uint32_t h = 0; h < kRows; ++h)
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e) more |= !(x[h][e] & kJRes) && x[h][e] >= lo;
        if (!__ballot(more)) break;
        if (hop >= kFinishLimit) {
          if (lane == 0) report(a.st, AX_E_DEVICE, ~0ull);
          return;
        }
        uint64_t w[kRows][4];
        uint32_t jn[kRows][4];
#pragma unroll
        for (uint32_t h = 0; h < kRows; ++h)
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e) {
            w[h][e] = 0, jn[h][e] = 0;
            const uint32_t y = x[h][e];
            if (!(y & kJRes) && y >= lo) {
              jn[h][e] = J[y];
              w[h][e] = kAll ? ~0ull : lm[y >> 6];
            }
          }
#pragma unroll
        for (uint32_t h = 0; h < kRows; ++h)
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e) {
            const uint32_t y = x[h][e];
            if (!(y & kJRes) && y >= lo) x[h][e] = (w[h][e] >> (y & 63)) & 1 ? jn[h][e] : kJRes | *po.at(y);
          }
      }
      uint32_t out[kRows];
#pragma unroll
      for (uint32_t h = 0; h < kRows; ++h) {
        const u32x4 y = x[h];
        if (!((y.x | y.w) & kJRes) && y.y == y.x + 1 && y.z == y.x + 2 && y.w == y.x + 3 &&
            (y.x >> a.s_log2) == (y.w >> a.s_log2)) {  // four consecutive settled bytes
          out[h] = *reinterpret_cast<const AX_GLOBAL u32_u*>(po.at(y.x));
        } else {
          out[h] = 0;
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e)
            out[h] |= (y[e] & kJRes ? y[e] & 0xFFu : uint32_t(*po.at(y[e]))) << (8 * e);
        }
      }
#pragma unroll
      for (uint32_t h = 0; h < kRows; ++h) {
        if (!bits[h]) continue;
        const gbytes o = po.at(p[h]);
        if (bits[h] == 0xFu) {
          *reinterpret_cast<AX_GLOBAL uint32_t*>(o) = out[h];
        } else {
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e)
            if ((bits[h] >> e) & 1) o[e] = uint8_t(out[h] >> (8 * e));
        }
      }
    }
  }
}

template <bool kAll>
__global__ __launch_bounds__(kCopyThreads) void k_sweep(SweepArgs a) {
  __shared__ WordQueue queues[kCopyThreads / 64];
  sweep_run<kAll>(a, blockIdx.x, gridDim.x, queues);
}
template <bool kAll>
__global__ __launch_bounds__(kCopyThreads) void k_finish(SweepArgs a) {
  __shared__ WordQueue queues[kCopyThreads / 64];
  finish_part<kAll>(a, blockIdx.x, gridDim.x, queues);
}
// both kinds: the first n_few workgroups (of a sweep a multiple of kXcds) take the blocks that are not marked
__global__ __launch_bounds__(kCopyThreads) void k_sweep_both(SweepArgs a, uint32_t n_few) {
  __shared__ WordQueue queues[kCopyThreads / 64];
  if (blockIdx.x < n_few) sweep_run<false>(a, blockIdx.x, n_few, queues);
  else sweep_run<true>(a, blockIdx.x - n_few, gridDim.x - n_few, queues);
}
__global__ __launch_bounds__(kCopyThreads) void k_finish_both(SweepArgs a, uint32_t n_few) {
  __shared__ WordQueue queues[kCopyThreads / 64];
  if (blockIdx.x < n_few) finish_part<false>(a, blockIdx.x, n_few, queues);
  else finish_part<true>(a, blockIdx.x - n_few, gridDim.x - n_few, queues);
}

// The tokens round 0 left: the sum of its sublist counters (one wave).
__global__ void k_pending0(const uint32_t* cnt, DevStatus* st) {
  uint32_t tot;
  (void)wave_excl_sum(threadIdx.x < kSub ? cnt[threadIdx.x * kCounterStride] : 0u, &tot);
  if (threadIdx.x == 0) st->pend0 = tot;
}

// Status reset before each window (the first also clears the error word).
__device__ inline void window_status_reset(DevStatus* st, int first) {
  if (first) {
    st->err = 0;
    st->bad_block = ~0ull;
  }
  st->ticket = 0;
  st->long_count = 0;
  st->n_pending = 0;
  st->jump_used = 0;
  st->n_jwords = 0;
  st->pend0 = 0;
}

__global__ void k_window_init(DevStatus* st, int first) {
  if (threadIdx.x == 0) window_status_reset(st, first);
}

// Everything a window's match layer needs zeroed or precomputed, in one
// launch before its entropy stage: the status words, the list counters and
// pass flags, the persistent chase's leftover bitmap, and for pointer
// jumping the leftover map (the last round sets its bits) and where every
// window block's output bytes start.  In a mapped plan (one window) also the
// slot table: its blocks take slots 0, 1, ... in window order (as a launch of
// its own: one 16 KiB range 83, now 81 us, 32 mixed ranges 345, now 325).
struct PrepArgs {
  DevStatus* st;
  int first;
  uint32_t* counts;
  uint32_t n_counts;
  uint32_t* pbits;
  uint32_t n_pbits;
  uint64_t* lmap;
  uint64_t n_lmap;
  uint8_t** ibase;  // null: no pointer jumping in this window
  const JobDev* jobs;
  const WinBlock* wbl;
  uint32_t n_items;
};

template <class O>
__global__ __launch_bounds__(kCopyThreads) void k_window_prep(PrepArgs a) {
  if (blockIdx.x == 0 && threadIdx.x == 0) window_status_reset(a.st, a.first);
  const uint64_t i0 = uint64_t(blockIdx.x) * kCopyThreads + threadIdx.x, step = uint64_t(gridDim.x) * kCopyThreads;
  for (uint64_t i = i0; i < a.n_counts; i += step) a.counts[i] = 0;
  for (uint64_t i = i0; i < a.n_pbits; i += step) a.pbits[i] = 0;
  for (uint64_t i = i0; i < a.n_lmap; i += step) a.lmap[i] = 0;
  constexpr bool kMapped = std::is_same<O, OutMapped>::value;
  if (!kMapped && !a.ibase) return;
  for (uint64_t x = i0; x < a.n_items; x += step) {
    const WinBlock wb = a.wbl[x];
    const JobDev& jd = a.jobs[wb.job];
    if (kMapped) gp(jd.slot)[wb.b] = uint32_t(x);
    if (a.ibase) a.ibase[x] = kMapped ? jd.out + x * jd.B : (uint8_t*)(O(jd).at(wb.b * jd.B));
  }
}

// --------------------------------------------------------------- host side --

inline uint64_t align256(uint64_t v) { return (v + 255) & ~255ull; }

}  // namespace

namespace ax {

struct Layout {
  uint64_t status, nsym, lit, cmd, off, len, tok, tblk, cov, done, counts, jflags, list0, list1, llist, pbits, pcnt,
      plist, lmap, amap, ibase, wlist, total;
  uint64_t jbytes;  // the jump array: the stream slots but the commands', dead once the parse is through
  uint64_t sub_cap;
};

// A decode plan: jobs (archives and where their bytes go), cut into windows
// of at most kWindowBlocks blocks.  A window's sources lie in earlier windows
// or inside it, so windows run one after another with bounded scratch.
struct Plan {
  std::vector<JobDev> jobs;
  std::vector<WinBlock> wbl;
  std::vector<uint64_t> gtok;  // per window block: its first token's index in its archive
  struct Win {
    uint64_t at;       // first WinBlock
    uint32_t items;    // blocks
    uint32_t tok;      // tokens
    uint32_t sure, open;  // its first blocks (DeepBlocks)
    uint64_t open_bytes;  // decoded bytes of the open ones
    uint32_t most;        // most blocks of one archive among them all
  };
  std::vector<Win> wins;
  uint32_t max_items = 0, max_tok = 0, slot_b = 0, off_cap = 0, len_cap = 0;
  uint64_t out_bytes = 0, n_tokens = 0;
  void* d_mem = nullptr;
  JobDev* d_jobs = nullptr;
  WinBlock* d_wbl = nullptr;
  JobDev* h_pinned = nullptr;  // staging for refreshing output pointers
  uint8_t* h_stage = nullptr;  // staging for plan_reset uploads
  size_t dev_cap = 0, stage_cap = 0, pinned_cap = 0;
  hipEvent_t staged = nullptr;  // the last upload from h_stage / h_pinned
  std::vector<uint8_t*> dev_out;  // output pointers as last uploaded
  Layout lay{};
  PlanOptions opt{};
  int copy_grid = 1;
  bool timing = false, events_ok = false;
  size_t timed_windows = 0;  // windows the last timed decode recorded
  // stage events, five per window: entropy, parse, bulk rounds, deep
  // remainder, end
  std::vector<hipEvent_t> ev;
  // jump passes launched per window: from a bound on the chain length at
  // first, then the count the device reported as needed (+1 spare pass,
  // which exits at once and reports it again); the gather finishes any
  // entry the passes leave, so the count never changes a byte
  std::vector<uint32_t> jpass;
  // per window, the passes the device reported as needed (0: not known);
  // once every window's count is known the spare pass is dropped
  std::vector<uint32_t> jneed;
  // pinned: per window, the passes that found work and the tokens round 0
  // filled (two words)
  uint32_t* h_jused = nullptr;
  size_t jused_cap = 0;
  hipEvent_t jfed = nullptr;     // h_jused is complete after this
  bool jfeed_pending = false, jsettled = false;
  // bulk rounds per window, learned from round 0's report when the caller
  // left the count to the library: a window whose round 0 fills less than a
  // tenth of its tokens (a deep archive) goes straight to the remainder (0:
  // the configured count)
  std::vector<uint8_t> wbulk;
  bool bulk_auto = true, bsettled = false;
  bool learn = true;             // plans rebuilt for every call (ranges) keep the bound
  bool mapped = false;           // one job whose output is a compact scratch addressed by slot
  hipGraphExec_t graph = nullptr;
  hipGraph_t graph_def = nullptr;
  void* graph_work = nullptr;
  int graph_mode = -1;
  bool graph_stale = false;  // rebuilt at the next decode that may allocate
  hipStream_t cap_stream = nullptr;
  ~Plan() {
    if (graph) (void)hipGraphExecDestroy(graph);
    if (graph_def) (void)hipGraphDestroy(graph_def);
    if (cap_stream) (void)hipStreamDestroy(cap_stream);
    for (auto& e : ev) (void)hipEventDestroy(e);
    if (staged) {
      (void)hipEventSynchronize(staged);
      (void)hipEventDestroy(staged);
    }
    if (jfed) {
      (void)hipEventSynchronize(jfed);
      (void)hipEventDestroy(jfed);
    }
    if (h_jused) (void)hipHostFree(h_jused);
    if (d_mem) (void)hipFree(d_mem);
    if (h_pinned) (void)hipHostFree(h_pinned);
    if (h_stage) (void)hipHostFree(h_stage);
  }
};

static Layout make_layout(const Plan& P) {
  Layout L{};
  const uint64_t W = std::max<uint32_t>(1, P.max_items), T = std::max<uint32_t>(1, P.max_tok);
  uint64_t at = 0;
  L.status = at, at = align256(at + sizeof(DevStatus));
  L.nsym = at, at = align256(at + 16 * W);
  L.cmd = at, at = align256(at + W * P.slot_b);
  L.lit = at, at = align256(at + W * P.slot_b);
  L.off = at, at = align256(at + W * P.off_cap);
  L.len = at, at = align256(at + W * P.len_cap);
  L.tok = at, at = align256(at + 16 * T);
  L.tblk = at, at = align256(at + 4 * T);
  L.cov = at, at = align256(at + 8 * T);
  L.done = at, at = align256(at + T);
  L.counts = at, at = align256(at + 4ull * 3 * kSub * kCounterStride);
  L.jflags = at, at = align256(at + 4ull * kJPasses * kJShards * kJFlagStride);  // cleared with the counters
  // a round over n <= T items launches G = min(ceil(T / 256), kMaxRoundGrid)
  // workgroups, each visiting at most ceil(n / (256 G)) * 256 items, and
  // sublist s takes the items of the ceil(G / kSub) workgroups g = s mod kSub:
  // at most n / kSub + 4 G + n / G + 256 <= ceil(T / kSub) + 256 (ceil(G /
  // kSub) + 2) (leftovers filed by token group, (t / 64) mod kSub, stay
  // within ceil(T / kSub) + 64)
  const uint64_t G = std::min<uint64_t>((T + kCopyThreads - 1) / kCopyThreads, kMaxRoundGrid);
  L.sub_cap = (T + kSub - 1) / kSub + uint64_t(kCopyThreads) * ((G + kSub - 1) / kSub + 2);
  L.list0 = at, at = align256(at + 4 * kSub * L.sub_cap);
  L.list1 = at, at = align256(at + 4 * kSub * L.sub_cap);
  L.llist = at, at = align256(at + 4 * T);
  L.pbits = at, at = align256(at + 4 * ((T + 31) / 32 + 64));
  L.pcnt = at, at = align256(at + 4 * ((T + 31) / 32 / kPackWords + 1));
  L.plist = at, at = align256(at + 4 * T);
  L.lmap = at, at = align256(at + W * P.slot_b / 8);
  L.ibase = at, at = align256(at + 8 * W);
  L.wlist = at, at = align256(at + W * P.slot_b / 16);                        // one u32 per map word
  L.amap = at, at = align256(at + W * P.slot_b / 8);
  L.total = at;
  // the jump array (4 B per window position) reuses the literal, offset and
  // length slots, dead once the parse is through: at least 4 B per window
  // position (the command slots hold the records by then)
  L.jbytes = L.len + W * P.len_cap - L.lit;
  return L;
}

static int hip_fail(hipError_t e, const char* what) {
  (void)what;
  return fail(AX_E_HIP, hipGetErrorString(e));
}

static void launch_ans(const AnsArgs& aa, hipStream_t s) {
  if (aa.n_items <= kWideBlocks) hipLaunchKernelGGL(k_ans<true>, dim3(4 * aa.n_items), dim3(64), 0, s, aa);
  else hipLaunchKernelGGL(k_ans<false>, dim3(4 * aa.n_items), dim3(64), 0, s, aa);
}

// Jump passes that resolve any chain of a window of `tok` tokens: a chain
// visits each pending token at most once, the first entries span one hop,
// and a pass triples the hops an entry spans.
static uint32_t jump_pass_bound(uint64_t tok) {
  uint32_t p = 1;
  uint64_t span = 3;
  while (p < kJPasses && span <= tok) ++p, span *= 3;
  return p;
}

// Archives taken to be deep: with a match per kDenseSpan bytes or more and less
// than kDenseMatch payload bytes a match.  A match costs three to five, so little
// is left for literals, most bytes are copies, and chains follow.  Marking costs
// four bytes of jump array per position, so where few bytes are copied walks win.
// 64 MiB marked and walked: text (7 payload bytes a match) 526 and 1279 us, log
// lines (4) 681 and 2242, rows that repeat the row before (4) 708 and 1831, text
// with every twentieth byte replaced (8, ratio 2.4) 584 and 1697; DNA (30) 439 and
// 242, protein (45) 416 and 241, 32 MiB of reads (25) 258 and 238.
// Of other archives, those of ratio kDeepRatio and more may owe it to the entropy
// coder, and those under kOpenMatch payload bytes a match may be either; they are
// marked if one byte in kCopiedShare is a copy (open): uniform ACGT (9 % copies) 394
// and 170, three symbols (26 %) 495 and 306, ACGT with blocks of text (24 / 36 / 69 %)
// 441 and 373, 461 and 489, 518 and 1021; log lines with long random fields (53 %)
// 481 and 985, zero pages among random ones (72 %) 416 and 540, text with matches of
// 16 and more 425 and 672.  Asking costs 3 to 6 %.
// In small plans the marking is cheap and its shorter chain of loads counts: 64
// KiB / 4 MiB of DNA 94 / 122 us marked and 140 / 148 walked.  Between 8 and 16 MiB
// it depends on the data: 12 MiB of DNA 121 and 136, but 16 MiB of protein 120 and
// 104, 10 MiB of DNA in 4 KiB blocks 140 and 115.
constexpr uint64_t kDeepRatio = 3;
constexpr uint64_t kDenseSpan = 256, kDenseMatch = 10, kOpenMatch = 20;
constexpr uint64_t kBlockOverhead = 64;  // payload bytes of a block that holds nothing
constexpr uint64_t kCopiedShare = 3;
constexpr uint64_t kDeepSmall = 8u << 20;  // positions of a small plan
// Marked blocks are finished run by run (eight launches, each reading settled
// bytes) where chains cross several runs: an archive of so many positions, and
// more than half of the window's.  Otherwise one launch follows the entries.  Whole
// decodes of text in eight launches and in one: 8 MiB 127 and 110 us, 16 MiB 167
// and 168, 24 MiB 207 and 227, 32 MiB 250 and 288, with 4, 8 or 16 KiB blocks; 24
// / 80 MiB and a small archive 234 and 245, 690 and 794.  Chains end in their own
// archive: two / four of 12 MiB 220 and 201, 404 and 369, two of 40 677 and 665,
// 100 of 1 875 and 849; one of 40 and eight of 4 631 and 638.
constexpr uint64_t kPartPositions = 16u << 20;

// Host tables of a plan: jobs, window blocks, windows, maxima.
static int build_tables(Plan* P, const std::vector<JobSpec>& specs) {
  try {
    P->jobs.assign(specs.size(), JobDev{});
    P->wbl.clear();
    P->gtok.clear();
    P->wins.clear();
    P->max_items = P->max_tok = P->slot_b = P->off_cap = P->len_cap = 0;
    P->out_bytes = P->n_tokens = 0;
    uint64_t gblocks = 0;
    for (size_t j = 0; j < specs.size(); ++j) {
      const aceapex_decoder* d = specs[j].dec;
      const aceapex_info& I = d->info;
      JobDev& J = P->jobs[j];
      J.arc = d->d_arc;
      J.out = specs[j].out;
      J.payload_at = I.header_bytes;
      J.n_bytes = I.n_bytes;
      J.nb = I.n_blocks;
      J.B = I.block_size;
      J.mm = I.min_match;
      J.slot = specs[j].slot;
      J.junk = specs[j].junk;
      P->slot_b = std::max(P->slot_b, I.block_size);
      P->off_cap = std::max(P->off_cap, uint32_t((10 * (I.block_size / I.min_match + 1) + 15) & ~15u));
      P->len_cap = std::max(P->len_cap, 3 * I.block_size);
      P->out_bytes += I.n_bytes;
      gblocks += specs[j].blocks.empty() ? I.n_blocks : specs[j].blocks.size();
    }
    P->wbl.reserve(gblocks);
    P->gtok.reserve(gblocks);
    // windows: consecutive (job, block) items, at most kWindowBlocks blocks
    // and kWindowTokens tokens each
    Plan::Win cur{};
    auto close = [&]() {
      if (!cur.items) return;
      for (uint64_t i = cur.at; i < cur.at + cur.items;) {  // per-job extents inside the window
        uint64_t k = i;
        while (k < cur.at + cur.items && P->wbl[k].job == P->wbl[i].job) ++k;
        for (uint64_t m = i; m < k; ++m) {
          P->wbl[m].first = uint32_t(i - cur.at);
          P->wbl[m].count = uint32_t(k - i);
        }
        if (i - cur.at < cur.sure + cur.open) cur.most = std::max(cur.most, uint32_t(k - i));
        i = k;
      }
      P->max_items = std::max(P->max_items, cur.items);
      P->max_tok = std::max(P->max_tok, cur.tok);
      P->n_tokens += cur.tok;
      P->wins.push_back(cur);
      cur = Plan::Win{};
      cur.at = P->wbl.size();
    };
    // jobs enter the windows deep archives first, then those that may be, then
    // densest first (matches per block): a window runs as long as its deepest
    // dependency chain, and match-dense archives carry the deep chains, so they
    // share windows instead of lengthening every one
    const bool small = gblocks * P->slot_b <= kDeepSmall;
    auto shallow = [&](size_t j) {  // 0 deep, 1 open, 2 not
      const aceapex_info& I = specs[j].dec->info;
      auto dense = [&](uint64_t per) {  // matches all over, at less than `per` payload bytes each
        return I.n_matches >= I.n_bytes / kDenseSpan && I.payload_bytes < I.n_blocks * kBlockOverhead + I.n_matches * per;
      };
      if (small || dense(kDenseMatch)) return 0;
      return I.payload_bytes < I.n_bytes / kDeepRatio || dense(kOpenMatch) ? 1 : 2;
    };
    std::vector<size_t> order(specs.size());
    for (size_t j = 0; j < order.size(); ++j) order[j] = j;
    auto density = [&](size_t j) {
      const aceapex_decoder* d = specs[j].dec;
      return d->info.n_blocks ? double(d->mpre[d->info.n_blocks]) / double(d->info.n_blocks) : 0.0;
    };
    std::stable_sort(order.begin(), order.end(), [&](size_t x, size_t y) {
      return shallow(x) != shallow(y) ? shallow(x) < shallow(y) : density(x) > density(y);
    });
    for (const size_t j : order) {
      const aceapex_decoder* d = specs[j].dec;
      const uint64_t nb = specs[j].blocks.empty() ? d->info.n_blocks : specs[j].blocks.size();
      const int kind = shallow(j);
      for (uint64_t i = 0; i < nb; ++i) {
        const uint64_t b = specs[j].blocks.empty() ? i : specs[j].blocks[i];
        if (b >= d->info.n_blocks) return fail(AX_E_RANGE, "block outside the archive");
        const uint64_t nt = d->mpre[b + 1] - d->mpre[b];
        if (cur.items == kWindowBlocks || uint64_t(cur.tok) + nt > kWindowTokens) close();
        P->wbl.push_back(WinBlock{b, uint32_t(j), cur.tok, 0, 0});
        P->gtok.push_back(d->mpre[b]);
        cur.items++;
        cur.sure += kind == 0;
        cur.open += kind == 1;
        if (kind == 1) cur.open_bytes += std::min<uint64_t>(d->info.block_size, d->info.n_bytes - b * d->info.block_size);
        cur.tok += uint32_t(nt);
      }
    }
    close();
    P->mapped = !specs.empty() && specs[0].slot != nullptr;
    P->jpass.assign(P->wins.size(), 0);
    for (size_t i = 0; i < P->wins.size(); ++i) P->jpass[i] = jump_pass_bound(P->wins[i].tok);
    P->jneed.assign(P->wins.size(), 0);
    P->jsettled = false;
    P->wbulk.assign(P->wins.size(), 0);
    P->bsettled = false;
  } catch (const std::bad_alloc&) {
    return fail(AX_E_NOMEM, "plan tables");
  }
  P->lay = make_layout(*P);
  return AX_OK;
}

static size_t table_bytes(const Plan* P, size_t* wbl_at) {
  const size_t jb = sizeof(JobDev) * std::max<size_t>(1, P->jobs.size());
  *wbl_at = align256(jb);
  return *wbl_at + sizeof(WinBlock) * std::max<size_t>(1, P->wbl.size());
}

// Device tables big enough for the current host tables (grown when needed).
static int ensure_device(Plan* P) {
  size_t wbl_at;
  const size_t need = table_bytes(P, &wbl_at);
  if (need > P->dev_cap) {
    if (P->d_mem) (void)hipFree(P->d_mem), P->d_mem = nullptr;
    const size_t cap = std::max(need, 2 * P->dev_cap);
    hipError_t e = hipMalloc(&P->d_mem, cap);
    if (e != hipSuccess) return hip_fail(e, "plan memory");
    P->dev_cap = cap;
  }
  const size_t jb = sizeof(JobDev) * std::max<size_t>(1, P->jobs.size());
  if (jb > P->pinned_cap) {
    if (P->h_pinned) (void)hipHostFree(P->h_pinned), P->h_pinned = nullptr;
    hipError_t e = hipHostMalloc(reinterpret_cast<void**>(&P->h_pinned), jb);
    if (e != hipSuccess) return hip_fail(e, "plan staging");
    P->pinned_cap = jb;
  }
  P->d_jobs = static_cast<JobDev*>(P->d_mem);
  P->d_wbl = reinterpret_cast<WinBlock*>(static_cast<uint8_t*>(P->d_mem) + wbl_at);
  if (!P->staged) {
    hipError_t e = hipEventCreateWithFlags(&P->staged, hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(e, "plan event");
  }
  // the jump-pass report of every window, so that a decode allocates nothing
  if (P->wins.size() > P->jused_cap) {
    if (P->jfeed_pending) (void)hipEventSynchronize(P->jfed), P->jfeed_pending = false;
    if (P->h_jused) (void)hipHostFree(P->h_jused), P->h_jused = nullptr;
    P->jused_cap = 0;
    hipError_t e = hipHostMalloc(reinterpret_cast<void**>(&P->h_jused), 8 * P->wins.size());
    if (e != hipSuccess) return hip_fail(e, "pass report staging");
    P->jused_cap = P->wins.size();
  }
  if (!P->jfed) {
    hipError_t e = hipEventCreateWithFlags(&P->jfed, hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(e, "pass report event");
  }
  return AX_OK;
}

static int device_setup(Plan* P) {
  int dev = 0, cus = 0, occ = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, reinterpret_cast<const void*>(k_tail<OutDirect>), kCopyThreads, 0);
  P->copy_grid = std::max(1, cus) * std::max(1, occ);
  return AX_OK;
}

int plan_create(const std::vector<JobSpec>& specs, Plan** out) {
  *out = nullptr;
  Plan* P = new (std::nothrow) Plan;
  if (!P) return fail(AX_E_NOMEM, "plan");
  int rc = build_tables(P, specs);
  if (!rc) rc = ensure_device(P);
  if (rc) {
    delete P;
    return rc;
  }
  hipError_t e = hipMemcpy(P->d_jobs, P->jobs.data(), sizeof(JobDev) * P->jobs.size(), hipMemcpyHostToDevice);
  if (e == hipSuccess && !P->wbl.empty())
    e = hipMemcpy(P->d_wbl, P->wbl.data(), sizeof(WinBlock) * P->wbl.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    delete P;
    return hip_fail(e, "plan upload");
  }
  P->dev_out.resize(P->jobs.size());
  for (size_t j = 0; j < P->jobs.size(); ++j) P->dev_out[j] = P->jobs[j].out;
  device_setup(P);
  *out = P;
  return AX_OK;
}

int plan_reset(Plan* P, const std::vector<JobSpec>& specs, hipStream_t s) {
  // staging may still feed the previous upload; a pass report of the old
  // windows may still be on its way
  if (P->staged) (void)hipEventSynchronize(P->staged);
  if (P->jfeed_pending) (void)hipEventSynchronize(P->jfed), P->jfeed_pending = false;
  int rc = build_tables(P, specs);
  if (!rc) rc = ensure_device(P);
  if (rc) return rc;
  size_t wbl_at;
  const size_t bytes = table_bytes(P, &wbl_at);
  if (bytes > P->stage_cap) {
    if (P->h_stage) (void)hipHostFree(P->h_stage), P->h_stage = nullptr;
    const size_t cap = std::max(bytes, 2 * P->stage_cap);
    hipError_t e = hipHostMalloc(reinterpret_cast<void**>(&P->h_stage), cap);
    if (e != hipSuccess) return hip_fail(e, "plan staging");
    P->stage_cap = cap;
  }
  std::memcpy(P->h_stage, P->jobs.data(), sizeof(JobDev) * P->jobs.size());
  if (!P->wbl.empty()) std::memcpy(P->h_stage + wbl_at, P->wbl.data(), sizeof(WinBlock) * P->wbl.size());
  hipError_t e = hipMemcpyAsync(P->d_mem, P->h_stage, bytes, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipEventRecord(P->staged, s);
  if (e != hipSuccess) return hip_fail(e, "plan upload");
  P->dev_out.resize(P->jobs.size());
  for (size_t j = 0; j < P->jobs.size(); ++j) P->dev_out[j] = P->jobs[j].out;
  if (P->graph) (void)hipGraphExecDestroy(P->graph), P->graph = nullptr;  // tables changed
  if (!P->copy_grid || P->copy_grid == 1) device_setup(P);
  return AX_OK;
}

static bool roots_schedule(const Plan* P, int copy_mode);

uint64_t plan_workspace_for(const aceapex_decoder* d, uint64_t max_blocks, uint64_t max_tokens) {
  Plan P;
  P.max_items = uint32_t(max_blocks);
  P.max_tok = uint32_t(max_tokens);
  P.slot_b = d->info.block_size;
  P.off_cap = uint32_t((10 * (d->info.block_size / d->info.min_match + 1) + 15) & ~15u);
  P.len_cap = 3 * d->info.block_size;
  return make_layout(P).total;
}

void plan_copy_options(Plan* dst, const Plan* src) { dst->opt = src->opt; }

int plan_check_mapped(const Plan* P) {
  return P->wins.size() > 1 ? fail(AX_E_CAPACITY, "a mapped plan holds one window") : AX_OK;
}
bool plan_roots(const Plan* P) { return roots_schedule(P, AX_COPY_PERIODIC); }
void plan_set_learn(Plan* P, bool learn) { P->learn = learn; }

int plan_parse_tokens(Plan* P, void* d_work, uint64_t work_len, hipStream_t s, uint64_t* src, uint64_t* dstlen) {
  if (work_len < P->lay.total) return fail(AX_E_CAPACITY, "workspace too small");
  uint8_t* w = static_cast<uint8_t*>(d_work);
  const Layout& L = P->lay;
  DevStatus* st = reinterpret_cast<DevStatus*>(w + L.status);
  bool stale = false;
  for (size_t j = 0; j < P->jobs.size(); ++j) stale |= P->dev_out[j] != P->jobs[j].out;
  if (stale) {
    hipError_t e = hipMemcpy(P->d_jobs, P->jobs.data(), sizeof(JobDev) * P->jobs.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e, "job table update");
    for (size_t j = 0; j < P->jobs.size(); ++j) P->dev_out[j] = P->jobs[j].out;
  }
  std::vector<uint64_t> tk;
  if (P->wins.empty()) hipLaunchKernelGGL(k_window_init, dim3(1), dim3(64), 0, s, st, 1);  // status only
  for (const Plan::Win& W : P->wins) {
    const WinBlock* wbl = P->d_wbl + W.at;
    hipLaunchKernelGGL(k_window_init, dim3(1), dim3(64), 0, s, st, int(&W == &P->wins.front()));
    AnsArgs aa{P->d_jobs, wbl, W.items, P->slot_b, w + L.lit, w + L.cmd, w + L.off, w + L.len, P->off_cap,
               P->len_cap, reinterpret_cast<uint32_t*>(w + L.nsym), st};
    launch_ans(aa, s);
    ParseArgs pa{P->d_jobs, wbl, W.items, W.tok, P->slot_b, w + L.lit, w + L.cmd, w + L.off, w + L.len, P->off_cap,
                 P->len_cap, reinterpret_cast<const uint32_t*>(w + L.nsym), reinterpret_cast<uint64_t*>(w + L.tok),
                 nullptr, nullptr, st, 0};
    hipLaunchKernelGGL((k_parse<OutDirect, 0, kParseThreads>), dim3(W.items), dim3(kParseThreads), 0, s, pa);
    try {
      tk.resize(2ull * W.tok);
    } catch (const std::bad_alloc&) {
      return fail(AX_E_NOMEM, "token staging");
    }
    hipError_t e = W.tok ? hipMemcpyAsync(tk.data(), w + L.tok, 16ull * W.tok, hipMemcpyDeviceToHost, s) : hipSuccess;
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "token copy");
    int32_t err = 0;
    uint64_t bad = 0;
    int rc = workspace_status(d_work, s, &err, &bad);
    if (rc) return rc;
    if (err) return fail(err, "device status during the index build");
    // window tokens are the tokens of its blocks in order
    for (uint32_t i = 0; i < W.items; ++i) {
      const WinBlock& wb = P->wbl[W.at + i];
      const uint32_t end = i + 1 < W.items ? P->wbl[W.at + i + 1].tok : W.tok;
      const uint64_t g0 = P->gtok[W.at + i];
      for (uint32_t t = wb.tok; t < end; ++t) {
        src[g0 + (t - wb.tok)] = tk[2ull * t];
        dstlen[g0 + (t - wb.tok)] = tk[2ull * t + 1];
      }
    }
  }
  return AX_OK;
}
int block_streams(const aceapex_decoder* d, uint64_t first, uint64_t count, void* d_work, uint64_t work_len,
                  hipStream_t s, uint8_t* h_out, uint64_t cap, uint32_t* n_syms) {
  if (count == 0) return AX_OK;
  if (first >= d->info.n_blocks || count > d->info.n_blocks - first || count > kWindowBlocks)
    return fail(AX_E_RANGE, "blocks outside the archive or beyond one window");
  std::vector<uint64_t> bl(count);
  for (uint64_t i = 0; i < count; ++i) bl[i] = first + i;
  Plan* P = nullptr;
  int rc = plan_create({JobSpec{d, nullptr, std::move(bl)}}, &P);
  if (rc) return rc;
  struct Guard {
    Plan* p;
    ~Guard() { delete p; }
  } guard{P};
  if (work_len < P->lay.total) return fail(AX_E_CAPACITY, "workspace too small");
  if (reinterpret_cast<uintptr_t>(d_work) & 255) return fail(AX_E_ARG, "workspace must be 256-byte aligned");
  uint8_t* w = static_cast<uint8_t*>(d_work);
  const Layout& L = P->lay;
  DevStatus* st = reinterpret_cast<DevStatus*>(w + L.status);
  const Plan::Win& W = P->wins.front();
  hipLaunchKernelGGL(k_window_init, dim3(1), dim3(64), 0, s, st, 1);
  AnsArgs aa{P->d_jobs, P->d_wbl, W.items, P->slot_b, w + L.lit, w + L.cmd, w + L.off, w + L.len, P->off_cap,
             P->len_cap, reinterpret_cast<uint32_t*>(w + L.nsym), st};
  launch_ans(aa, s);
  hipError_t e = hipMemcpyAsync(n_syms, w + L.nsym, 16 * count, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "stream counts");
  int32_t err = 0;
  uint64_t bad = 0;
  rc = workspace_status(d_work, s, &err, &bad);
  if (rc) return rc;
  if (err) return fail(err, "device status of the entropy stage");
  // packed: per block LIT, LEN, OFF, CMD (the slot order of the counts)
  const uint64_t at[4] = {L.lit, L.len, L.off, L.cmd};
  const uint64_t stride[4] = {P->slot_b, P->len_cap, P->off_cap, P->slot_b};
  uint64_t need = 0;
  for (uint64_t i = 0; i < 4 * count; ++i) need += n_syms[i];
  if (need > cap) return fail(AX_E_CAPACITY, "host buffer smaller than the streams");
  uint64_t o = 0;
  for (uint64_t i = 0; i < count && e == hipSuccess; ++i)
    for (int k = 0; k < 4 && e == hipSuccess; ++k) {
      const uint32_t n = n_syms[4 * i + k];
      if (n) e = hipMemcpyAsync(h_out + o, w + at[k] + i * stride[k], n, hipMemcpyDeviceToHost, s);
      o += n;
    }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  return e == hipSuccess ? AX_OK : hip_fail(e, "stream copy");
}

void plan_destroy(Plan* P) { delete P; }
uint64_t plan_workspace(const Plan* P) { return P->lay.total; }
uint64_t plan_tokens(const Plan* P) { return P->n_tokens; }
uint64_t plan_blocks(const Plan* P) { return P->wbl.size(); }

int plan_set_out(Plan* P, size_t job, uint8_t* out) {
  if (job >= P->jobs.size()) return fail(AX_E_ARG, "job index");
  P->jobs[job].out = out;
  return AX_OK;
}

int plan_set_option(Plan* P, int option, int64_t value) {
  switch (option) {
    case AX_OPT_BULK_ROUNDS:
      if (value < 1 || value > 250) return fail(AX_E_ARG, "bulk rounds must be in [1, 250]");
      P->opt.bulk_rounds = int(value);
      P->bulk_auto = false;
      std::fill(P->wbulk.begin(), P->wbulk.end(), uint8_t(0));
      break;
    case AX_OPT_TAIL_CHUNKS:
      if (value < 1 || value > 64) return fail(AX_E_ARG, "tail chunks must be in [1, 64]");
      P->opt.tail_chunks = int(value);
      break;
    case AX_OPT_ROUND0_TILE:
      if (value < 0 || value > 1) return fail(AX_E_ARG, "round-0 schedule must be 0 or 1");
      P->opt.round0_tile = int(value);
      break;
    case AX_OPT_FILL_ROUNDS:
    case AX_OPT_FILL_TAIL:
      if (value < 0 || value > 1) return fail(AX_E_ARG, "fill mode must be 0 or 1");
      (option == AX_OPT_FILL_ROUNDS ? P->opt.fill_round : P->opt.fill_tail) = int(value);
      break;
    case AX_OPT_GRAPH:
      if (value < 0 || value > 1) return fail(AX_E_ARG, "graph must be 0 or 1");
      P->opt.graph = int(value);
      break;
    case AX_OPT_TAIL_MODE:
      if (value < 0 || value > 1) return fail(AX_E_ARG, "tail mode must be 0 or 1");
      P->opt.tail_mode = int(value);
      break;
    case AX_OPT_JUMP_PASSES:
      if (value < 0 || value > int64_t(kJPasses)) return fail(AX_E_ARG, "jump passes must be in [0, 32]");
      P->opt.jump_passes = int(value);
      break;
    case AX_OPT_RANGE_JUMP_TOKENS:
      if (value < 0 || value > int64_t(kWindowTokens)) return fail(AX_E_ARG, "range jump tokens out of range");
      P->opt.range_jump_tokens = value;
      break;
    case AX_OPT_SCHEDULE:
      if (value < 0 || value > 2) return fail(AX_E_ARG, "schedule must be 0, 1 or 2");
      P->opt.schedule = int(value);
      break;
    default:
      return fail(AX_E_ARG, "unknown option");
  }
  if (option == AX_OPT_RANGE_JUMP_TOKENS) P->opt.range_knob_set = true;
  else if (option != AX_OPT_GRAPH && option != AX_OPT_SCHEDULE) P->opt.knob_set = true;
  if (P->graph) {  // knobs are baked into a captured graph
    (void)hipGraphExecDestroy(P->graph);
    P->graph = nullptr;
  }
  return AX_OK;
}

int plan_get_option(const Plan* P, int option, int64_t* value) {
  switch (option) {
    case AX_OPT_BULK_ROUNDS: *value = P->opt.bulk_rounds; return AX_OK;
    case AX_OPT_TAIL_CHUNKS: *value = P->opt.tail_chunks; return AX_OK;
    case AX_OPT_ROUND0_TILE: *value = P->opt.round0_tile; return AX_OK;
    case AX_OPT_FILL_ROUNDS: *value = P->opt.fill_round; return AX_OK;
    case AX_OPT_FILL_TAIL: *value = P->opt.fill_tail; return AX_OK;
    case AX_OPT_GRAPH: *value = P->opt.graph; return AX_OK;
    case AX_OPT_TAIL_MODE: *value = P->opt.tail_mode; return AX_OK;
    case AX_OPT_JUMP_PASSES: *value = P->opt.jump_passes; return AX_OK;
    case AX_OPT_RANGE_JUMP_TOKENS: *value = P->opt.range_jump_tokens; return AX_OK;
    case AX_OPT_SCHEDULE: *value = P->opt.schedule; return AX_OK;
    default: return fail(AX_E_ARG, "unknown option");
  }
}

// Stage events for every window of the plan (created when timing is on).
static int ensure_events(Plan* P) {
  const size_t need = 5 * P->wins.size();
  while (P->ev.size() < need) {
    hipEvent_t e;
    hipError_t er = hipEventCreate(&e);
    if (er != hipSuccess) return hip_fail(er, "hipEventCreate");
    P->ev.push_back(e);
  }
  return AX_OK;
}

int plan_set_timing(Plan* P, int enable) {
  if (enable && !P->events_ok) {
    int rc = ensure_events(P);
    if (rc) return rc;
    P->events_ok = true;
  }
  P->timing = enable != 0;
  return AX_OK;
}

int plan_stage_ms(Plan* P, float* ans, float* parse, float* copy, float* remainder) {
  if (!P->events_ok || P->timed_windows == 0) return fail(AX_E_ARG, "timing not enabled");
  float t[4] = {0, 0, 0, 0};
  for (size_t wi = 0; wi < P->timed_windows; ++wi) {
    hipEvent_t* e = P->ev.data() + 5 * wi;
    hipError_t er = hipEventSynchronize(e[4]);
    if (er != hipSuccess) return hip_fail(er, "hipEventSynchronize");
    for (int k = 0; k < 4; ++k) {
      float ms = 0;
      (void)hipEventElapsedTime(&ms, e[k], e[k + 1]);
      t[k] += ms;
    }
  }
  *ans = t[0];
  *parse = t[1];
  *copy = t[2] + t[3];
  if (remainder) *remainder = t[3];
  return AX_OK;
}

// Whether a decode runs the roots schedule (k_roots): the default one, until the
// caller sets a knob of the rounds (a value that is the default one included: it
// asks for so many rounds, not for none) or names the schedule.  The serial copy
// mode is one of rounds.
static bool roots_schedule(const Plan* P, int copy_mode) {
  const PlanOptions& o = P->opt;
  if (copy_mode != AX_COPY_PERIODIC || o.schedule == 2) return false;
  return o.schedule == 1 || !(o.knob_set || (P->mapped && o.range_knob_set));
}

// The roots match layer of one window.
template <class O>
static void enqueue_roots(Plan* P, const Plan::Win& W, const WinBlock* wbl, uint8_t* w, hipStream_t s, hipEvent_t* ev) {
  const Layout& L = P->lay;
  DevStatus* st = reinterpret_cast<DevStatus*>(w + L.status);
  const uint32_t s_log2 = uint32_t(__builtin_ctz(P->slot_b));
  uint32_t* J = reinterpret_cast<uint32_t*>(w + L.lit);  // the stream slots, dead once the parse is through
  uint64_t* lmap = reinterpret_cast<uint64_t*>(w + L.lmap);
  const uint32_t deep = W.sure + W.open, walks = W.items - W.sure;  // marked and walked blocks, the open ones in both
  const DeepBlocks db{W.sure, W.open, uint32_t(W.open_bytes / kCopiedShare), reinterpret_cast<const uint32_t*>(w + L.counts)};
  const RootArgs ra{P->d_jobs, wbl, W.items, W.tok, s_log2, reinterpret_cast<const uint64_t*>(w + L.tok), w + L.cmd,
                    J, lmap, st, db, uint64_t(deep) << s_log2 <= kDeepSmall ? kMarkSmallLog2 : kMarkLog2};
  const uint32_t marks = deep << (s_log2 - ra.mark_log2);
  const bool both = deep && walks;
  if (both) hipLaunchKernelGGL(k_settle<O>, dim3(W.items - deep + marks), dim3(kCopyThreads), 0, s, ra);
  else if (deep) hipLaunchKernelGGL(k_mark<O>, dim3(marks), dim3(kCopyThreads), 0, s, ra);
  else hipLaunchKernelGGL(k_roots<O>, dim3(walks), dim3(kCopyThreads), 0, s, ra);
  if (ev) (void)hipEventRecord(ev[3], s);
  SweepArgs sa{s_log2, J, lmap, P->d_jobs, wbl, P->jobs.size() == 1 ? 1u : 0u,
               reinterpret_cast<uint8_t* const*>(w + L.ibase), st, W.items, db, kXcds};
  // workgroups of a sweep or finish over n blocks: a wave per chunk of map words
  auto grid_of = [&](uint32_t n, uint32_t chunk) {
    const uint64_t waves = (uint64_t(n) << (s_log2 - 6)) / chunk;
    return std::max(1u, uint32_t(std::min<uint64_t>((waves + 3) / 4, kSweepGrid)));
  };
  auto whole = [](uint32_t grid) { return (grid + kXcds - 1) / kXcds * kXcds; };
  const uint32_t g_all = deep ? whole(grid_of(deep, kAllChunk)) : 0;
  const uint32_t f_few = walks ? grid_of(walks, kFewChunk) : 0, g_few = whole(f_few);
  if (both) hipLaunchKernelGGL(k_sweep_both, dim3(g_few + g_all), dim3(kCopyThreads), 0, s, sa, g_few);
  else if (deep) hipLaunchKernelGGL(k_sweep<true>, dim3(g_all), dim3(kCopyThreads), 0, s, sa);
  else hipLaunchKernelGGL(k_sweep<false>, dim3(g_few), dim3(kCopyThreads), 0, s, sa);
  const uint32_t f_all = deep ? grid_of(deep, kFinishWords) : 0;
  if (uint64_t(W.most) << s_log2 >= kPartPositions && W.most > deep / 2) {
    for (uint32_t k = 0; k < kXcds; ++k) {
      SweepArgs part = sa;
      part.part = k;
      hipLaunchKernelGGL(k_finish<true>, dim3(f_all), dim3(kCopyThreads), 0, s, part);
    }
    if (walks) hipLaunchKernelGGL(k_finish<false>, dim3(f_few), dim3(kCopyThreads), 0, s, sa);
  } else if (both) {
    hipLaunchKernelGGL(k_finish_both, dim3(f_few + f_all), dim3(kCopyThreads), 0, s, sa, f_few);
  } else if (deep) {
    hipLaunchKernelGGL(k_finish<true>, dim3(f_all), dim3(kCopyThreads), 0, s, sa);
  } else {
    hipLaunchKernelGGL(k_finish<false>, dim3(f_few), dim3(kCopyThreads), 0, s, sa);
  }
}

// Enqueue the plan's kernels on s (also used inside a graph capture).
template <class O>
static void enqueue_out(Plan* P, uint8_t* w, int copy_mode, hipStream_t s, bool timed, bool feedback) {
  const Layout& L = P->lay;
  DevStatus* st = reinterpret_cast<DevStatus*>(w + L.status);
  if (P->wins.empty()) hipLaunchKernelGGL(k_window_init, dim3(1), dim3(64), 0, s, st, 1);  // status only
  for (size_t wi = 0; wi < P->wins.size(); ++wi) {
    const Plan::Win& W = P->wins[wi];
    const bool first = wi == 0;
    const WinBlock* wbl = P->d_wbl + W.at;
    uint32_t* counts = reinterpret_cast<uint32_t*>(w + L.counts);
    const uint32_t ntok = W.tok;
    const bool roots = roots_schedule(P, copy_mode);
    const bool jump = P->opt.tail_mode == 0 && copy_mode != AX_COPY_SERIAL;
    const uint32_t n_words = (ntok + 31) / 32;
    const uint64_t mwords = uint64_t(W.items) * (P->slot_b / 64);  // leftover-map words
    // eight listed words per wave step, four waves per workgroup
    const uint32_t jgrid = uint32_t(std::min<uint64_t>((mwords + 31) / 32, kJMaxGrid));
    {
      const bool jmap = jump && ntok;
      const uint32_t n_counts = uint32_t((L.jflags - L.counts) / 4 + kJPasses * kJShards * kJFlagStride);
      const PrepArgs pr{st, int(first), counts, !roots ? n_counts : W.open ? kCopiedShards * kCounterStride : 0u, reinterpret_cast<uint32_t*>(w + L.pbits),
                        ntok && !roots ? n_words : 0u, reinterpret_cast<uint64_t*>(w + L.lmap), jmap && !roots ? mwords : 0u,
                        jmap && !(roots && P->jobs.size() == 1) ? reinterpret_cast<uint8_t**>(w + L.ibase) : nullptr, P->d_jobs,
                        wbl, W.items};
      const uint32_t pgrid = roots ? (W.items + kCopyThreads - 1) / kCopyThreads : jgrid;
      hipLaunchKernelGGL(k_window_prep<O>, dim3(std::max(1u, pgrid)), dim3(kCopyThreads), 0, s, pr);
    }
    AnsArgs aa{P->d_jobs, wbl, W.items, P->slot_b, w + L.lit, w + L.cmd, w + L.off, w + L.len, P->off_cap,
               P->len_cap, reinterpret_cast<uint32_t*>(w + L.nsym), st};
    hipEvent_t* ev = timed ? P->ev.data() + 5 * wi : nullptr;
    if (ev) (void)hipEventRecord(ev[0], s);
    launch_ans(aa, s);
    if (ev) (void)hipEventRecord(ev[1], s);
    const int bulk = P->wbulk[wi] ? int(P->wbulk[wi]) : P->opt.bulk_rounds;
    const bool recs = roots || bulk <= 1;
    ParseArgs pa{P->d_jobs, wbl, W.items, W.tok, P->slot_b, w + L.lit, w + L.cmd, w + L.off, w + L.len, P->off_cap,
                 P->len_cap, reinterpret_cast<const uint32_t*>(w + L.nsym), reinterpret_cast<uint64_t*>(w + L.tok),
                 roots ? nullptr : reinterpret_cast<uint32_t*>(w + L.tblk), w + L.done, st, 1,
                 W.sure, roots ? W.sure + W.open : W.sure, counts};
    auto parse = [&](auto recs_tag, auto threads_tag) {
      constexpr uint32_t kT = decltype(threads_tag)::value;
      hipLaunchKernelGGL((k_parse<O, decltype(recs_tag)::value, kT>), dim3(W.items), dim3(kT), 0, s, pa);
    };
    using Narrow = std::integral_constant<uint32_t, kParseThreads>;
    using Mid = std::integral_constant<uint32_t, kParseMid>;
    using Wide = std::integral_constant<uint32_t, kParseWide>;
    const std::integral_constant<int, 1> records;
    const std::integral_constant<int, 2> counted;
    if (!recs) parse(std::integral_constant<int, 0>{}, Narrow{});
    else if (roots && W.open) W.items <= kParseMidBlocks ? parse(counted, Mid{}) : parse(counted, Narrow{});
    else if (W.items <= kParseWideBlocks) parse(records, Wide{});
    else if (W.items <= kParseMidBlocks) parse(records, Mid{});
    else parse(records, Narrow{});
    if (ev) (void)hipEventRecord(ev[2], s);
    if (roots) {
      if (ntok) enqueue_roots<O>(P, W, wbl, w, s, ev);
      else if (ev) (void)hipEventRecord(ev[3], s);
      if (ev) (void)hipEventRecord(ev[4], s);
      continue;
    }
    const int last_mark = jump ? kMarkJump : kMarkList;
    if (ntok) {
      uint32_t* lists[2] = {reinterpret_cast<uint32_t*>(w + L.list0), reinterpret_cast<uint32_t*>(w + L.list1)};
      auto cset = [&](int r) { return counts + (r % 3) * kSub * kCounterStride; };
      const uint32_t pgrid = (n_words + kPackWords - 1) / kPackWords;
      CopyArgs ca{P->d_jobs, wbl, W.items, reinterpret_cast<const uint64_t*>(w + L.tok),
                  reinterpret_cast<const uint32_t*>(w + L.tblk), ntok, reinterpret_cast<uint32_t*>(w + L.cov),
                  w + L.done, nullptr, lists[0], nullptr, cset(0), cset(1), uint32_t(L.sub_cap),
                  reinterpret_cast<uint32_t*>(w + L.llist), &st->long_count, 0, st,
                  reinterpret_cast<uint32_t*>(w + L.pbits), reinterpret_cast<const uint32_t*>(w + L.plist),
                  bulk <= 1 ? last_mark : 0, 1ull << 22, copy_mode == AX_COPY_SERIAL, P->opt.fill_round,
                  P->opt.fill_tail, uint32_t(P->opt.tail_chunks), reinterpret_cast<uint32_t*>(w + L.lit),
                  reinterpret_cast<uint64_t*>(w + L.lmap), P->slot_b, recs ? w + L.cmd : nullptr,
                  P->jobs.size() == 1 ? 1u : 0u};
      // pointer jumping over window positions (the deep remainder); the
      // jump array is the stream slots, dead once the parse is through
      JumpArgs ja{P->d_jobs, wbl, W.items, ntok, P->slot_b, ca.tok, ca.tblk, ca.done,
                  reinterpret_cast<uint32_t*>(w + L.lit), reinterpret_cast<uint64_t*>(w + L.lmap),
                  reinterpret_cast<uint64_t*>(w + L.amap), reinterpret_cast<uint32_t*>(w + L.jflags),
                  reinterpret_cast<uint8_t**>(w + L.ibase), uint32_t(__builtin_ctz(P->slot_b)),
                  nullptr, nullptr, uint32_t(L.sub_cap), reinterpret_cast<uint32_t*>(w + L.wlist), st, 0};
      const uint32_t grid = uint32_t(std::min<uint64_t>((ntok + kCopyThreads - 1) / kCopyThreads, kMaxRoundGrid));
      if (P->opt.round0_tile && ca.cmd)
        hipLaunchKernelGGL((k_round0<O, true>), dim3(W.items), dim3(kCopyThreads), 0, s, ca);
      else if (P->opt.round0_tile)
        hipLaunchKernelGGL((k_round0<O, false>), dim3(W.items), dim3(kCopyThreads), 0, s, ca);
      else hipLaunchKernelGGL(k_round0_waves<O>, dim3(grid), dim3(kCopyThreads), 0, s, ca);
      hipLaunchKernelGGL(k_long<O>, dim3(std::min<uint32_t>(grid, 2048)), dim3(kCopyThreads), 0, s, ca);
      if (feedback && bulk > 1) hipLaunchKernelGGL(k_pending0, dim3(1), dim3(64), 0, s, cset(0), st);
      for (int r = 1; r < bulk; ++r) {
        ca.round = uint32_t(r);
        ca.list_in = lists[(r - 1) & 1];
        ca.list_out = lists[r & 1];
        ca.cnt_in = cset(r - 1);
        ca.cnt_out = cset(r);
        ca.cnt_clear = cset(r + 1);
        ca.mark = r + 1 == bulk ? last_mark : 0;
        // later rounds see the previous round's leftovers only
        hipLaunchKernelGGL(k_round<O>, dim3(grid), dim3(kCopyThreads), 0, s, ca);
      }
      ca.round = uint32_t(bulk);
      if (ev) (void)hipEventRecord(ev[3], s);
      if (!jump) {
        uint32_t* pcnt = reinterpret_cast<uint32_t*>(w + L.pcnt);
        hipLaunchKernelGGL(k_pcount, dim3(pgrid), dim3(kCopyThreads), 0, s, ca.pbits, n_words, pcnt);
        hipLaunchKernelGGL(k_pscatter, dim3(pgrid), dim3(kCopyThreads), 0, s, ca.pbits, n_words, pcnt,
                           reinterpret_cast<uint32_t*>(w + L.plist), st);
      }
      if (jump) {
        // the last round marked the remainder (long tokens are marked here):
        // list the map's busy words, settle the first entries, jump, write
        ja.llist = ca.list_out;  // the last round's output sublists hold the long pending tokens
        ja.lcnt = ca.cnt_out;
        hipLaunchKernelGGL(k_jmarklong<O>, dim3(grid), dim3(kCopyThreads), 0, s, ja);
        const uint32_t lgrid = uint32_t((mwords + kJListWords - 1) / kJListWords);
        hipLaunchKernelGGL(k_jlist, dim3(lgrid), dim3(kCopyThreads), 0, s, ja);
        hipLaunchKernelGGL(k_jinit, dim3(jgrid), dim3(kCopyThreads), 0, s, ja);
        // passes 0 .. used-1 leave no active entry (pass `used` found none);
        // the spare pass that reports it again runs only while learning
        uint32_t passes = P->jsettled && P->jneed[wi] ? std::min(P->jpass[wi], P->jneed[wi]) : P->jpass[wi];
        if (P->opt.jump_passes) passes = std::min<uint32_t>(passes, P->opt.jump_passes);
        for (uint32_t p = 0; p < passes; ++p) {
          ja.pass = p;
          hipLaunchKernelGGL(k_jpass, dim3(jgrid), dim3(kCopyThreads), 0, s, ja);
        }
        hipLaunchKernelGGL(k_jgather, dim3(jgrid), dim3(kCopyThreads), 0, s, ja);
        if (feedback) (void)hipMemcpyAsync(P->h_jused + 2 * wi, &st->jump_used, 4, hipMemcpyDeviceToHost, s);
      } else {
        const uint64_t waves = (ntok + 64ull * P->opt.tail_chunks - 1) / (64ull * P->opt.tail_chunks);
        const uint32_t tgrid = uint32_t(std::min<uint64_t>((waves + 3) / 4, uint64_t(P->copy_grid)));
        hipLaunchKernelGGL(k_tail<O>, dim3(tgrid), dim3(kCopyThreads), 0, s, ca);
      }
      if (feedback) (void)hipMemcpyAsync(P->h_jused + 2 * wi + 1, &st->pend0, 4, hipMemcpyDeviceToHost, s);
    }
    if (ev && !ntok) (void)hipEventRecord(ev[3], s);
    if (ev) (void)hipEventRecord(ev[4], s);
  }
}

// The launch sequence for the plan's output addressing.
static void enqueue(Plan* P, uint8_t* w, int copy_mode, hipStream_t s, bool timed, bool feedback) {
  if (P->mapped) enqueue_out<OutMapped>(P, w, copy_mode, s, timed, feedback);
  else enqueue_out<OutDirect>(P, w, copy_mode, s, timed, feedback);
}

// A decode: checks, then the launch sequence on s.  no_alloc: no graph and no
// stage timing (both may create runtime objects); everything else a decode
// uses was allocated with the plan.
static int run_plan(Plan* P, void* d_work, uint64_t work_len, int copy_mode, hipStream_t s, bool no_alloc) {
  if (!d_work) return fail(AX_E_ARG, "null workspace");
  if (work_len < P->lay.total) return fail(AX_E_CAPACITY, "workspace too small");
  if (reinterpret_cast<uintptr_t>(d_work) & 255) return fail(AX_E_ARG, "workspace must be 256-byte aligned");
  if (copy_mode != AX_COPY_PERIODIC && copy_mode != AX_COPY_SERIAL) return fail(AX_E_ARG, "bad copy mode");
  for (size_t j = 0; j < P->jobs.size(); ++j) {
    if (!P->jobs[j].out && P->jobs[j].n_bytes) return fail(AX_E_ARG, "job without an output buffer");
    if (reinterpret_cast<uintptr_t>(P->jobs[j].out) & 15) return fail(AX_E_ARG, "outputs must be 16-byte aligned");
  }
  // refresh output pointers that changed since the last upload
  bool stale = false;
  for (size_t j = 0; j < P->jobs.size(); ++j) stale |= P->dev_out[j] != P->jobs[j].out;
  if (stale) {
    if (P->staged) (void)hipEventSynchronize(P->staged);  // h_pinned may feed the previous update
    std::memcpy(P->h_pinned, P->jobs.data(), sizeof(JobDev) * P->jobs.size());
    hipError_t e = hipMemcpyAsync(P->d_jobs, P->h_pinned, sizeof(JobDev) * P->jobs.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess && P->staged) e = hipEventRecord(P->staged, s);
    if (e != hipSuccess) return hip_fail(e, "job table update");
    for (size_t j = 0; j < P->jobs.size(); ++j) P->dev_out[j] = P->jobs[j].out;
  }
  uint8_t* w = static_cast<uint8_t*>(d_work);
  const bool timed = P->timing && P->events_ok;
  // learned bulk-round and jump-pass counts: take the previous decode's
  // report once it is in (a window whose bulk count changes starts its pass
  // count over from the bound)
  if (P->jfeed_pending && hipEventQuery(P->jfed) == hipSuccess) {
    P->jfeed_pending = false;
    bool all = true;
    for (size_t i = 0; i < P->wins.size(); ++i) {
      const uint32_t used = P->h_jused[2 * i], pend0 = P->h_jused[2 * i + 1];
      if (P->bulk_auto && !P->bsettled) {
        const uint8_t b = 10ull * pend0 > 9ull * P->wins[i].tok ? 1 : 0;
        if (b != P->wbulk[i]) {
          P->wbulk[i] = b;
          P->jpass[i] = jump_pass_bound(P->wins[i].tok);
          P->jneed[i] = 0;
          all = false;
          continue;
        }
      }
      if (used) P->jpass[i] = std::min(P->jpass[i], used + 1), P->jneed[i] = used;
      else all = false;
    }
    if (P->bulk_auto) P->bsettled = true;
    P->jsettled = all;
    P->graph_stale = P->graph != nullptr;  // counts changed
  }
  if (P->graph_stale && !no_alloc) (void)hipGraphExecDestroy(P->graph), P->graph = nullptr, P->graph_stale = false;
  const bool rounds = !roots_schedule(P, copy_mode);
  const bool fb_jump = rounds && !P->jsettled && P->opt.tail_mode == 0 && !P->opt.jump_passes && copy_mode != AX_COPY_SERIAL;
  const bool fb_bulk = rounds && P->bulk_auto && !P->bsettled;
  const bool feedback = P->learn && (fb_jump || fb_bulk) && !P->jfeed_pending && !P->wins.empty() &&
                        P->jused_cap >= P->wins.size() && P->jfed;
  if (feedback) std::fill(P->h_jused, P->h_jused + 2 * P->wins.size(), 0u);
  if (P->opt.graph && !timed && !no_alloc) {
    // the launch sequence of every window and round, captured once and replayed
    if (!P->graph || P->graph_work != d_work || P->graph_mode != copy_mode) {
      if (P->graph) (void)hipGraphExecDestroy(P->graph), P->graph = nullptr;
      if (P->graph_def) (void)hipGraphDestroy(P->graph_def), P->graph_def = nullptr;
      if (!P->cap_stream) {
        hipError_t e = hipStreamCreateWithFlags(&P->cap_stream, hipStreamNonBlocking);
        if (e != hipSuccess) return hip_fail(e, "capture stream");
      }
      hipError_t e = hipStreamBeginCapture(P->cap_stream, hipStreamCaptureModeThreadLocal);
      if (e != hipSuccess) return hip_fail(e, "graph capture");
      enqueue(P, w, copy_mode, P->cap_stream, false, false);
      e = hipStreamEndCapture(P->cap_stream, &P->graph_def);
      if (e == hipSuccess) e = hipGraphInstantiate(&P->graph, P->graph_def, nullptr, nullptr, 0);
      if (e != hipSuccess) return hip_fail(e, "graph instantiate");
      P->graph_work = d_work;
      P->graph_mode = copy_mode;
    }
    hipError_t e = hipGraphLaunch(P->graph, s);
    if (e != hipSuccess) return hip_fail(e, "graph launch");
    return AX_OK;
  }
  const bool timed_now = timed && !no_alloc;
  if (timed_now) {
    int rc = ensure_events(P);
    if (rc) return rc;
  }
  enqueue(P, w, copy_mode, s, timed_now, feedback);
  if (timed_now) P->timed_windows = P->wins.size();
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  if (feedback) {
    e = hipEventRecord(P->jfed, s);
    if (e != hipSuccess) return hip_fail(e, "pass report event");
    P->jfeed_pending = true;
  }
  return AX_OK;
}

int plan_run(Plan* P, void* d_work, uint64_t work_len, int copy_mode, hipStream_t s) {
  return run_plan(P, d_work, work_len, copy_mode, s, false);
}
int plan_run_no_alloc(Plan* P, void* d_work, uint64_t work_len, int copy_mode, hipStream_t s) {
  return run_plan(P, d_work, work_len, copy_mode, s, true);
}

int workspace_status(void* d_work, hipStream_t s, int32_t* dev_err, uint64_t* bad_block) {
  DevStatus hs;
  hipError_t e = hipMemcpyAsync(&hs, d_work, sizeof(hs), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "status read");
  *dev_err = hs.err;
  *bad_block = hs.bad_block;
  return AX_OK;
}

}  // namespace ax

// ------------------------------------------------- allocation-free decode --
//
// Workspace of aceapex_decode_all_static: a library-owned device array, so
// that callers that cannot allocate device memory can still decode.  Every
// device the library runs on holds its own copy (at its own address, looked
// up once per device with that device current) until the process ends.  All
// such decodes on one device share it: calls that overlap on one device race.
// The launch sequence initialises every part of a workspace it reads, so the
// contents a previous call left do not matter.
static __device__ __align__(256) uint8_t scratch[AX_STATIC_SCRATCH_BYTES];

namespace {
constexpr uint64_t kStaticScratchBytes = AX_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_at[kMaxDevices] = {};

// Device address of the static scratch on the current device.
int static_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return ax::fail(AX_E_HIP, hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return ax::fail(AX_E_UNSUPPORTED, "device index beyond the scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_at[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return ax::fail(AX_E_HIP, hipGetErrorString(e));
    if (!p || (reinterpret_cast<uintptr_t>(p) & 255)) return ax::fail(AX_E_HIP, "static scratch address");
    g_scratch_at[dev] = p;
  }
  *out = g_scratch_at[dev];
  return AX_OK;
}
}  // namespace

extern "C" {

int aceapex_read_info(const uint8_t* h, uint64_t len, aceapex_info* info) {
  if (!h || !info || len < 64) return ax::fail(AX_E_ARG, "need at least the 64-byte header");
  if (ax::get32(h) != ax::kMagic || ax::get16(h + 4) != 1) return ax::fail(AX_E_CORRUPT, "bad magic or version");
  aceapex_info I{};
  I.flags = ax::get16(h + 6);
  I.block_size = ax::get32(h + 8);
  I.min_match = ax::get16(h + 12);
  I.depth_cap = ax::get16(h + 14);
  I.n_bytes = ax::get64(h + 16);
  I.n_blocks = ax::get64(h + 24);
  I.xxh3 = ax::get64(h + 32);
  I.payload_bytes = ax::get64(h + 40);
  I.n_matches = ax::get64(h + 48);
  const uint32_t B = I.block_size;
  if (B < 4096 || B > 65536 || (B & (B - 1)) || I.min_match < 1 || I.min_match > 255)
    return ax::fail(AX_E_CORRUPT, "bad block size or min_match");
  if (I.n_blocks != (I.n_bytes + B - 1) / B) return ax::fail(AX_E_CORRUPT, "block count mismatch");
  if (I.n_blocks > (1ull << 40)) return ax::fail(AX_E_CORRUPT, "block count too large");
  I.header_bytes = 64 + 16 * (I.n_blocks + 1);
  I.archive_bytes = I.header_bytes + I.payload_bytes;
  if (I.archive_bytes < I.header_bytes) return ax::fail(AX_E_CORRUPT, "size overflow");
  *info = I;
  return AX_OK;
}

int aceapex_decoder_create(const uint8_t* h, uint64_t h_len, const uint8_t* d_arc, uint64_t arc_len,
                           aceapex_decoder** out) {
  if (!out) return ax::fail(AX_E_ARG, "null out");
  *out = nullptr;
  aceapex_info I;
  int rc = aceapex_read_info(h, h_len, &I);
  if (rc) return rc;
  if (h_len < I.header_bytes) return ax::fail(AX_E_ARG, "host copy shorter than header + index");
  if (!d_arc || arc_len < I.archive_bytes) return ax::fail(AX_E_ARG, "device archive shorter than the header says");
  if (I.block_size > kMaxB) return ax::fail(AX_E_UNSUPPORTED, "device decoder takes blocks up to 16384 bytes");
  aceapex_decoder* d = new (std::nothrow) aceapex_decoder;
  if (!d) return ax::fail(AX_E_NOMEM, "decoder handle");
  d->info = I;
  d->d_arc = d_arc;
  d->arc_len = arc_len;
  const uint64_t nb = I.n_blocks, B = I.block_size;
  try {
    d->offs.resize(nb + 1);
    d->mpre.resize(nb + 1);
  } catch (const std::bad_alloc&) {
    delete d;
    return ax::fail(AX_E_NOMEM, "index copy");
  }
  const uint8_t* ix = h + 64;
  for (uint64_t b = 0; b <= nb; ++b) d->offs[b] = ax::get64(ix + 8 * b), d->mpre[b] = ax::get64(ix + 8 * (nb + 1) + 8 * b);
  bool ok = d->offs[0] == 0 && d->offs[nb] == I.payload_bytes && d->mpre[0] == 0 && d->mpre[nb] == I.n_matches;
  const uint64_t max_tok = B / I.min_match;
  for (uint64_t b = 0; b < nb && ok; ++b) {
    ok &= d->offs[b + 1] >= d->offs[b] + 16 && ((d->offs[b + 1] - d->offs[b]) & 15) == 0;
    ok &= d->mpre[b + 1] >= d->mpre[b] && d->mpre[b + 1] - d->mpre[b] <= max_tok;
  }
  if (!ok) {
    delete d;
    return ax::fail(AX_E_CORRUPT, "bad index");
  }
  rc = ax::plan_create({ax::JobSpec{d, nullptr, {}}}, &d->plan);
  if (rc) {
    delete d;
    return rc;
  }
  *out = d;
  return AX_OK;
}

void aceapex_decoder_destroy(aceapex_decoder* d) {
  if (!d) return;
  aceapex_range_plan_destroy(d->range);
  ax::plan_destroy(d->plan);
  delete d;
}

int aceapex_decoder_info(const aceapex_decoder* d, aceapex_info* info) {
  if (!d || !info) return ax::fail(AX_E_ARG, "null argument");
  *info = d->info;
  return AX_OK;
}

int aceapex_decoder_workspace(const aceapex_decoder* d, uint64_t* bytes) {
  if (!d || !bytes) return ax::fail(AX_E_ARG, "null argument");
  *bytes = ax::plan_workspace(d->plan);
  return AX_OK;
}

int aceapex_decoder_set_timing(aceapex_decoder* d, int enable) {
  if (!d) return ax::fail(AX_E_ARG, "null decoder");
  return ax::plan_set_timing(d->plan, enable);
}

int aceapex_decoder_set_option(aceapex_decoder* d, int option, int64_t value) {
  if (!d) return ax::fail(AX_E_ARG, "null decoder");
  return ax::plan_set_option(d->plan, option, value);
}

int aceapex_decoder_stage_ms(aceapex_decoder* d, float* ans, float* parse, float* copy, float* remainder) {
  if (!d || !ans || !parse || !copy) return ax::fail(AX_E_ARG, "null argument");
  return ax::plan_stage_ms(d->plan, ans, parse, copy, remainder);
}

int aceapex_decode_all(aceapex_decoder* d, uint8_t* d_out, uint64_t out_cap, void* d_work, uint64_t work_len,
                       int copy_mode, void* stream) {
  if (!d || (!d_out && d->info.n_bytes) || !d_work) return ax::fail(AX_E_ARG, "null argument");
  if (out_cap < d->info.n_bytes) return ax::fail(AX_E_CAPACITY, "output smaller than the decoded size");
  ax::plan_set_out(d->plan, 0, d_out);
  return ax::plan_run(d->plan, d_work, work_len, copy_mode, reinterpret_cast<hipStream_t>(stream));
}

int aceapex_decode_all_static(aceapex_decoder* d, uint8_t* d_out, uint64_t out_cap, int copy_mode, void* stream) {
  if (!d || (!d_out && d->info.n_bytes)) return ax::fail(AX_E_ARG, "null argument");
  if (out_cap < d->info.n_bytes) return ax::fail(AX_E_CAPACITY, "output smaller than the decoded size");
  if (ax::plan_workspace(d->plan) > kStaticScratchBytes)
    return ax::fail(AX_E_CAPACITY, "the archive needs more workspace than the static scratch holds");
  void* w = nullptr;
  int rc = static_scratch(&w);
  if (rc) return rc;
  ax::plan_set_out(d->plan, 0, d_out);
  return ax::plan_run_no_alloc(d->plan, w, kStaticScratchBytes, copy_mode, reinterpret_cast<hipStream_t>(stream));
}

int aceapex_decoder_streams(aceapex_decoder* d, uint64_t first, uint64_t count, void* d_work, uint64_t work_len,
                            void* stream, uint8_t* h_out, uint64_t cap, uint32_t* n_syms) {
  if (!d || (count && (!d_work || !n_syms || (!h_out && cap)))) return ax::fail(AX_E_ARG, "null argument");
  return ax::block_streams(d, first, count, d_work, work_len, reinterpret_cast<hipStream_t>(stream), h_out, cap,
                           n_syms);
}

int aceapex_decoder_status(aceapex_decoder* d, void* d_work, void* stream, int32_t* dev_err, uint64_t* bad_block) {
  if (!d || !dev_err || !bad_block) return ax::fail(AX_E_ARG, "null argument");
  if (!d_work) {  // the static scratch of aceapex_decode_all_static on the current device
    int rc = static_scratch(&d_work);
    if (rc) return rc;
  }
  return ax::workspace_status(d_work, reinterpret_cast<hipStream_t>(stream), dev_err, bad_block);
}

int aceapex_workspace_status(void* d_work, void* stream, int32_t* dev_err, uint64_t* bad_block) {
  if (!d_work || !dev_err || !bad_block) return ax::fail(AX_E_ARG, "null argument");
  return ax::workspace_status(d_work, reinterpret_cast<hipStream_t>(stream), dev_err, bad_block);
}

// ------------------------------------------------------------------ batch --

struct aceapex_batch {
  ax::Plan* plan = nullptr;
};

int aceapex_batch_create(const aceapex_job* jobs, uint32_t n, aceapex_batch** out) {
  if (!out || (!jobs && n)) return ax::fail(AX_E_ARG, "null argument");
  *out = nullptr;
  std::vector<ax::JobSpec> specs;
  try {
    specs.reserve(n);
    for (uint32_t i = 0; i < n; ++i) {
      if (!jobs[i].dec) return ax::fail(AX_E_ARG, "job without a decoder");
      if (jobs[i].out_cap < jobs[i].dec->info.n_bytes) return ax::fail(AX_E_CAPACITY, "job output too small");
      specs.push_back(ax::JobSpec{jobs[i].dec, jobs[i].d_out, {}});
    }
  } catch (const std::bad_alloc&) {
    return ax::fail(AX_E_NOMEM, "batch jobs");
  }
  aceapex_batch* bt = new (std::nothrow) aceapex_batch;
  if (!bt) return ax::fail(AX_E_NOMEM, "batch handle");
  int rc = ax::plan_create(specs, &bt->plan);
  if (rc) {
    delete bt;
    return rc;
  }
  *out = bt;
  return AX_OK;
}

void aceapex_batch_destroy(aceapex_batch* bt) {
  if (!bt) return;
  ax::plan_destroy(bt->plan);
  delete bt;
}

int aceapex_batch_workspace(const aceapex_batch* bt, uint64_t* bytes) {
  if (!bt || !bytes) return ax::fail(AX_E_ARG, "null argument");
  *bytes = ax::plan_workspace(bt->plan);
  return AX_OK;
}

int aceapex_batch_set_option(aceapex_batch* bt, int option, int64_t value) {
  if (!bt) return ax::fail(AX_E_ARG, "null batch");
  return ax::plan_set_option(bt->plan, option, value);
}

int aceapex_batch_set_timing(aceapex_batch* bt, int enable) {
  if (!bt) return ax::fail(AX_E_ARG, "null batch");
  return ax::plan_set_timing(bt->plan, enable);
}

int aceapex_batch_stage_ms(aceapex_batch* bt, float* ans, float* parse, float* copy, float* remainder) {
  if (!bt || !ans || !parse || !copy) return ax::fail(AX_E_ARG, "null argument");
  return ax::plan_stage_ms(bt->plan, ans, parse, copy, remainder);
}

int aceapex_decode_batch(aceapex_batch* bt, void* d_work, uint64_t work_len, int copy_mode, void* stream) {
  if (!bt) return ax::fail(AX_E_ARG, "null batch");
  return ax::plan_run(bt->plan, d_work, work_len, copy_mode, reinterpret_cast<hipStream_t>(stream));
}

}  // extern "C"
