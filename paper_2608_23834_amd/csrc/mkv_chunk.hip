// Causal chunked-prefill attention over mixed FP8/TQ3 pages on MFMA (the
// query chunk makes it a dense contraction).  The paper runs prefill on a
// generic dense path (Sec. 4.1); this variant keeps the pages in their two
// physical formats and applies the same score algebra as decode (Sec. 3.3):
// rotated queries against TQ3 key codes times the FP16 key-norm correction,
// plain queries against FP8 keys, one online softmax per query row.
//
// Launch: a list kernel (per request the TQ3 and the FP8 pages in logical order,
// Sec. 4.1), a plan kernel (the row blocks, how far each has to read, and how the
// blocks are cut along the pages when there are too few of them for the chip),
// the attention kernel, and a merge of the cut blocks' parts where any can be.
// Grid (work item, KV head); 512 threads = 8 waves, one workgroup per CU, two
// waves per SIMD.  A query row is a (query token, head of the GQA group) pair; a
// workgroup owns 128 rows and a range of their passes, a pass being a pair of
// pages of one format (first the TQ3 pairs, then the FP8 pairs):
//  * four score waves of 32 rows each hold their rows' rotated queries as
//    three E4M3 terms in registers and unpack TQ3 pairs into MFMA operand
//    layouts in LDS (key codes -> E4M3 codebook bytes, value codes
//    as bytes, the V scale split for exact fp16 products).  Pass p issues S^T = K
//    Q^T of pair p on v_mfma_f32_32x32x64_f8f6f4 (M = the pair's 32 tokens, N =
//    the 32 rows, K = 64 channels; three MFMAs per k-step, one per query term)
//    and, between those MFMAs, finishes pair p - 1: the causal mask, the online
//    softmax in base 2 (lazy rescale, threshold 2^8) and the weights as fp16
//    hi + lo pairs, handed over in LDS;
//  * four PV waves, wave v owning the 32-channel blocks 2v, 2v + 1 of all
//    128 rows, hold O^T accumulators (32 channels x 32 rows per block and
//    score wave) and compute O^T += V^T P^T on v_mfma_f32_32x32x16_f16 (M =
//    32 channels, N = 32 rows, K = the 16 tokens of one page; a lane's score
//    outputs are exactly the 8 tokens per page its weight operand holds):
//    values as exact fp16 operands (scale_hi * code, scale_lo * code), the
//    zero term as one rank-2 product of the pages' zeros and weight sums,
//    applying the rescale the score waves passed along first.
// The pages and the page lists are copied (direct HBM -> LDS copies into a ring) by
// the score waves at d = 256, by the PV waves at d = 128 (see COPY_PV).
// Pass p (one barrier): the score waves issue pair p's product and finish
// pair p - 1 while the PV waves take pair p - 2.  FP8 pairs: the score waves
// score them on the f16 MFMA against the plain query (the fp8 MFMA keeps too
// few bits where FP8 keys carry large norms) and fold the pages' V scales, less
// their powers of two, into the weights; the PV waves read the pages' values from
// the ring and scale them by those.  The
// workgroups of one (request, KV head) read the same pages at about the same
// time, so the page bytes come from L2 after the first reader.
#include <hip/hip_runtime.h>

#include <atomic>
#include <type_traits>

#include "mkv_attn.h"
#include "mkv_internal.h"
#include "../../include/minima_kv.h"

namespace mkv {

constexpr int NSW = 4;       // score waves per chunk workgroup (one PV wave each)
constexpr int CW = 2 * NSW;  // waves per chunk workgroup
constexpr int CSLOTS = 8;    // slots of the page ring: a TQ3 pair or one FP8 page each
// FP8 pairs take two slots for three passes; while they run, the buffers of
// unpacked TQ3 operands behind the ring are four slots more
constexpr int CSLOTS8 = 12;
constexpr int CMASK_LP = 0x3FFFFFFF / PAGE;

struct ChunkArgs {
  PoolView P;
  int layer, n_req, max_pages, n_q_total, stride;
  const uint16_t* q;
  const int32_t* cu_q;
  const int32_t* seq_lens;
  float* out;
  const int2* list8;   // [n_req][stride] (logical page, physical id), in pairs
  const int2* list3;
  const int32_t* hdr;  // [0] work items, [1] blocks cut into parts
  const int4* items;   // two per work item, see chunk_plan_kernel
  float* parts;        // the parts of cut blocks, see chunk_part_floats
  float sm_log2;       // log2(e) / sqrt(d)
};

static size_t al256(size_t b) { return (b + 255) / 256 * 256; }

// CUs a KV head's row blocks can spread over, and the most work items that cut
// blocks are planned for (two rounds)
static int cu_share(int n_kv_heads) { return n_kv_heads >= 256 ? 1 : 256 / n_kv_heads; }
constexpr int MAX_ITEMS = 512;  // 2 * cu_share at most
constexpr int MAX_PARTS = 32;   // parts of one block at most
// cost units of the plan (see chunk_plan_kernel): a pass of each format, a part beside
// its passes, the least size of a part
constexpr int COST3 = 4, COST8 = 4;
constexpr int CUT_COST = 12 * COST3, MIN_PART = 4 * COST3;
// No block is cut where the dearest one costs no more than this: a round of the smallest
// parts is estimated at MIN_PART + CUT_COST, and whole blocks take one round of the
// dearest where cut ones could take one, two where they take two.
constexpr int CUT_FROM = MIN_PART + CUT_COST;
static int64_t chunk_blocks(int n_q_total, int group) { return ((int64_t)n_q_total * group + NSW * 32 - 1) / (NSW * 32); }
// Blocks are cut only where at least that many of them (the query ranges not
// overlapping) leave room in two rounds.
static bool chunk_may_cut(int n_q_total, int group, int n_kv_heads) {
  return chunk_blocks(n_q_total, group) <= 2 * cu_share(n_kv_heads);
}
// One part of one KV head: O^T accumulators of the PV waves as they stand in
// registers ([PV wave][block][score wave][4][lane] float4s), then (m, l) per row.
__host__ __device__ constexpr int64_t chunk_part_floats(int d) { return 128LL * d + 256; }

// workspace: the two page lists (even rows with room for a masked last page;
// the kernel copies them in 1 KiB blocks, so 1 KiB of slack follows), the pages'
// running counts, the row blocks, the cut blocks, the work items and the parts of
// cut blocks.  Only what lies before the items and MAX_ITEMS of them is needed:
// where the room ends the parts end (fewer blocks are cut, or none) and before them
// the items (the blocks go in several launches).  So any workspace that a call of
// these requests and pages was sized for serves every other one.
struct ChunkWs {
  size_t list8, list3, cum, rbo, hdr, splits, items, parts, total;
  int stride, n_items, n_parts;
};
static size_t chunk_part_bytes(int n_kv_heads, int d) { return n_kv_heads * (size_t)chunk_part_floats(d) * sizeof(float); }
static ChunkWs chunk_ws(int n_req, int max_pages, int n_q_total, int n_kv_heads, int group, int d, size_t room) {
  ChunkWs w;
  w.stride = (max_pages + 2) & ~1;
  const size_t lb = al256((size_t)n_req * w.stride * sizeof(int2) + 1024);
  w.list8 = 0;
  w.list3 = lb;
  w.cum = 2 * lb;
  w.rbo = 3 * lb;
  w.hdr = w.rbo + al256((size_t)(n_req + 1) * sizeof(int32_t));
  w.splits = w.hdr + 256;
  w.items = w.splits + MAX_ITEMS * sizeof(int4);
  const int64_t blocks = chunk_blocks(n_q_total, group) + n_req;
  int64_t n_items = blocks < MAX_ITEMS ? MAX_ITEMS : blocks;
  const int64_t items_fit = room < w.items ? 0 : (int64_t)((room - w.items) / (2 * sizeof(int4)));
  if (n_items > items_fit) n_items = items_fit;
  w.n_items = (int)n_items;
  w.parts = w.items + al256((size_t)n_items * 2 * sizeof(int4));
  // a part holds at least one pass: short tables cannot be cut into many.  Blocks
  // are cut in small calls only, but what a small call can use, a large one reports
  const int64_t passes = max_pages / 2 + 1;
  int64_t n_parts = passes * (COST3 > COST8 ? COST3 : COST8) > CUT_FROM ? 2LL * cu_share(n_kv_heads) : 0;
  const int64_t most = blocks * (passes < MAX_PARTS ? passes : MAX_PARTS);
  if (n_parts > most) n_parts = most;
  const int64_t parts_fit = room < w.parts ? 0 : (int64_t)((room - w.parts) / chunk_part_bytes(n_kv_heads, d));
  if (n_parts > parts_fit) n_parts = parts_fit;
  w.n_parts = (int)n_parts;
  w.total = w.parts + (size_t)n_parts * chunk_part_bytes(n_kv_heads, d);
  return w;
}
size_t chunk_ws_bytes(int n_req, int max_pages, int n_q_total, int n_kv_heads, int group, int d) {
  return chunk_ws(n_req, max_pages, n_q_total, n_kv_heads, group, d, SIZE_MAX / 2).total;
}
size_t chunk_ws_least(int n_req, int max_pages) {
  return chunk_ws(n_req, max_pages, 1, 1, 1, 128, 0).items + MAX_ITEMS * 2 * sizeof(int4);
}

// Page lists of a chunk call, one workgroup per request: the TQ3 and the FP8
// pages in logical order, so entries 2 j and 2 j + 1 are pair j of their format
// (an odd list ends with a masked page), and per logical page the counts of both
// formats up to and including it.  Pages whose id lies outside their pool are left out
// (a pool without TQ3 pages has no memory that could stand in), and set the range error
// bit.  Four consecutive pages per thread, one scan of both counts per 4,096 pages: the
// cost is round trips.
constexpr int LIST_NT = 1024, LIST_KB = 4;
__global__ __launch_bounds__(LIST_NT) void chunk_lists_kernel(const int32_t* bt, const uint8_t* tags,
                                                              int max_pages, int stride,
                                                              const int32_t* seq_lens, int n_fp8,
                                                              int n_tq3, int2* list8, int2* list3,
                                                              int2* cum, int32_t* err) {
  __shared__ int scratch[32];
  const int r = blockIdx.x, tid = threadIdx.x;
  const int S = seq_lens[r];
  const int np = S >= 1 ? (S - 1) / PAGE + 1 : 0;
  if (S < 1 || np > max_pages) {  // its blocks write zeros
    if (tid == 0) atomicOr(err, (int)MKV_DEVERR_RANGE);
    return;
  }
  int2* l8 = list8 + (int64_t)r * stride;
  int2* l3 = list3 + (int64_t)r * stride;
  int2* cm = cum + (int64_t)r * stride;
  int b8 = 0, b3 = 0, bad = 0;
  for (int c0 = 0; c0 < np; c0 += LIST_NT * LIST_KB) {
    int tg[LIST_KB], id[LIST_KB];
#pragma unroll
    for (int j = 0; j < LIST_KB; ++j) {
      const int p = c0 + LIST_KB * tid + j;
      const int64_t i = (int64_t)r * max_pages + min(p, np - 1);
      tg[j] = tags[i];
      id[j] = bt[i];
      if (p >= np) tg[j] = -1;
    }
    bool is3[LIST_KB], is8[LIST_KB];
    int v = 0;
#pragma unroll
    for (int j = 0; j < LIST_KB; ++j) {
      is3[j] = tg[j] == TAG_S;
      is8[j] = tg[j] == TAG_R || tg[j] == TAG_A;
      if (tg[j] >= 0 && !is3[j] && !is8[j]) bad |= MKV_DEVERR_BAD_TAG;
      if ((is3[j] || is8[j]) && (id[j] < 0 || id[j] >= (is3[j] ? n_tq3 : n_fp8))) {
        bad |= MKV_DEVERR_RANGE;
        is3[j] = is8[j] = false;
      }
      v += is3[j] ? 1 << 16 : is8[j] ? 1 : 0;
    }
    int tot;
    const int pre = block_excl_scan(v, scratch, &tot);
    int r8 = b8 + (pre & 0xFFFF), r3 = b3 + (pre >> 16);
#pragma unroll
    for (int j = 0; j < LIST_KB; ++j) {
      const int p = c0 + LIST_KB * tid + j;
      if (tg[j] < 0) continue;
      if (is3[j]) l3[r3++] = make_int2(p, id[j]);
      if (is8[j]) l8[r8++] = make_int2(p, id[j]);
      cm[p] = make_int2(r8, r3);
      if (p == np - 1) {  // the masked partners of odd lists
        l8[r8] = make_int2(CMASK_LP, 0);
        l3[r3] = make_int2(CMASK_LP, 0);
      }
    }
    b8 += tot & 0xFFFF;
    b3 += tot >> 16;
  }
  if (bad) atomicOr(err, bad);
}

// Plan of a chunk call (one workgroup).
// Row blocks: request r gets ceil(n_r G / 128) blocks of 128 rows (at least one,
// and one for a request whose query range is invalid, so that its error is
// reported).  Query ranges that do not overlap need at most `grid` blocks; ranges
// that overlap and need more set the range error bit and the call writes nothing.
// A block reads the pages up to its last row's position, so the pages of the
// chunk that only later rows see are left out.
// Cutting: a block's passes run one after the other on one CU, so a call with
// fewer blocks than CUs, or of uneven lengths, leaves the chip idle (six chunks
// of 1-300 queries after 0.5-8 K tokens: 691 us, the longest request's blocks
// alone at the end; cut, and with FP8 pages in pairs, 415).  With U the most cost units a part may hold, the blocks make
// sum ceil(cost / U) parts; the plan tries eight sizes U for one and for two rounds
// of the chip, estimates a round as U + CUT_COST (a part's own start, its
// partial results' way through memory and the merge, measured) and takes the
// best, or leaves the blocks whole where that is estimated as good.  Cost
// units: 4 per pass, of either format (2.02 us per TQ3 pair and 1.88 per FP8 pair at
// d = 256, 1.31 and 1.54 at d = 128, one workgroup on every CU; with 3 per FP8 pair a
// 6,001-token prefill's twelve calls took 2,738 us, with 4 2,688).
// items: two int4 per work item, {request, block of the request, first TQ3 pair,
// TQ3 pairs}, {first FP8 pair, FP8 pairs, part slot or -1, -}; splits: {request,
// block of the request, first part slot, parts}.
// The table holds n_items items from row block b0 on; a call whose blocks do not fit
// comes in several launches, its blocks whole (cut blocks fit any table).
__global__ __launch_bounds__(1024) void chunk_plan_kernel(int n_req, const int32_t* cu_q, int n_q_total,
                                                          const int32_t* seq_lens, int max_pages,
                                                          int group, int grid, int b0, int n_items, int share,
                                                          int may_cut, int max_slots, int stride, const int2* cum,
                                                          int32_t* rbo, int32_t* hdr, int4* items,
                                                          int4* splits, int32_t* err) {
  __shared__ int scratch[32];
  __shared__ int s_rbo[1025];
  __shared__ int s_r[MAX_ITEMS], s_x[MAX_ITEMS], s_t3[MAX_ITEMS], s_f8[MAX_ITEMS];
  __shared__ int s_max, s_est[16], s_u[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int per = (n_req + 1023) / 1024;
  const int ra = min(n_req, tid * per), rb = min(n_req, ra + per);
  auto blocks = [&](int r) {
    const int q0 = cu_q[r], q1 = cu_q[r + 1];
    const bool ok = q0 >= 0 && q1 >= q0 && q1 <= n_q_total;
    return ok ? max(1, (int)(((int64_t)(q1 - q0) * group + NSW * 32 - 1) / (NSW * 32))) : 1;
  };
  int64_t sum64 = 0;
  for (int r = ra; r < rb; ++r) sum64 += blocks(r);
  // (a thread's sum stops at one more than `grid`: 1,024 of them fit an int for grids below
  // 2^17, and for larger ones where a first scan, in units of 1,024 blocks, finds no more
  // than the grid)
  const int sum = (int)min(sum64, (int64_t)grid + 1);
  int nblk;
  if (grid >= 1 << 17) {
    block_excl_scan(sum >> 10, scratch, &nblk);
    if ((int64_t)nblk << 10 > grid) {  // workgroup-uniform
      if (tid == 0) {
        atomicOr(err, (int)MKV_DEVERR_RANGE);
        hdr[0] = hdr[1] = 0;
      }
      return;
    }
  }
  int base = block_excl_scan(sum, scratch, &nblk);
  const bool in_lds = n_req <= 1024;
  for (int r = ra; r < rb; ++r) {
    if (in_lds) s_rbo[r] = base;
    else rbo[r] = base;
    base += blocks(r);
  }
  if (tid == 0) s_max = 0;
  __syncthreads();
  if (nblk > grid) {  // workgroup-uniform
    if (tid == 0) {
      atomicOr(err, (int)MKV_DEVERR_RANGE);
      hdr[0] = hdr[1] = 0;
    }
    return;
  }
  // block b -> request, block of the request, TQ3 and FP8 pairs it reads
  auto locate = [&](int b, int& r, int& x, int& t3, int& f8) {
    int lo = 0, hi = n_req - 1;  // the last request whose first block is <= b
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if ((in_lds ? s_rbo[mid] : rbo[mid]) <= b) lo = mid;
      else hi = mid - 1;
    }
    r = lo;
    x = b - (in_lds ? s_rbo[lo] : rbo[lo]);
    t3 = f8 = 0;
    const int q0 = cu_q[r], q1 = cu_q[r + 1], nq = q1 - q0, S = seq_lens[r];
    if (q0 < 0 || nq < 1 || q1 > n_q_total || S < nq || S > (int64_t)max_pages * PAGE) return;
    const int last = min(nq * group, (x + 1) * (NSW * 32)) - 1;  // the block's last row
    const int2 c = cum[(int64_t)r * stride + (S - nq + last / group) / PAGE];
    t3 = (c.y + 1) / 2;
    f8 = (c.x + 1) / 2;
  };
  const bool cut = may_cut && nblk <= 2 * share;
  if (!cut || b0 > 0) {
    const int n = max(0, min(nblk - b0, n_items));  // (none after a call's cut blocks)
    for (int b = tid; b < n; b += 1024) {
      int r, x, t3, f8;
      locate(b0 + b, r, x, t3, f8);
      items[2 * b] = make_int4(r, x, 0, t3);
      items[2 * b + 1] = make_int4(0, f8, -1, 0);
    }
    if (tid == 0) {
      hdr[0] = n;
      hdr[1] = 0;
    }
    return;
  }
  int cost = 0;
  if (tid < nblk) {  // nblk <= 2 * share <= MAX_ITEMS
    locate(tid, s_r[tid], s_x[tid], s_t3[tid], s_f8[tid]);
    cost = COST3 * s_t3[tid] + COST8 * s_f8[tid];
    atomicMax(&s_max, cost);
  }
  int total;
  block_excl_scan(cost, scratch, &total);  // its barriers also publish the blocks
  const int cmax = s_max;
  if (cmax <= CUT_FROM) {  // workgroup-uniform
    if (tid < nblk) {
      items[2 * tid] = make_int4(s_r[tid], s_x[tid], 0, s_t3[tid]);
      items[2 * tid + 1] = make_int4(0, s_f8[tid], -1, 0);
    }
    if (tid == 0) {
      hdr[0] = nblk;
      hdr[1] = 0;
    }
    return;
  }
  // wave w tries size k = w % 8 for 1 + w / 8 rounds
  {
    const int R = 1 + (wv >> 3), room = min(R * share, max_slots);
    // (a part of at least half of MIN_PART: two passes or more)
    const int U = max(max(MIN_PART, (cmax + MAX_PARTS - 1) / MAX_PARTS), (int)((int64_t)total * (16 + 3 * (wv & 7)) / (16LL * R * share)) + 1);
    int n = 0;
    for (int b = lane; b < nblk; b += 64) {
      const int c = COST3 * s_t3[b] + COST8 * s_f8[b];
      n += max(1, (c + U - 1) / U);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    if (lane == 0) {
      s_est[wv] = n <= room ? R * (min(U, cmax) + CUT_COST) : 0x7FFFFFFF;
      s_u[wv] = U;
    }
  }
  __syncthreads();
  int U = max(1, cmax), best = (nblk + share - 1) / share * cmax;  // left whole
  for (int w = 0; w < 16; ++w)
    if (s_est[w] < best) {
      best = s_est[w];
      U = s_u[w];
    }
  // item and part slots
  const int ns = tid < nblk ? max(1, (cost + U - 1) / U) : 0;
  int n_used, n_slots, n_split;
  const int it0 = block_excl_scan(ns, scratch, &n_used);
  const int sl0 = block_excl_scan(ns > 1 ? ns : 0, scratch, &n_slots);
  const int sp0 = block_excl_scan(ns > 1 ? 1 : 0, scratch, &n_split);
  if (tid < nblk) {
    const int r = s_r[tid], x = s_x[tid], t3 = s_t3[tid], f8 = s_f8[tid];
    // cost units -> passes
    auto pass_at = [&](int c) { return c <= COST3 * t3 ? c / COST3 : t3 + (c - COST3 * t3) / COST8; };
    int j0 = 0;
    for (int k = 0; k < ns; ++k) {
      const int j1 = k + 1 == ns ? t3 + f8 : pass_at((int)((int64_t)cost * (k + 1) / ns));
      const int a3 = min(j0, t3), b3 = min(j1, t3), a8 = max(j0 - t3, 0), b8 = max(j1 - t3, 0);
      items[2 * (it0 + k)] = make_int4(r, x, a3, b3 - a3);
      items[2 * (it0 + k) + 1] = make_int4(a8, b8 - a8, ns > 1 ? sl0 + k : -1, 0);
      j0 = j1;
    }
    if (ns > 1) splits[sp0] = make_int4(r, x, sl0, ns);
  }
  if (tid == 0) {
    hdr[0] = n_used;
    hdr[1] = n_split;
  }
}

// fp16 value with its low 3 significand bits cleared (8 significant bits left)
__device__ __forceinline__ half2v hi8x2(half2v x) {
  const uint32_t b = __builtin_bit_cast(uint32_t, x);
  return __builtin_bit_cast(half2v, b & 0xFFF8FFF8u);
}
__device__ __forceinline__ half2v bcast(_Float16 x) { return half2v{x, x}; }
// (a, b) as fp16 pairs hi = (a, b) rounded to nearest, lo = the rounded
// remainders: together 22 significant bits.  (The round-toward-zero packed
// conversion flushes fp16 subnormals, so the low part of every weight below
// 2^-4 vanished and chunk outputs moved by up to 1.3e-3.)  The remainders
// a - hi are single mixed-precision FMAs (hi read as fp16) with neg1 = -1
// held in a register.
__device__ __forceinline__ void split2(float a, float b, float neg1, uint32_t& hi, uint32_t& lo) {
  const half2v h = {(_Float16)a, (_Float16)b};
  const half2v l = {(_Float16)__builtin_fmaf((float)h[0], neg1, a), (_Float16)__builtin_fmaf((float)h[1], neg1, b)};
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, l);
}
__device__ __forceinline__ half8 h8u(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  typedef uint32_t u4v __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(half8, u4v{a, b, c, d});
}
// Power of two of an FP8 page's V scale: the PV waves give it to the values'
// conversion (exact: E4M3 values times 2^-15 .. 2^7 are fp16 numbers) and the score
// waves fold what is left of the scale, 1 to 2, into the weights.  With the whole scale
// folded in, the weights' low halves fell among the fp16 subnormals, whose last bit is
// 2^-24 whatever the weight: 150 rows over 850 FP8 tokens (d = 128) were 6.5e-6 (2-norm)
// off their 64-bit value, and 1.2e-3 with values 2^-8 of that size; now 4.4e-6 for both.
__device__ __forceinline__ float vscale_pow2(float s) {
  return fminf(fmaxf(__uint_as_float(__float_as_uint(s) & 0x7F800000u), 0x1p-15f), 0x1p7f);
}
__device__ __forceinline__ float vscale_rest(float s) {  // s over its power of two, exactly
  return s * __int_as_float(0x7F000000 - __float_as_int(vscale_pow2(s)));
}
constexpr float CM_INIT = -1.0e30f;  // running max before the first score (finite: no inf - inf)

// LDS of a chunk workgroup (bytes): the ring of raw stages, two buffers of
// unpacked key operands, two of unpacked value operands, two of the weights
// the score waves hand to the PV waves, the rows' softmax denominators for
// the final normalization, and four blocks of the page lists.
template <int D>
struct ChunkLds {
  static constexpr int NK8 = D / 64, NMB = D / 32;
  static constexpr int STAGE = 2 * (int)tq3_region_bytes(D);
  static constexpr int KB = NK8 * 64 * 32;            // key bytes [k-step][lane][32]
  static constexpr int VX = 2 * NMB * 64 * 8;         // value codes [page][block][lane][8]
  static constexpr int SX = 2 * NMB * 32 * 4;         // V scale (hi, lo) fp16 [page][block][row]
  static constexpr int VB = VX + SX + 2 * NMB * 32 * 2;  // + V zero fp16 [page][block][row]
  // weights of one stage from one score wave: 5 half8 operands per lane
  // ([field][lane][16]: page a hi, lo, page b hi, lo, zero term) and the
  // rescale factor per lane
  static constexpr int WF_ALPHA = 5 * 1024, WPW = WF_ALPHA + 256;
  static constexpr int KB0 = CSLOTS * STAGE;
  static constexpr int VB0 = KB0 + 2 * KB;
  static constexpr int WB0 = VB0 + 2 * VB;
  static constexpr int LB0 = WB0 + 2 * NSW * WPW;     // row denominators [score wave][32]
  static constexpr int LS0 = LB0 + NSW * 32 * 4;      // page-list blocks [LBUF][64 pairs][16]
  static constexpr int LBUF = 4;
  static constexpr int TOTAL = LS0 + LBUF * 1024;
  static_assert(CSLOTS8 * STAGE <= WB0, "the FP8 pairs' slots end before the weights");
  static_assert(KB % 16 == 0 && VB % 16 == 0 && STAGE % 16 == 0 && WPW % 16 == 0,
                "16-byte aligned buffers");
  static_assert(TOTAL <= 160 * 1024, "one workgroup's LDS");
};

// One work item: passes of the 128-row block xb of request r and KV head h (the
// body of a chunk workgroup; every wave of the workgroup runs it).
template <int D>
__device__ __forceinline__ void chunk_block(const ChunkArgs& a, int4 it0, int4 it1, int h, uint8_t* smem) {
  constexpr int NDW = 3 * D / 128, CL = D / 16, QQ = D / 4;
  constexpr int NKS = D / 16;   // k-steps of the FP8-page score product (16 channels each)
  constexpr int NK8 = D / 64;   // k-steps of the TQ3 score product (64 channels each)
  constexpr int NMB = D / 32;   // 32-channel blocks of the output
  constexpr int R3 = (int)tq3_region_bytes(D);
  constexpr int R8 = (int)fp8_region_bytes(D);
  constexpr int STAGE = 2 * R3;       // a TQ3 page pair, or one FP8 page + its two scales
  constexpr int MAIN_KB = 16 * D / 1024;  // whole KiB of a TQ3 page (its last 32 bytes aside)
  constexpr int OPS_W = 2 * MAIN_KB / NSW;  // 1-KiB copies per score wave per stage
  constexpr int NI = D / 64;                // 1-KiB copies per half of an FP8 page
  using LY = ChunkLds<D>;
  static_assert(2 * MAIN_KB % NSW == 0 && 2 * NI == NSW * OPS_W, "copies split evenly");
  static_assert(R3 == 1024 * MAIN_KB + 32, "TQ3 page = whole KiB + a 32-byte tail");
  static_assert(R8 + 8 <= STAGE, "an FP8 page and its scales fit one stage");
  static_assert(CL == 2 * NMB, "a chunk row of V covers two channels per block");
  static_assert(CW == 2 * NSW, "one PV wave per score wave");
  const PoolView& P = a.P;
  const int r = it0.x, xb = it0.y;
  const int st3 = it0.w, n_f8 = it1.y;  // TQ3 and FP8 pairs of this item
  const int n_st = st3 + n_f8;          // its passes
  const int slot_out = it1.z;           // part slot of a cut block, else -1
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool score_wave = wid < NSW;
  const int sw = wid % NSW;  // score wave: its rows (PV waves: unused)
  // MFMA lane roles: li = lane % 32 (row of A, column of B and of the
  // output), lg = lane / 32 (k-slot group)
  const int li = lane & 31, lg = lane >> 5;
  const int G = P.group, H = P.n_kv_heads, Hq = H * G;
  const int mp = a.max_pages;

  // ---- request and rows of this wave pair
  const int q0 = a.cu_q[r], q1 = a.cu_q[r + 1];
  const int nq = q1 - q0;
  const int S = a.seq_lens[r];
  const bool range_ok = q0 >= 0 && nq >= 0 && q1 <= a.n_q_total;
  const int rows_r = range_ok ? nq * G : 0;
  const int rb = xb * (NSW * 32) + sw * 32;
  if (!range_ok || nq < 1 || S < nq || S > mp * PAGE) {  // workgroup-uniform
    if (xb == 0 && tid == 0) atomicOr(&P.ctrl[CTRL_ERR], (int)MKV_DEVERR_RANGE);
    // rows that can be located get zeros
    const int rho = rb + li;
    if (score_wave && rho < rows_r) {
      float* o = a.out + ((int64_t)(q0 + rho / G) * Hq + h * G + rho % G) * D;
      for (int c = lg; c < D; c += 2) o[c] = 0.0f;
    }
    return;
  }
  // Score waves whose rows all lie past the request's rows still take part
  // in the copies, the unpacking and the barriers; their scores are all
  // masked.
  const int P0 = S - nq;  // position of the chunk's first query
  // this lane's query row rb + li: last token it may see, min(S - 1,
  // position); -1 for rows past the request's rows (all masked)
  const int rho_l = rb + li;
  const int lim = rho_l < rows_r ? min(S - 1, P0 + rho_l / G) : -1;
  float* const part = slot_out < 0 ? nullptr : a.parts + ((int64_t)slot_out * H + h) * chunk_part_floats(D);
  uint8_t* const kbuf = smem + LY::KB0;
  uint8_t* const vbuf = smem + LY::VB0;
  uint8_t* const wbuf = smem + LY::WB0;
  float* const lbuf = reinterpret_cast<float*>(smem + LY::LB0);
  auto barrier = [&]() {
    wait_lgkm0();  // this wave's LDS reads and writes are done
    __builtin_amdgcn_s_barrier();
    __asm__ __volatile__("" ::: "memory");
  };
  struct TqW {
    half8 ha, la, hb, lb, z;  // weights of pages a and b (hi, lo); zero-term operand
  };
  // this pair's weight slot of stage j
  auto wslot = [&](int j) { return wbuf + ((j & 1) * NSW + sw) * LY::WPW; };

  // Stage j of the loops below is a TQ3 pair for j < st3, else an FP8 pair.
  // Pass p (one barrier each, p = 0 .. n_st): the score waves issue stage
  // p's score product and finish stage p - 1 (scores, softmax, weights into
  // LDS) while the PV waves take stage p - 2 with the weights handed over in
  // pass p - 1.
  // Ring units: a TQ3 pair is one unit (one slot), an FP8 pair two (page a, page
  // b).  FP8 unit i = u - st3 follows the TQ3 units round the eight slots, then
  // takes the four behind them, and so on round all twelve.
  const int n_units = st3 + 2 * n_f8;
  // a place in the ring: the unit's FP8 index modulo the twelve slots (0 for a TQ3
  // unit), the byte of its slot
  struct Place {
    int k;
    uint32_t so;
  };
  auto next8 = [&](Place& c) {  // the place of the next FP8 unit
    if (++c.k == CSLOTS8) {
      c.k = 0;
      c.so = (uint32_t)(st3 % CSLOTS) * STAGE;
    } else if (c.k == CSLOTS) {
      c.so = CSLOTS * STAGE;
    } else {
      c.so += STAGE;
      if (c.k < CSLOTS && c.so == CSLOTS * STAGE) c.so = 0;
    }
  };
  const Place first8 = {0, (uint32_t)(st3 % CSLOTS) * STAGE};
  // The item's pairs reach LDS in blocks of 64 (1 KiB), the TQ3 pairs' blocks
  // first, four buffers, copied by every copying wave itself with the counted copies
  // of the pages (so its own wait for a page makes the block visible to it, and
  // the barrier of a pass to the other waves); block k + 2 is copied just
  // before the first page of block k, as block k + 1 may be the last, short one of
  // the TQ3 pairs.
  const uint8_t* lsb = smem + LY::LS0;
  const int nb3 = (st3 + 63) / 64, n_blk = nb3 + (n_f8 + 63) / 64;
  // stage j -> {lp_a, id_a, lp_b, id_b}.  A reader keeps one block in registers, lane
  // l holding its entry l, and takes an entry with lane reads: one LDS read per
  // 64 stages.
  struct Reader {
    int4 v;
    int k;
  };
  auto stage_at = [&](int j, Reader& rd) {
    j = __builtin_amdgcn_readfirstlane(j);
    if (j >= n_st) return make_int4(CMASK_LP, 0, CMASK_LP, 0);  // past the list: never used
    if (j >= st3) j += 64 * nb3 - st3;
    if ((j >> 6) != rd.k) {
      rd.k = j >> 6;
      rd.v = *reinterpret_cast<const int4*>(lsb + ((j >> 6) % LY::LBUF) * 1024 + lane * 16);
      wait_lgkm0();  // here, so that the lane reads after the join wait for nothing
    }
    const int l = j & 63;
    return make_int4(__builtin_amdgcn_readlane(rd.v.x, l), __builtin_amdgcn_readlane(rd.v.y, l),
                     __builtin_amdgcn_readlane(rd.v.z, l), __builtin_amdgcn_readlane(rd.v.w, l));
  };
  // ---- the copies.  At d = 256 the PV waves' products bound a TQ3 pass, so the
  // score waves copy; at d = 128 they have half the products and the score waves'
  // chain of scores, softmax and weights bounds a pass, so the PV waves copy
  // (per TQ3 and FP8 pass, one workgroup on every CU: d = 256 2.02 and 1.88 us with
  // the score waves copying, 2.21 and 2.12 with the PV waves; d = 128 1.46 and 1.67,
  // 1.31 and 1.54).
  constexpr bool COPY_PV = D == 128;
  const int cwv = wid % NSW;
  // This wave's share of a unit's copies: OPS_W whole KiB (TQ3: KiB w OPS_W ..
  // of the two pages laid end to end, so waves 0 and 1 copy page a and waves
  // 2 and 3 page b; FP8: copies w OPS_W .. of the page's 2 NI, waves 0 and 1 its
  // K and waves 2 and 3 its V, block-permuted as in dma_fp8_page), and for the
  // even waves one small copy (TQ3: the 32-byte tail of the wave's page; FP8:
  // the two scales, copied by both so that every unit costs each wave the same
  // number of copies).
  const int layer = a.layer;
  const int hw = cwv >> 1;  // page of a TQ3 pair; K or V of an FP8 page
  const bool tail_wave = !(cwv & 1);
  const uint32_t ring_lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem);
  const uint8_t* stab3 = reinterpret_cast<const uint8_t*>(a.list3 + (int64_t)r * a.stride + 2 * it0.z);
  const uint8_t* stab8 = reinterpret_cast<const uint8_t*>(a.list8 + (int64_t)r * a.stride + 2 * it1.x);
  const uint8_t* tq3_h = P.tq3 + ((int64_t)layer * P.n_tq3 * H + h) * R3;
  const uint8_t* fp8_h = P.fp8 + ((int64_t)layer * P.n_fp8 * H + h) * R8 + hw * (16 * D) + (cwv & 1) * OPS_W * 64;
  const uint8_t* scl_h = reinterpret_cast<const uint8_t*>(P.fp8_scales + ((int64_t)layer * P.n_fp8 * H + h) * 2);
  const uint32_t v3 = 16u * lane + 1024u * (OPS_W * (cwv & 1));
  const uint32_t v8 = (uint32_t)((lane >> 2) * D + 16 * ((lane & 3) ^ (lane >> 4)));
  const uint32_t dst3 = ring_lds + hw * R3 + (cwv & 1) * OPS_W * 1024, tail3 = ring_lds + hw * R3 + 16 * D;
  const uint32_t dst8 = ring_lds + hw * (16 * D) + (cwv & 1) * OPS_W * 1024, tail8 = ring_lds + R8;
  const uint32_t lst_lds = ring_lds + LY::LS0;
  static_assert(OPS_W * 2 == MAIN_KB && OPS_W * 2 == NI, "two waves copy one page, or one half of an FP8 page");
  // unit at byte `so` of the ring: the TQ3 page of this wave, or its share of an FP8 page
  auto issue3 = [&](uint32_t id, uint32_t so) {
    const uint8_t* src = tq3_h + (uint64_t)id * (uint32_t)(H * R3);
#pragma unroll
    for (int i = 0; i < OPS_W; ++i) dma16<0>(v3 + 1024u * i, src, dst3 + so + 1024 * i);
    if (tail_wave && lane < 8) dma4(16 * D + 4 * lane, src, tail3 + so);
  };
  auto issue8 = [&](uint32_t id, uint32_t so) {
    const uint8_t* src = fp8_h + (uint64_t)id * (uint32_t)(H * R8);
#pragma unroll
    for (int i = 0; i < OPS_W; ++i) dma16<0>(v8, src + 64 * i, dst8 + so + 1024 * i);
    if (tail_wave && lane < 2) dma4(4 * lane, scl_h + (uint64_t)id * (uint32_t)(8 * H), tail8 + so);
  };
  auto issue_list = [&](int k) {  // block k of the lists -> buffer k % LBUF
    dma16<0>(16u * lane, k < nb3 ? stab3 + 1024 * k : stab8 + 1024 * (k - nb3), lst_lds + (k % LY::LBUF) * 1024);
  };
  // Ring bookkeeping: `issued` units have been copied so far.  The slot of
  // TQ3 pair s is free from pass s + 2 on (its keys are unpacked in pass s - 1,
  // its values and key-norm corrections read in pass s + 1), those of the FP8
  // pair of pass s from pass s + 3 on (read by the score waves in pass s, by
  // the copying waves in pass s + 2), the slots behind the ring from pass st3 + 2
  // on (the last TQ3 values are read in pass st3 + 1).
  int issued = 0;
  auto stage_of_unit = [&](int u) { return u < st3 ? u : st3 + (u - st3) / 2; };
  Reader rd_iss = {make_int4(0, 0, 0, 0), -1};
  int4 e_iss = make_int4(0, 0, 0, 0);  // the entry of unit `issued`'s stage
  Place pl = {0, 0};                   // its place
  auto refill = [&](int pass) {
    while (issued < n_units) {
      const int i = issued - st3;
      int ready;  // the pass from which the unit's slot is free
      if (i < CSLOTS) ready = issued < CSLOTS ? -1 : issued - CSLOTS + 2;
      else if (i < CSLOTS8) ready = st3 > 0 ? st3 + 2 : -1;
      else ready = st3 + (i - CSLOTS8) / 2 + 3;
      if (ready > pass) break;
      // a masked page b reads page a (its weights are zero, its values have to be finite);
      // page a of a pair is never masked
      const int id_b = e_iss.z == CMASK_LP ? e_iss.y : e_iss.w;
      const bool first = i < 0 || !(i & 1);  // the first unit of its stage
      if (first) {
        const int j = i < 0 ? issued : (i >> 1) + 64 * nb3;
        if ((j & 63) == 0 && (j >> 6) + 2 < n_blk) issue_list((j >> 6) + 2);
      }
      ++issued;
      if (i < 0) {
        issue3(__builtin_amdgcn_readfirstlane(hw ? id_b : e_iss.y), pl.so);
        pl.so += STAGE;
        if (pl.so == CSLOTS * STAGE) pl.so = 0;
      } else {
        issue8(__builtin_amdgcn_readfirstlane(first ? e_iss.y : id_b), pl.so);
        next8(pl);
      }
      if (i < 0 || (i & 1)) e_iss = stage_at(stage_of_unit(issued), rd_iss);
    }
  };
  // before the barrier of pass p: pair p + 1 of the TQ3 pairs (its keys are
  // unpacked in pass p), pair p of the FP8 pairs has landed; the copies after it
  // (four units once the ring is full) stay in flight
  auto wait_for = [&](int p) {
    int u;
    if (p + 1 < st3) u = p + 1;
    else if (p >= st3 && p < n_st) u = st3 + 2 * (p - st3) + 1;
    else return;
    if (issued - 1 - u >= 4) {
      if (tail_wave) wait_vmcnt<4 * (OPS_W + 1)>();
      else wait_vmcnt<4 * OPS_W>();
    } else {
      wait_vmcnt<0>();
    }
  };
  auto start_copies = [&]() {
    for (int k = 0; k < min(n_blk, 2); ++k) issue_list(k);
    wait_vmcnt<0>();
    e_iss = stage_at(0, rd_iss);
    refill(-1);
  };
  if (score_wave) {
    // ======================= score waves =======================
    // The score waves' instructions go first on the SIMD (their weights gate
    // the next pass); the PV waves fill the gaps.
    __builtin_amdgcn_s_setprio(2);
    float neg1 = -1.0f;  // kept in a register (see split2)
    __asm__ __volatile__("" : "+v"(neg1));
    const int rho_c = min(rho_l, rows_r - 1);  // a valid row to load for masked lanes
    const uint16_t* qrow_ptr = a.q + ((int64_t)(q0 + rho_c / G) * Hq + h * G + rho_c % G) * D;
    if constexpr (!COPY_PV) start_copies();
    // ---- rotated query of this lane's row, q_rot = R q (R = d^-1/2 H
    // diag(sigma)), times the softmax scale log2(e)/sqrt(d) (scores come out
    // in base 2) and a power-of-two row scale qsc that puts the row's
    // largest entry in [128, 256), as three E4M3 terms t0 + t1 + t2 (each
    // the E4M3 rounding of what the earlier ones left; the remainder is at
    // most 2^-14 of an entry, or 2^-10 where that is more).  B operand of
    // the 32x32x64 fp8 MFMA: lane (li, lg) holds, for k-step s, channels 64 s +
    // 32 lg + j (j < 32) of row rb + li; the key operand uses the same order.
    v8i qt[3][NK8];
    float qinv;
    {
      float x[NK8][32];
#pragma unroll
      for (int s = 0; s < NK8; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const uint4 raw = *reinterpret_cast<const uint4*>(qrow_ptr + 64 * s + 32 * lg + 8 * v);
          const uint16_t* hb = reinterpret_cast<const uint16_t*>(&raw);
          // the signs sit 4-byte aligned in the control buffer
          const uint32_t* sgw = reinterpret_cast<const uint32_t*>(P.sigma + 64 * s + 32 * lg + 8 * v);
          const uint2 sg2 = make_uint2(sgw[0], sgw[1]);
          const int8_t* sg = reinterpret_cast<const int8_t*>(&sg2);
#pragma unroll
          for (int j = 0; j < 8; ++j) x[s][8 * v + j] = bf16_to_f32(hb[j]) * (float)sg[j];
        }
      // Walsh-Hadamard butterflies over the channel bits: j (strides 1-16)
      // and s (strides 64 ..) inside the lane, lg (stride 32) across lanes
      // l ^ 32; the stages commute
#pragma unroll
      for (int st = 1; st < 32; st <<= 1)
#pragma unroll
        for (int s = 0; s < NK8; ++s)
#pragma unroll
          for (int j = 0; j < 32; ++j)
            if (!(j & st)) {
              const float x0 = x[s][j], x1 = x[s][j + st];
              x[s][j] = x0 + x1;
              x[s][j + st] = x0 - x1;
            }
#pragma unroll
      for (int st = 1; st < NK8; st <<= 1)
#pragma unroll
        for (int s = 0; s < NK8; ++s)
          if (!(s & st)) {
#pragma unroll
            for (int j = 0; j < 32; ++j) {
              const float x0 = x[s][j], x1 = x[s + st][j];
              x[s][j] = x0 + x1;
              x[s + st][j] = x0 - x1;
            }
          }
      const float sgn32 = (lane & 32) ? -1.0f : 1.0f;
      const float qscale = rsqrtf((float)D) * a.sm_log2;
      float amax = 0.0f;
#pragma unroll
      for (int s = 0; s < NK8; ++s)
#pragma unroll
        for (int j = 0; j < 32; ++j) {
          x[s][j] = fmaf(sgn32, x[s][j], lane_xor<32>(x[s][j], lane)) * qscale;
          amax = fmaxf(amax, fabsf(x[s][j]));
        }
      amax = fmaxf(amax, lane_xor<32>(amax, lane));
      int ex = 0;
      (void)frexpf(amax, &ex);  // amax in [2^(ex-1), 2^ex)
      const bool ok = rho_l < rows_r && amax > 0.0f;
      const float qsc = ok ? ldexpf(1.0f, 8 - ex) : 0.0f;
      qinv = ok ? ldexpf(1.0f, ex - 8) : 1.0f;  // (the terms of such a row are all zero)
#pragma unroll
      for (int s = 0; s < NK8; ++s)
#pragma unroll
        for (int w = 0; w < 8; ++w) {
          uint32_t b0 = 0, b1 = 0, b2 = 0;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            float v = x[s][4 * w + k] * qsc;
            const uint32_t e0 = f32_to_e4m3(v);
            v -= e4m3_to_f32(e0);
            const uint32_t e1 = f32_to_e4m3(v);
            v -= e4m3_to_f32(e1);
            const uint32_t e2 = f32_to_e4m3(v);
            b0 |= e0 << (8 * k);
            b1 |= e1 << (8 * k);
            b2 |= e2 << (8 * k);
          }
          qt[0][s][w] = (int)b0;
          qt[1][s][w] = (int)b1;
          qt[2][s][w] = (int)b2;
        }
    }

    float m_run = CM_INIT, l_run = 0.0f;  // this lane's row; l_run over its tokens
    const float smk = a.sm_log2;
    // Online softmax over the base-2 scores sc[16] of this lane's query row
    // (its 16 tokens of the tile; the other 16 sit in lane l ^ 32).  The
    // reference max moves (lazily, when a score passes it by 2^8): alpha is
    // the factor the PV accumulators still owe, exactly 1 where the
    // reference stayed (the PV wave skips the rescale when no row of its
    // tile moved).
    auto softmax = [&](float* sc, float& alpha) {
      float mx = sc[0];
#pragma unroll
      for (int k = 1; k < 16; ++k) mx = fmaxf(mx, sc[k]);
      mx = fmaxf(mx, lane_xor<32>(mx, lane));
      const float m_new = mx > m_run + 8.0f ? mx : m_run;
      alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      float lsum = 0.0f;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        sc[k] = __builtin_amdgcn_exp2f(sc[k] - m_new);  // -inf -> 0
        lsum += sc[k];
      }
      l_run = fmaf(l_run, alpha, lsum);
    };
    // weights p[0..7] as an fp16 hi + lo pair (one token can carry most of
    // a row's mass, and its weight, taken against a lagging reference max,
    // is then not a power of two; a single fp16 rounding of it moves the
    // output by up to 2^-12 of that token's value)
    auto split8 = [&](const float* p, half8& hi, half8& lo) {
      uint32_t hh4[4], ll4[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) split2(p[2 * k], p[2 * k + 1], neg1, hh4[k], ll4[k]);
      hi = h8u(hh4[0], hh4[1], hh4[2], hh4[3]);
      lo = h8u(ll4[0], ll4[1], ll4[2], ll4[3]);
    };
    // hand the weights of stage j (and the rescale the PV accumulators owe
    // before them; a TQ3 pair's zero term) to the PV waves
    auto put_weights = [&](int j, const TqW& w, float alpha, auto zero) {
      uint8_t* ws = wslot(j);
      *reinterpret_cast<half8*>(ws + 0 * 1024 + 16 * lane) = w.ha;
      *reinterpret_cast<half8*>(ws + 1 * 1024 + 16 * lane) = w.la;
      *reinterpret_cast<half8*>(ws + 2 * 1024 + 16 * lane) = w.hb;
      *reinterpret_cast<half8*>(ws + 3 * 1024 + 16 * lane) = w.lb;
      if constexpr (decltype(zero)::value) *reinterpret_cast<half8*>(ws + 4 * 1024 + 16 * lane) = w.z;
      reinterpret_cast<float*>(ws + LY::WF_ALPHA)[lane] = alpha;
    };

    // ---- unpacking of a TQ3 pair (the 256 threads of the score waves, from
    // the raw stage at rs):
    //  keys: threads 0-127, one code chunk (token, channel quarter) each:
    //    codes -> E4M3 codebook bytes (one v_perm per 4 codes) in the score
    //    product's A layout, kb[k-step][lane (32 lg + token of the pair)][32];
    //  values: threads 128-255, one code chunk (16 channels, 4 tokens) each:
    //    code bytes in the PV product's A layout, vb[page][block][lane][8]
    //    (lane 32 hk + rr: channel CL (rr % 16) + 2 mb + rr / 16, tokens 4
    //    hk .. 4 hk + 3 then 8 + 4 hk .. 8 + 4 hk + 3, the order in which
    //    the score tile hands each lane its weights);
    //  per (page, block, row rr): the V scale split as (hi, lo) fp16 (hi
    //    keeps 8 significant bits, so code x hi is exact in fp16) and the V
    //    zero.
    // The keys of a pair are unpacked one pass before its score product, its
    // values one pass after it (with its scores).
    auto unpack_k = [&](const uint8_t* rs, uint8_t* kb) {  // threads 0-127
      const int p = tid >> 6, tok = tid & 15, g = (tid >> 4) & 3;
      uint32_t dw[NDW];
      read_chunk<NDW>(dw, rs + p * R3, 16 * g + tok);
#pragma unroll
      for (int q8 = 0; q8 < CL / 8; ++q8) {
        uint32_t o[8];
#pragma unroll
        for (int w = 0; w < 8; ++w) o[w] = __builtin_amdgcn_perm(KLUT_HI, KLUT_LO, quad_sel<NDW>(dw, 8 * q8 + w));
        const int c0 = g * QQ + 32 * q8;  // first channel of these 32 bytes
        uint4* dst = reinterpret_cast<uint4*>(kb + ((c0 / 64) * 64 + 32 * ((c0 / 32) & 1) + 16 * p + tok) * 32);
        dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
        dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
      }
    };
    auto unpack_v = [&](const uint8_t* rs, uint8_t* vb) {  // threads 128-255
      const int u = tid - 128;
      const int p = u >> 6, r0 = u & 15, g = (u >> 4) & 3;
      uint32_t dw[NDW];
      read_chunk<NDW>(dw, rs + p * R3 + 6 * D, 16 * g + r0);
      uint8_t* base = vb + (p * NMB * 64 + 32 * (g & 1) + r0) * 8 + 4 * (g >> 1);
#pragma unroll
      for (int q = 0; q < CL; ++q)
        *reinterpret_cast<uint32_t*>(base + ((q >> 1) * 64 + 16 * (q & 1)) * 8) = quad_sel<NDW>(dw, q);
    };
    auto unpack_side = [&](const uint8_t* rs, uint8_t* vb) {
      if (NMB * 32 >= 64 * NSW || tid < NMB * 32) {  // whole waves (every score wave at d = 256)
        const int mb = tid >> 5, rr = tid & 31, ch = CL * (rr & 15) + 2 * mb + (rr >> 4);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const half2v s1 = bcast(*reinterpret_cast<const _Float16*>(rs + p * R3 + 12 * D + 32 + 2 * ch));
          const half2v sh = hi8x2(s1);
          const half2v sp = {sh[0], s1[0] - sh[0]};  // exact split
          *reinterpret_cast<half2v*>(vb + LY::VX + ((p * NMB + mb) * 32 + rr) * 4) = sp;
          *reinterpret_cast<_Float16*>(vb + LY::VX + LY::SX + ((p * NMB + mb) * 32 + rr) * 2) =
              *reinterpret_cast<const _Float16*>(rs + p * R3 + 14 * D + 32 + 2 * ch);
        }
      }
    };

    // S^T = K Q^T of the pair whose keys are unpacked in kb: M = the pair's
    // 32 tokens (page a, then page b), N = the wave's 32 rows, one chain of
    // three MFMAs (one per query term) per k-step
    auto tq3_qk = [&](const uint8_t* kb, float16v& st, auto rev) {
      st = float16v{};
#pragma unroll
      for (int s_ = 0; s_ < NK8; ++s_) {
        const int s = decltype(rev)::value ? NK8 - 1 - s_ : s_;
        const v8i A = *reinterpret_cast<const v8i*>(kb + (s * 64 + lane) * 32);
#pragma unroll
        for (int t = 0; t < 3; ++t)
          st = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A, qt[t][s], st, 0, 0, 0, 0, 0, 0);
      }
    };
    // Scores and weights of the TQ3 pair e from its score product st and the
    // key-norm corrections gamma in its raw stage rs.  Lane (li, lg)
    // receives tokens 4 lg .. 4 lg + 3 and 8 + 4 lg .. of each page, which
    // are exactly the k-slots of its weight operand.  `masked`: some token
    // of the pair lies past the chunk's first query.
    auto tq3_scores = [&](const uint8_t* rs, const float16v& st, const int4& e, TqW& w, float& alpha,
                          auto masked) {
      // element e: token 8 (e / 4) + 4 lg + e % 4 of the pair (page a below 16)
      uint2 gw[4];
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)
        gw[e4] = *reinterpret_cast<const uint2*>(rs + (e4 >> 1) * R3 + 12 * D + 16 * (e4 & 1) + 8 * lg);
      float sc[16];
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const int t0 = (e4 < 2 ? e.x : e.z) * PAGE + 8 * (e4 & 1) + 4 * lg;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float v = st[4 * e4 + u] * qinv * (float)reinterpret_cast<const _Float16*>(&gw[e4])[u];
          if constexpr (decltype(masked)::value)
            sc[4 * e4 + u] = t0 + u <= lim ? v : -INFINITY;
          else
            sc[4 * e4 + u] = v;
        }
      }
      softmax(sc, alpha);
      split8(sc, w.ha, w.la);
      split8(sc + 8, w.hb, w.lb);
      const float ra_ = ((sc[0] + sc[1]) + (sc[2] + sc[3])) + ((sc[4] + sc[5]) + (sc[6] + sc[7]));
      const float rb_ = ((sc[8] + sc[9]) + (sc[10] + sc[11])) + ((sc[12] + sc[13]) + (sc[14] + sc[15]));
      uint32_t zh, zl;
      split2(ra_, rb_, neg1, zh, zl);
      w.z = h8u(zh, zl, 0u, 0u);  // (R_a, R_b) hi, then lo
    };
    // a pair whose pages both end before the chunk's first query needs no mask
    auto unmasked = [&](const int4& e) { return (max(e.x, e.z) + 1) * PAGE <= P0 + 1; };

    // ---- passes over the TQ3 pairs.  Pass p (after barrier p + 1) issues
    // the score product of pair p (keys unpacked in pass p - 1) and, while
    // the matrix unit works on it, finishes pair p - 1 (scores from the
    // product issued in pass p - 1, softmax, weights into LDS) and unpacks
    // the keys of pair p + 1 and the values of pair p - 1; the PV waves take
    // pair p - 2.  One straight block per wave kind; scheduling fences place
    // the twelve MFMAs between segments of the VALU and LDS work (left to
    // itself the compiler issued all twelve first).
    float16v st_prev = {};                // score product of stage p - 1
    int4 e_prev = make_int4(0, 0, 0, 0);  // entries of stage p - 1
    auto tq3_pass = [&](int p, float16v& st, auto masked, auto key_kind) {
      constexpr bool KK = decltype(key_kind)::value;  // this wave unpacks keys (else values)
      const uint8_t* kb = kbuf + (p & 1) * LY::KB;
      uint8_t* kb_next = kbuf + ((p + 1) & 1) * LY::KB;
      uint8_t* vb_prev = vbuf + ((p + 1) & 1) * LY::VB;  // buffer (p - 1) & 1
      const uint8_t* rs_prev = smem + ((p + CSLOTS - 1) % CSLOTS) * STAGE;
      const uint8_t* rs_next = smem + ((p + 1) % CSLOTS) * STAGE;
      // k-step of the i-th step of the product (the two kinds take the
      // k-steps in opposite orders, which keeps the compiler from merging
      // the two blocks' products)
      auto kstep = [&](int i) { return KK ? i : NK8 - 1 - i; };
      auto ld_a = [&](int i) { return *reinterpret_cast<const v8i*>(kb + (kstep(i) * 64 + lane) * 32); };
      v8i A[2];
      A[0] = ld_a(0);
      A[1] = ld_a(1);
      uint2 gw[4];
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)
        gw[e4] = *reinterpret_cast<const uint2*>(rs_prev + (e4 >> 1) * R3 + 12 * D + 16 * (e4 & 1) + 8 * lg);
      st = float16v{};
      // MFMA m of the product (k-step m / 3, query term m % 3); the operand of
      // the k-step after next is read once the last MFMA of a k-step is issued
      auto mf = [&](int m) {
        const int i = m / 3, t = m % 3;
        if (i >= NK8) return;  // d = 128: six MFMAs
        st = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A[i & 1], qt[t][kstep(i)], st, 0, 0, 0, 0, 0,
                                                             0);
        if (t == 2 && i + 2 < NK8) A[i & 1] = ld_a(i + 2);
        __builtin_amdgcn_sched_barrier(0);
      };
      // pair p - 1: scores, softmax and weights, between the MFMAs
      float sc[16];
      auto scores = [&](int e4) {
        const int t0 = (e4 < 2 ? e_prev.x : e_prev.z) * PAGE + 8 * (e4 & 1) + 4 * lg;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          // st * gamma as one mixed-precision FMA; the power-of-two row
          // factor qinv enters with the max and the exponent (exact)
          const float v = __builtin_fmaf((float)reinterpret_cast<const _Float16*>(&gw[e4])[u], st_prev[4 * e4 + u], 0.0f);
          if constexpr (decltype(masked)::value)
            sc[4 * e4 + u] = t0 + u <= lim ? v : -INFINITY;
          else
            sc[4 * e4 + u] = v;
        }
      };
      float m_new, alpha, lsum = 0.0f;
      auto ex = [&](int k0, int k1) {
#pragma unroll
        for (int k = k0; k < k1; ++k) {
          sc[k] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[k], qinv, -m_new));  // -inf -> 0
          lsum += sc[k];
        }
      };
      TqW w;
      mf(0);
      scores(0);
      scores(1);
      __builtin_amdgcn_sched_barrier(0);
      mf(1);
      scores(2);
      scores(3);
      __builtin_amdgcn_sched_barrier(0);
      mf(2);
      {
        float mx = sc[0];
#pragma unroll
        for (int k = 1; k < 16; ++k) mx = fmaxf(mx, sc[k]);
        mx = fmaxf(mx, lane_xor<32>(mx, lane)) * qinv;
        m_new = mx > m_run + 8.0f ? mx : m_run;
        alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
      }
      __builtin_amdgcn_sched_barrier(0);
      mf(3);
      ex(0, 6);
      __builtin_amdgcn_sched_barrier(0);
      mf(4);
      ex(6, 11);
      __builtin_amdgcn_sched_barrier(0);
      mf(5);
      ex(11, 16);
      l_run = fmaf(l_run, alpha, lsum);
      __builtin_amdgcn_sched_barrier(0);
      mf(6);
      split8(sc, w.ha, w.la);
      __builtin_amdgcn_sched_barrier(0);
      mf(7);
      split8(sc + 8, w.hb, w.lb);
      __builtin_amdgcn_sched_barrier(0);
      mf(8);
      {
        const float ra_ = ((sc[0] + sc[1]) + (sc[2] + sc[3])) + ((sc[4] + sc[5]) + (sc[6] + sc[7]));
        const float rb_ = ((sc[8] + sc[9]) + (sc[10] + sc[11])) + ((sc[12] + sc[13]) + (sc[14] + sc[15]));
        uint32_t zh, zl;
        split2(ra_, rb_, neg1, zh, zl);
        w.z = h8u(zh, zl, 0u, 0u);  // (R_a, R_b) hi, then lo
      }
      put_weights(p - 1, w, alpha, std::true_type{});
      __builtin_amdgcn_sched_barrier(0);
      // then this wave's share of the unpacking: keys of pair p + 1 or
      // values of pair p - 1, and the values' side data of pair p - 1
      mf(9);
      if constexpr (KK)
        unpack_k(rs_next, kb_next);
      else
        unpack_v(rs_prev, vb_prev);
      __builtin_amdgcn_sched_barrier(0);
      mf(10);
      unpack_side(rs_prev, vb_prev);
      __builtin_amdgcn_sched_barrier(0);
      mf(11);
    };
    Reader rd_prev = {make_int4(0, 0, 0, 0), -1};
    if constexpr (!COPY_PV) wait_for(-1);
    barrier();  // pair 0 has landed
    if (st3 > 0 && wid < 2) unpack_k(smem, kbuf);
    for (int p = 0; p < st3; ++p) {
      if constexpr (!COPY_PV) wait_for(p);
      barrier();  // keys of pair p unpacked; raw pair p + 1 landed
      // (in the last pass the key unpacking reads a slot that holds no pair
      // and writes a buffer nobody reads any more)
      float16v st;
      if (p == 0) {
        if (wid < 2) {
          tq3_qk(kbuf, st, std::false_type{});
          unpack_k(smem + (1 % CSLOTS) * STAGE, kbuf + LY::KB);
        } else {
          tq3_qk(kbuf, st, std::true_type{});
        }
      } else if (unmasked(e_prev)) {
        if (wid < 2)
          tq3_pass(p, st, std::false_type{}, std::true_type{});
        else
          tq3_pass(p, st, std::false_type{}, std::false_type{});
      } else {
        if (wid < 2)
          tq3_pass(p, st, std::true_type{}, std::true_type{});
        else
          tq3_pass(p, st, std::true_type{}, std::false_type{});
      }
      if constexpr (!COPY_PV) refill(p);
      st_prev = st;
      e_prev = stage_at(p, rd_prev);
    }
    // ---- passes over the FP8 pairs: pass p scores pair p with plain queries as
    // fp16 (bf16 -> fp16 is exact for the query range) against its FP8 keys,
    // straight from the ring, and between those MFMAs finishes the weights of
    // stage p - 1 (for p = st3 the last TQ3 pair, whose values it also unpacks);
    // the last pass only finishes.  Score rows 0-15 are page a's tokens, 16-31
    // page b's; lane (li, lg) holds, for k-step s, channels (D/2) lg + 8 s + b
    // (b < 8) of its row.
    {
      half8 qop[NKS];
      if (n_f8 > 0) {
        const uint16_t* qrow = qrow_ptr + (D / 2) * lg;
#pragma unroll
        for (int s = 0; s < NKS; ++s) {
          const uint4 raw = *reinterpret_cast<const uint4*>(qrow + 8 * s);
          const uint16_t* hb = reinterpret_cast<const uint16_t*>(&raw);
#pragma unroll
          for (int j = 0; j < 8; ++j) qop[s][j] = (_Float16)bf16_to_f32(hb[j]);
        }
      }
      // key and value scales of the pages of FP8 stage p - 1, of the value scales the rest
      // already where it is found under a pass's last products (d = 128 has none left there)
      constexpr bool REST_EARLY = NKS > 10;
      float2 ksa_prev = make_float2(0.0f, 0.0f), ksb_prev = ksa_prev;
      Place pl8 = first8;  // of the next pair's page a
      for (int p = st3; p <= n_st; ++p) {
        const uint32_t so_a = pl8.so;
        next8(pl8);
        const uint32_t so_b = pl8.so;
        next8(pl8);
        if constexpr (!COPY_PV) wait_for(p);
        barrier();  // pair p visible
        if constexpr (!COPY_PV) refill(p);
        // (in the last pass the product reads slots that hold no pair and is not used)
        float16v st = {};
        uint4 kw[NKS / 2];  // this lane's key bytes: 16-byte block w holds k-steps 2 w, 2 w + 1
        const uint8_t* ra = smem + so_a;
        const uint8_t* rb_ = smem + so_b;
        // block-permuted page (see dma_fp8_page): token t's blocks NI 2 lg + w
        const int tok = li & 15;
        const uint8_t* pk = (li < 16 ? ra : rb_) + 512 * NI * lg + 64 * tok;
        const int sw = 16 * (tok >> 2);
#pragma unroll
        for (int w = 0; w < NKS / 2; ++w)
          kw[w] = *reinterpret_cast<const uint4*>(pk + 1024 * (w / 4) + (sw ^ (16 * (w % 4))));
        float2 ksa = *reinterpret_cast<const float2*>(ra + R8), ksb = *reinterpret_cast<const float2*>(rb_ + R8);
        auto rest_early = [&]() {
          if constexpr (REST_EARLY) {
            ksa.y = vscale_rest(ksa.y);
            ksb.y = vscale_rest(ksb.y);
          }
        };
        auto mf = [&](int s) {
          if (s < NKS) {
            const uint32_t k0 = s & 1 ? kw[s / 2].z : kw[s / 2].x, k1 = s & 1 ? kw[s / 2].w : kw[s / 2].y;
            const half8 K = h8(cvt_lo(k0), cvt_hi(k0), cvt_lo(k1), cvt_hi(k1));
            st = __builtin_amdgcn_mfma_f32_32x32x16_f16(K, qop[s], st, 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        };
        if (p == st3) {
#pragma unroll
          for (int s = 0; s < NKS; ++s) mf(s);
          rest_early();
          if (p > 0) {  // the last TQ3 pair
            TqW w;
            float alpha;
            const uint8_t* rs_prev = smem + ((p + CSLOTS - 1) % CSLOTS) * STAGE;
            uint8_t* vb_prev = vbuf + ((p + 1) & 1) * LY::VB;
            if (unmasked(e_prev))
              tq3_scores(rs_prev, st_prev, e_prev, w, alpha, std::false_type{});
            else
              tq3_scores(rs_prev, st_prev, e_prev, w, alpha, std::true_type{});
            if (wid >= 2) unpack_v(rs_prev, vb_prev);
            unpack_side(rs_prev, vb_prev);
            put_weights(p - 1, w, alpha, std::true_type{});
          }
        } else {
          TqW w;
          float sc[16], alpha, lsum = 0.0f, m_new;
          auto scores = [&](int e4) {
            const int t0 = (e4 < 2 ? e_prev.x : e_prev.z) * PAGE + 8 * (e4 & 1) + 4 * lg;
            const float kk = (e4 < 2 ? ksa_prev.x : ksb_prev.x) * smk;
#pragma unroll
            for (int u = 0; u < 4; ++u) sc[4 * e4 + u] = t0 + u <= lim ? st_prev[4 * e4 + u] * kk : -INFINITY;
          };
          auto ex = [&](int k0) {
#pragma unroll
            for (int k = k0; k < k0 + 4; ++k) {
              sc[k] = __builtin_amdgcn_exp2f(sc[k] - m_new);  // -inf -> 0
              lsum += sc[k];
            }
          };
          // weights of page a (k0 = 0) or b (k0 = 8), the rest of the page's V scale folded in
          auto split = [&](int k0, float vs, half8& hi, half8& lo) {
            const float vr = REST_EARLY ? vs : vscale_rest(vs);
            float pw[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) pw[k] = sc[k0 + k] * vr;
            split8(pw, hi, lo);
          };
          mf(0);
          scores(0);
          scores(1);
          mf(1);
          scores(2);
          scores(3);
          mf(2);
          {
            float mx = sc[0];
#pragma unroll
            for (int k = 1; k < 16; ++k) mx = fmaxf(mx, sc[k]);
            mx = fmaxf(mx, lane_xor<32>(mx, lane));
            m_new = mx > m_run + 8.0f ? mx : m_run;
            alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
          }
          mf(3);
          ex(0);
          mf(4);
          ex(4);
          mf(5);
          split(0, ksa_prev.y, w.ha, w.la);
          mf(6);
          ex(8);
          mf(7);
          ex(12);
          l_run = fmaf(l_run, alpha, lsum);
          mf(8);
          split(8, ksb_prev.y, w.hb, w.lb);
          mf(9);
          put_weights(p - 1, w, alpha, std::false_type{});
          rest_early();
#pragma unroll
          for (int s = 10; s < NKS; ++s) mf(s);
        }
        st_prev = st;
        ksa_prev = ksa;
        ksb_prev = ksb;
        e_prev = stage_at(p, rd_prev);
      }
    }
    barrier();  // the PV waves' last pass
    const float L = l_run + lane_xor<32>(l_run, lane);
    if (lg == 0) {
      if (part) reinterpret_cast<float2*>(part + 128 * D)[sw * 32 + li] = make_float2(m_run, L);
      else lbuf[sw * 32 + li] = L;
    }
    barrier();
  } else {
    // ========================= PV waves =========================
    // PV wave v owns the 32-channel blocks mb = NBW v .. NBW v + NBW - 1 of
    // the output for all 128 rows of the workgroup (the rows of every score
    // wave g), so each value operand is built once per workgroup.
    // Accumulators: O^T tile (32 channels x the 32 rows of score wave g) per
    // (block, g).  Lane (li, lg), element e holds row 32 g + li and tile row
    // rr = 8 (e / 4) + 4 lg + e % 4, which is channel CL (rr % 16) + 2 mb +
    // rr / 16 (the value unpacking lays its operands out for this order).
    constexpr int NBW = NMB / NSW;
    static_assert(NMB % NSW == 0 && NBW <= 2, "whole blocks per PV wave");
    const int pv = wid - NSW;
    float16v acc[NBW][NSW];
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
      for (int g = 0; g < NSW; ++g) acc[b][g] = float16v{};
    // weights of stage j from score wave g
    auto wsl = [&](int j, int g) { return wbuf + ((j & 1) * NSW + g) * LY::WPW; };
    // the rescales the weights of stage j carry, one per score wave (skipped
    // when every factor is 1: no reference max moved)
    auto rescale = [&](int j) {
      float al[NSW];
      bool any = false;
#pragma unroll
      for (int g = 0; g < NSW; ++g) {
        al[g] = reinterpret_cast<const float*>(wsl(j, g) + LY::WF_ALPHA)[lane];
        any |= al[g] != 1.0f;
      }
      if (__any(any)) {
#pragma unroll
        for (int b = 0; b < NBW; ++b)
#pragma unroll
          for (int g = 0; g < NSW; ++g) acc[b][g] *= al[g];  // column = this lane's row
      }
    };
    constexpr int REFILL_AT = 1, VP_AT = 5;
    // O^T += V^T P^T for the TQ3 pair of stage j (values unpacked in vb),
    // with exact V operands: v = zero + scale * code is split as scale_hi *
    // code + scale_lo * code + zero.  The products that reach fp32 accuracy:
    // (hi + lo weights) x scale_hi term, hi weights x scale_lo term (lo x
    // scale_lo sits below 2^-19 of the value), and the zero term as zero_a
    // (sum of weights over page a) + zero_b (same for b), whose sums the
    // MFMA completes across the two lane groups.
    // Order: page a's products for each score wave's rows, then page b's, then the
    // zero terms, so the first product waits for page a's operands only; page b's
    // are built between page a's products (a few VALU instructions in the shadow
    // of each MFMA), and the weights are read two steps ahead.
    struct VOp {
      half2v h[4], l[4];
    };
    struct W2 {
      half8 h, l;
    };
    // weights (hi, lo) of step t = 4 p + g: page p, score wave g
    auto ld_w2 = [&](int j, int t, W2& w) {
      const uint8_t* ws = wsl(j, t % NSW) + 2 * (t / NSW) * 1024 + 16 * lane;
      w.h = *reinterpret_cast<const half8*>(ws);
      w.l = *reinterpret_cast<const half8*>(ws + 1024);
    };
    auto tq3_pv = [&](int j) {
      const uint8_t* vb = vbuf + (j & 1) * LY::VB;
      const _Float16* zx = reinterpret_cast<const _Float16*>(vb + LY::VX + LY::SX);
      uint2 cw[2][NBW];
      half2v s2[2][NBW];
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int b = 0; b < NBW; ++b) {
          const int mb = NBW * pv + b;
          cw[p][b] = *reinterpret_cast<const uint2*>(vb + ((p * NMB + mb) * 64 + lane) * 8);
          s2[p][b] = *reinterpret_cast<const half2v*>(vb + LY::VX + ((p * NMB + mb) * 32 + li) * 4);
        }
      W2 w[3];
      ld_w2(j, 0, w[0]);
      ld_w2(j, 1, w[1]);
      rescale(j);
      // quarter q (two tokens) of the operand of (page p, block b)
      auto build = [&](VOp& o, int p, int b, int q) {
        const half2v sh = bcast(s2[p][b][0]), sl = bcast(s2[p][b][1]);
        const uint32_t c4 = q < 2 ? cw[p][b].x : cw[p][b].y;
        const half2v c = q & 1 ? cvt_code<true>(c4) : cvt_code<false>(c4);
        o.h[q] = c * sh;
        o.l[q] = c * sl;
      };
      VOp op[2][NBW];
#pragma unroll
      for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) build(op[0][b], 0, b, q);
      half8 zw[2], Az[NBW];
      auto ld_z = [&](int g) { zw[g & 1] = *reinterpret_cast<const half8*>(wsl(j, g) + 4 * 1024 + 16 * lane); };
#pragma unroll
      for (int t = 0; t < 2 * NSW; ++t) {
        const int p = t / NSW, g = t % NSW;
        if (t + 2 < 2 * NSW) ld_w2(j, t + 2, w[(t + 2) % 3]);
        if (t == 2 * NSW - 2) {
#pragma unroll
          for (int b = 0; b < NBW; ++b) {
            const int mb = NBW * pv + b;
            const _Float16 za = zx[mb * 32 + li], zb = zx[(NMB + mb) * 32 + li];
            Az[b] = half8{za, zb, za, zb, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f};
          }
          ld_z(0);
        }
        if (t == 2 * NSW - 1) ld_z(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
          for (int b = 0; b < NBW; ++b) {
            const VOp& o = op[p][b];
            const half8 A = k == 1 ? h8(o.l[0], o.l[1], o.l[2], o.l[3]) : h8(o.h[0], o.h[1], o.h[2], o.h[3]);
            acc[b][g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A, k == 2 ? w[t % 3].l : w[t % 3].h, acc[b][g], 0, 0, 0);
            if (p == 0 && k == 0) build(op[1][b], 1, b, g);
            __builtin_amdgcn_sched_barrier(0);
          }
        if constexpr (COPY_PV)
          if (t == REFILL_AT) refill(j + 2);  // the slots this pass frees
      }
#pragma unroll
      for (int g = 0; g < NSW; ++g) {
        const half8 z = zw[g & 1];
        if (g + 2 < NSW) ld_z(g + 2);
#pragma unroll
        for (int b = 0; b < NBW; ++b)
          acc[b][g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Az[b], z, acc[b][g], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // O^T += V^T P^T for the FP8 pair of stage j (weights hi + lo, the rest of the pages'
    // V scales folded in, their powers of two in the values): lane-chunks (rrow, lg) and
    // (rrow, lg + 2) of V, dword m = tokens 4 g' .. 4 g' + 3 of channel CL rrow + m
    Place pl8 = first8;  // of the next FP8 pair's page a
    // powers of two of the V scales of the pair at pl8, found a pass early (it has landed
    // by then) but for the first pair's
    float vp[2], vp_next[2];
    auto ld_vp = [&](Place c) {
      vp_next[0] = vscale_pow2(*reinterpret_cast<const float*>(smem + c.so + R8 + 4));
      next8(c);
      vp_next[1] = vscale_pow2(*reinterpret_cast<const float*>(smem + c.so + R8 + 4));
    };
    auto fp8_pv = [&](int j) {
      const int rrow = li & 15, hh = li >> 4;
      if (j == st3) ld_vp(pl8);
      vp[0] = vp_next[0];
      vp[1] = vp_next[1];
      uint32_t vw[2][NBW][2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const uint8_t* pvp = smem + pl8.so + PAGE * D + 64 * rrow;
        next8(pl8);
#pragma unroll
        for (int b = 0; b < NBW; ++b) {
          const int mb = NBW * pv + b;
          // block y of the row (see dma_fp8_page): KiB y / 4, place y % 4 ^ rrow / 4
          const int y = lg * NI + mb / 2;
          const uint8_t* pb = pvp + 1024 * (y >> 2) + 16 * ((y & 3) ^ (rrow >> 2)) + 8 * (mb & 1);
          const uint2 v0 = *reinterpret_cast<const uint2*>(pb);
          const uint2 v2 = *reinterpret_cast<const uint2*>(pb + 1024 * (NI / 2));
          vw[p][b][0] = hh ? v0.y : v0.x;
          vw[p][b][1] = hh ? v2.y : v2.x;
        }
      }
      W2 w[3];
      ld_w2(j, 0, w[0]);
      ld_w2(j, 1, w[1]);
      rescale(j);
      auto op_of = [&](int p, int b) {
        auto cvt = [&](uint32_t x, auto hi) { return __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(x, vp[p], decltype(hi)::value); };
        return h8(cvt(vw[p][b][0], std::false_type{}), cvt(vw[p][b][0], std::true_type{}),
                  cvt(vw[p][b][1], std::false_type{}), cvt(vw[p][b][1], std::true_type{}));
      };
      half8 A[2][NBW];
#pragma unroll
      for (int b = 0; b < NBW; ++b) A[0][b] = op_of(0, b);
#pragma unroll
      for (int t = 0; t < 2 * NSW; ++t) {
        const int p = t / NSW, g = t % NSW;
        if (t + 2 < 2 * NSW) ld_w2(j, t + 2, w[(t + 2) % 3]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int b = 0; b < NBW; ++b) {
            acc[b][g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[p][b], k ? w[t % 3].l : w[t % 3].h, acc[b][g], 0, 0, 0);
            if (t == 0 && k == 0) A[1][b] = op_of(1, b);
            __builtin_amdgcn_sched_barrier(0);
          }
        if (t == VP_AT) ld_vp(pl8);  // (past the last pair: some slot's bytes, not used)
        if constexpr (COPY_PV)
          if (t == REFILL_AT) refill(j + 2);
      }
    };
    if constexpr (COPY_PV) {
      start_copies();
      wait_for(-1);
    }
    barrier();  // pair 0 has landed
    for (int p = 0; p < 2; ++p) {  // the score product, then the weights of stage 0
      if constexpr (COPY_PV) wait_for(p);
      barrier();
      if constexpr (COPY_PV) refill(p);
    }
    for (int j = 0; j < st3; ++j) {  // pass j + 2
      if constexpr (COPY_PV) wait_for(j + 2);
      barrier();
      tq3_pv(j);
    }
    for (int j = st3; j < n_st; ++j) {
      if constexpr (COPY_PV) wait_for(j + 2);
      barrier();
      fp8_pv(j);
    }
    barrier();  // the rows' denominators
    if (part) {  // a part of a cut block: the accumulators as they stand
      float4* o = reinterpret_cast<float4*>(part) + (int64_t)pv * NBW * NSW * 256 + lane;
#pragma unroll
      for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int g = 0; g < NSW; ++g)
#pragma unroll
          for (int k = 0; k < 4; ++k)
            o[((b * NSW + g) * 4 + k) * 64] = make_float4(acc[b][g][4 * k], acc[b][g][4 * k + 1],
                                                          acc[b][g][4 * k + 2], acc[b][g][4 * k + 3]);
      return;
    }
    // ---- normalize and store: tile row rr = 8 kk + 4 lg + u (kk, u: the
    // lane's elements 4 kk + u and 8 + 4 kk + u) is chunk row rr % 16 = rr
    // for both halves hh = 0, 1 of every block, so this wave's channels
    // CL rr + 2 NBW pv .. + 2 NBW - 1 are contiguous: channel CL rr + 2 mb +
    // hh <- acc[mb - NBW pv][g][4 kk + 8 hh + u]
#pragma unroll
    for (int g = 0; g < NSW; ++g) {
      const int rho = xb * (NSW * 32) + g * 32 + li;
      if (rho < rows_r) {
        const float L = lbuf[g * 32 + li];
        const float inv = L > 0.0f ? 1.0f / L : 0.0f;
        float* o = a.out + ((int64_t)(q0 + rho / G) * Hq + h * G + rho % G) * D + 2 * NBW * pv;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int rr = 8 * kk + 4 * lg + u;
            if constexpr (NBW == 2)
              *reinterpret_cast<float4*>(o + CL * rr) =
                  make_float4(acc[0][g][4 * kk + u] * inv, acc[0][g][4 * kk + 8 + u] * inv,
                              acc[1][g][4 * kk + u] * inv, acc[1][g][4 * kk + 8 + u] * inv);
            else
              *reinterpret_cast<float2*>(o + CL * rr) =
                  make_float2(acc[0][g][4 * kk + u] * inv, acc[0][g][4 * kk + 8 + u] * inv);
          }
      }
    }
  }
}

// Grid (work item, KV head).
template <int D>
__global__ __launch_bounds__(64 * CW, 1) void chunk_kernel(ChunkArgs a) {
  extern __shared__ __align__(16) uint8_t smem[];
  const int gb = blockIdx.x;
  const int4 it0 = a.items[2 * gb], it1 = a.items[2 * gb + 1];  // (in the table whether planned or not)
  if (gb >= a.hdr[0]) return;
  chunk_block<D>(a, it0, it1, blockIdx.y, smem);
}

// Merge of the parts of cut blocks (Eq. softmax-merge): grid (cut block, KV
// head, score wave), one thread per lane of a PV wave, with its accumulators' layout.
template <int D>
__global__ __launch_bounds__(64 * NSW) void chunk_merge_kernel(ChunkArgs a, const int4* splits) {
  constexpr int CL = D / 16, NBW = D / 32 / NSW;
  if ((int)blockIdx.x >= a.hdr[1]) return;
  const int4 sp = splits[blockIdx.x];
  const int r = sp.x, xb = sp.y, n = sp.w, h = blockIdx.y, g = blockIdx.z;
  const int lane = threadIdx.x & 63, pv = threadIdx.x >> 6, li = lane & 31, lg = lane >> 5;
  const int G = a.P.group, H = a.P.n_kv_heads, Hq = H * G;
  const int q0 = a.cu_q[r], rows_r = (a.cu_q[r + 1] - q0) * G;
  const int rho = xb * (NSW * 32) + g * 32 + li;
  if (xb * (NSW * 32) + g * 32 >= rows_r) return;
  const float* base = a.parts + ((int64_t)sp.z * H + h) * chunk_part_floats(D);
  const int64_t step = (int64_t)H * chunk_part_floats(D);
  float M = -INFINITY;
  for (int k = 0; k < n; ++k) {
    const float2 ml = reinterpret_cast<const float2*>(base + k * step + 128 * D)[g * 32 + li];
    if (ml.y > 0.0f) M = fmaxf(M, ml.x);
  }
  float L = 0.0f;
  float4 o[NBW][4];
#pragma unroll
  for (int b = 0; b < NBW; ++b)
#pragma unroll
    for (int k = 0; k < 4; ++k) o[b][k] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 2
  for (int k = 0; k < n; ++k) {
    const float2 ml = reinterpret_cast<const float2*>(base + k * step + 128 * D)[g * 32 + li];
    const float f = ml.y > 0.0f ? __builtin_amdgcn_exp2f(ml.x - M) : 0.0f;
    L = fmaf(f, ml.y, L);
    const float4* src = reinterpret_cast<const float4*>(base + k * step) + (int64_t)pv * NBW * NSW * 256 + lane;
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float4 x = src[((b * NSW + g) * 4 + e) * 64];
        o[b][e].x = fmaf(f, x.x, o[b][e].x);
        o[b][e].y = fmaf(f, x.y, o[b][e].y);
        o[b][e].z = fmaf(f, x.z, o[b][e].z);
        o[b][e].w = fmaf(f, x.w, o[b][e].w);
      }
  }
  if (rho >= rows_r) return;
  const float inv = L > 0.0f ? 1.0f / L : 0.0f;
  float* dst = a.out + ((int64_t)(q0 + rho / G) * Hq + h * G + rho % G) * D + 2 * NBW * pv;
  // element 4 k' + u of block b is tile row 8 k' + 4 lg + u: chunk row rr = 8 kk +
  // 4 lg + u of half hh, k' = kk + 2 hh, channel CL rr + 2 b + hh of this wave's
  auto el = [](const float4& v, int u) { return u == 0 ? v.x : u == 1 ? v.y : u == 2 ? v.z : v.w; };
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int rr = 8 * kk + 4 * lg + u;
      if constexpr (NBW == 2)
        *reinterpret_cast<float4*>(dst + CL * rr) = make_float4(el(o[0][kk], u) * inv, el(o[0][kk + 2], u) * inv,
                                                                el(o[1][kk], u) * inv, el(o[1][kk + 2], u) * inv);
      else
        *reinterpret_cast<float2*>(dst + CL * rr) = make_float2(el(o[0][kk], u) * inv, el(o[0][kk + 2], u) * inv);
    }
}

hipError_t launch_chunk(const PoolView& P, int layer, int n_req, const uint16_t* q,
                        const int32_t* cu_q, int n_q_total, const int32_t* bt, const uint8_t* tags,
                        int max_pages, const int32_t* seq_lens, float* out, void* ws,
                        size_t ws_bytes, hipStream_t s) {
  ChunkArgs a;
  a.P = P;
  a.layer = layer;
  a.n_req = n_req;
  a.max_pages = max_pages;
  a.n_q_total = n_q_total;
  a.q = q;
  a.cu_q = cu_q;
  a.seq_lens = seq_lens;
  a.out = out;
  uint8_t* w = reinterpret_cast<uint8_t*>(ws);
  const ChunkWs wl = chunk_ws(n_req, max_pages, n_q_total, P.n_kv_heads, P.group, P.d, ws_bytes);
  int2* list8 = reinterpret_cast<int2*>(w + wl.list8);
  int2* list3 = reinterpret_cast<int2*>(w + wl.list3);
  int2* cum = reinterpret_cast<int2*>(w + wl.cum);
  int32_t* rbo = reinterpret_cast<int32_t*>(w + wl.rbo);
  int32_t* hdr = reinterpret_cast<int32_t*>(w + wl.hdr);
  int4* items = reinterpret_cast<int4*>(w + wl.items);
  int4* splits = reinterpret_cast<int4*>(w + wl.splits);
  a.stride = wl.stride;
  a.list8 = list8;
  a.list3 = list3;
  a.hdr = hdr;
  a.items = items;
  a.parts = reinterpret_cast<float*>(w + wl.parts);
  a.sm_log2 = 1.4426950408889634f / sqrtf((float)P.d);
  hipLaunchKernelGGL(chunk_lists_kernel, dim3(n_req), dim3(LIST_NT), 0, s, bt, tags, max_pages, wl.stride,
                     seq_lens, P.n_fp8, P.n_tq3, list8, list3, cum, P.ctrl + CTRL_ERR);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = P.d == 256 ? (size_t)ChunkLds<256>::TOTAL : (size_t)ChunkLds<128>::TOTAL;
  const void* kern = P.d == 256 ? (const void*)chunk_kernel<256> : (const void*)chunk_kernel<128>;
  // the dynamic-LDS limit is raised once per kernel instance and device
  static std::atomic<uint32_t> attr_done[64];
  int dev = 0;
  e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint32_t bit = P.d == 256 ? 2u : 1u;
  if (dev < 0 || dev >= 64 || !(attr_done[dev].load() & bit)) {
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) attr_done[dev].fetch_or(bit);
  }
  // row blocks of all requests: at most ceil(n_q_total G / 128) + n_req when
  // the query ranges do not overlap
  const int blocks = (int)chunk_blocks(n_q_total, P.group) + n_req;
  const int share = cu_share(P.n_kv_heads);
  // (where the cut falls depends on every request of the call; deterministic pools keep
  // a row's bits to its own request)
  const bool cut = !P.deterministic && wl.n_parts > 0 && chunk_may_cut(n_q_total, P.group, P.n_kv_heads);
  for (int b0 = 0; b0 < blocks; b0 += wl.n_items) {  // one turn where the workspace holds the call's items
    hipLaunchKernelGGL(chunk_plan_kernel, dim3(1), dim3(1024), 0, s, n_req, cu_q, n_q_total, seq_lens, max_pages,
                       P.group, blocks, b0, wl.n_items, share, cut ? 1 : 0, wl.n_parts, wl.stride, cum, rbo, hdr,
                       items, splits, P.ctrl + CTRL_ERR);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    int n = blocks - b0 < wl.n_items ? blocks - b0 : wl.n_items;
    if (cut && b0 == 0 && n < 2 * share) n = 2 * share;
    void* args[] = {&a};
    e = hipLaunchKernel(kern, dim3(n, P.n_kv_heads), dim3(64 * CW), args, lds, s);
    if (e != hipSuccess) return e;
    if (!cut || b0 > 0) continue;
    const dim3 mgrid(blocks < share ? blocks : share, P.n_kv_heads, NSW);
    if (P.d == 256)
      hipLaunchKernelGGL(chunk_merge_kernel<256>, mgrid, dim3(64 * NSW), 0, s, a, splits);
    else
      hipLaunchKernelGGL(chunk_merge_kernel<128>, mgrid, dim3(64 * NSW), 0, s, a, splits);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mkv
