// Pool-state kernels: FP8 append (Alg. 1 Append; Sec. 3.1 Recent tier), FP8 ->
// TQ3 migration (Alg. 1 Retier; Sec. 4.3 normalize-rotate-pack), TQ3 -> FP8
// promotion (Alg. 1 Promote), the compact per-format page lists (Sec. 4.1)
// and a zero-fill helper.
//
// Every result that the CPU oracle fixes bit for bit (page ids, tags, free
// lists, FP8 codes and scales, TQ3 codes, gamma, V scale/zero) is produced by
// integer arithmetic or by single IEEE operations in a fixed order; this file
// is compiled with -ffp-contract=off.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "mkv_append.h"
#include "mkv_internal.h"
#include "../../include/minima_kv.h"

namespace mkv {

static int grid_for(int64_t items, int cap) {
  return (int)(items < 1 ? 1 : (items < cap ? items : cap));
}

// ===========================================================================
// Append
// ===========================================================================

// One workgroup: validate the whole call, then hand out FP8 ids in ascending
// (request, page) order and list every page that receives tokens.  The touched
// pages of up to PLAN_NT requests form one run of entries, PLAN_KB consecutive
// ones per thread (request found by a binary search in the run's prefix sums,
// then stepped), every table load of a batch in flight together: the cost is
// round trips, so requests are not walked one after the other.  A call whose
// entries fit one batch (most prompts of a few requests) is loaded once,
// validated and listed after one scan; a longer one takes a validating pass
// and a listing pass.
constexpr int PLAN_NT = 1024, PLAN_KB = 4;
constexpr int PLAN_BATCH = PLAN_NT * PLAN_KB;
__global__ __launch_bounds__(PLAN_NT) void append_plan_kernel(int n_req, int32_t* bt, uint8_t* tags,
                                                              int max_pages, const int32_t* sb,
                                                              const int32_t* cu, int32_t* ctrl,
                                                              const int32_t* fp8_stack, int32_t* list,
                                                              int n_fp8, int n_new_total, int32_t* rc8) {
  __shared__ int scratch[32];
  __shared__ int s_err, s_need;
  __shared__ int s_base[PLAN_NT], s_p0[PLAN_NT];  // per request of the run: first entry, first page
  const int tid = threadIdx.x;
  if (tid == 0) {
    s_err = 0;
    s_need = 0;
  }
  __syncthreads();
  const int top = ctrl[CTRL_FP8_TOP];
  int err = 0;
  // rows of request r are cu[r] .. cu[r+1]-1 of an n_new_total-row input
  if (tid == 0 && (cu[0] != 0 || cu[n_req] != n_new_total)) err = MKV_DEVERR_RANGE;
  // requests r0 .. r0 + PLAN_NT - 1 -> their run of entries; returns its length
  auto load_run = [&](int r0) {
    const int r = r0 + tid;
    int touch = 0, p0 = 0;
    if (r < n_req) {
      const int n = cu[r + 1] - cu[r], s0 = sb[r];
      if (n < 0 || s0 < 0) {
        err |= MKV_DEVERR_RANGE;
      } else if (n > 0) {
        p0 = s0 / PAGE;
        const int p1 = (int)(((int64_t)s0 + n - 1) / PAGE);
        if (p1 >= max_pages) err |= MKV_DEVERR_RANGE;
        else touch = p1 - p0 + 1;
      }
    }
    int total;
    s_base[tid] = block_excl_scan(touch, scratch, &total);
    s_p0[tid] = p0;
    __syncthreads();
    return total;
  };
  // request (-1: no entry, and none before a batch is loaded: a call without tokens
  // loads none), page, table entry
  int e_r[PLAN_KB], e_p[PLAN_KB], e_id[PLAN_KB];
#pragma unroll
  for (int j = 0; j < PLAN_KB; ++j) {
    e_r[j] = -1;
    e_p[j] = e_id[j] = 0;
  }
  // entries e0 + PLAN_KB tid .. of the run; counts the unmapped ones
  auto load_batch = [&](int r0, int e0, int total) {
    const int f0 = e0 + PLAN_KB * tid;
    int lo = 0, hi = min(n_req - r0, PLAN_NT) - 1;  // the last request whose first entry is <= f0
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_base[mid] <= f0) lo = mid;
      else hi = mid - 1;
    }
    const int nr = min(n_req - r0, PLAN_NT);
    int tg[PLAN_KB];
#pragma unroll
    for (int j = 0; j < PLAN_KB; ++j) {
      const int f = f0 + j;
      while (lo + 1 < nr && s_base[lo + 1] <= f) ++lo;  // (requests without entries are stepped over)
      const bool in = f < total;
      e_r[j] = in ? r0 + lo : -1;
      e_p[j] = in ? s_p0[lo] + (f - s_base[lo]) : 0;
      const int64_t i = in ? (int64_t)e_r[j] * max_pages + e_p[j] : 0;
      e_id[j] = bt[i];
      tg[j] = tags[i];
    }
    int fresh = 0;
#pragma unroll
    for (int j = 0; j < PLAN_KB; ++j) {
      if (e_r[j] < 0) continue;
      if (e_id[j] < 0) ++fresh;
      else if (tg[j] != TAG_R) err |= MKV_DEVERR_NOT_RECENT;
      else if (e_id[j] >= n_fp8) err |= MKV_DEVERR_RANGE;
    }
    return fresh;
  };
  // the batch's list entries from base_list + e0 on, fresh ids from rank on
  auto write_batch = [&](int base_list, int e0, int rank) {
#pragma unroll
    for (int j = 0; j < PLAN_KB; ++j) {
      if (e_r[j] < 0) continue;
      int id = e_id[j];
      if (id < 0) {
        const int64_t i = (int64_t)e_r[j] * max_pages + e_p[j];
        id = fp8_stack[top - 1 - rank++];
        bt[i] = id;
        tags[i] = TAG_R;
        rc8[id] = 1;  // one request reference
      }
      int32_t* e = list + 4LL * (base_list + e0 + PLAN_KB * tid + j);
      e[0] = e_r[j];
      e[1] = e_p[j];
      e[2] = id;
      e[3] = 0;
    }
  };
  int64_t n_list = 0;
  int fresh = 0, need = 0, rank = 0;
  bool one = false;  // the whole call is one batch, kept in registers
  for (int r0 = 0; r0 < n_req; r0 += PLAN_NT) {
    const int total = load_run(r0);
    one = n_req <= PLAN_NT && total <= PLAN_BATCH;
    for (int e0 = 0; e0 < total; e0 += PLAN_BATCH) fresh += load_batch(r0, e0, total);
    n_list += total;
    if (r0 + PLAN_NT < n_req) __syncthreads();  // the run's arrays are free
  }
  if (err) atomicOr(&s_err, err);
  if (one) {
    rank = block_excl_scan(fresh, scratch, &need);  // its barriers also publish s_err
  } else {
    if (fresh) atomicAdd(&s_need, fresh);
    __syncthreads();
    need = s_need;
  }
  err = s_err;
  if (err == 0 && need > top) err |= MKV_DEVERR_FP8_EXHAUSTED;
  if (err == 0 && n_list > n_fp8) err |= MKV_DEVERR_RANGE;
  if (err) {
    if (tid == 0) {
      atomicOr(&ctrl[CTRL_ERR], err);
      ctrl[CTRL_ABORT] = 1;
      ctrl[CTRL_NLIST] = 0;
    }
    return;
  }
  if (one) {
    write_batch(0, 0, rank);
  } else {
    int base_list = 0, base_fresh = 0;
    for (int r0 = 0; r0 < n_req; r0 += PLAN_NT) {
      __syncthreads();
      const int total = load_run(r0);
      for (int e0 = 0; e0 < total; e0 += PLAN_BATCH) {
        const int c = load_batch(r0, e0, total);
        int tot;
        const int pre = block_excl_scan(c, scratch, &tot);
        write_batch(base_list, e0, base_fresh + pre);
        base_fresh += tot;
      }
      base_list += total;
    }
  }
  if (tid == 0) {
    ctrl[CTRL_FP8_TOP] = top - need;
    ctrl[CTRL_NLIST] = (int)n_list;
    ctrl[CTRL_ABORT] = 0;
  }
}

// x / s correctly rounded, for a fixed divisor whose correctly rounded
// reciprocal y = 1 / s is at hand: a Newton step on the quotient, then Markstein's
// final step (with y correctly rounded and q within an ulp of x / s, q + (x - q s)
// y rounds to the correctly rounded quotient).  Needs the remainders exact: div_fast(s).
// A quotient small enough to lose them is far below every E4M3 code's rounding
// boundary; its sign is x's (a zero quotient included).
__device__ __forceinline__ float div_by(float x, float s, float y) {
  float q = x * y;
  q = __builtin_fmaf(__builtin_fmaf(-q, s, x), y, q);
  q = __builtin_fmaf(__builtin_fmaf(-q, s, x), y, q);
  return __builtin_copysignf(q, x);
}
__device__ __forceinline__ bool div_fast(float s) { return s >= 0x1p-60f && s <= 0x1p60f; }
// four fp32 values -> four E4M3 bytes, as f32_to_e4m3
__device__ __forceinline__ uint32_t pack_e4m3(float a, float b, float c, float d) {
  auto sat = [](float x) { return fminf(fmaxf(x, -448.0f), 448.0f); };
  const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(sat(a), sat(b), 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(sat(c), sat(d), lo, true);
}

// Quantize one tensor (K or V) of one page-head with one wave.  Slots [0, t0)
// already hold codes with the page's scale; the new bf16 values are rows
// row0 + t (t in [t0, t1)) of src, [row][H][D].  The scale only grows: when the
// new amax exceeds 448 * s_old the old codes are re-rounded to the new scale.
// Lane l holds channels 4 (l % (D/4)) .. + 3 of NT consecutive tokens, so it has
// every byte of its K dwords (one token, four channels) and of its V dwords (one
// channel, the four tokens of a group; four consecutive dwords per group, see
// fp8_off): all stores are whole dwords.  A page that already holds tokens
// (t0 > 0) has its old dwords loaded beside the new rows.  The bound is memory:
// 32 K tokens x 4 heads x 4 layers at d = 256 read and write 0.8 GB; storing V
// byte by byte the launch took 367 us, now 160 us (5.0 TB/s).
template <int D, bool kv>
__device__ __forceinline__ void quant_task(uint8_t* reg, float* sc, const uint16_t* src, int64_t row0,
                                           int t0, int t1, int H, int h, int lane) {
  constexpr int CL = D / 16, D4 = D / 4, NT = PAGE * D4 / 64, NG = NT / 4;
  const int cg = lane % D4, tb = (lane / D4) * NT;  // channel group, first token
  const uint16_t* srow = src + (row0 * H + h) * D + 4 * cg;  // token t at srow[t * H * D]
  const int64_t tstride = (int64_t)H * D;
  uint32_t* rw = reinterpret_cast<uint32_t*>(reg + (kv ? PAGE * D : 0));
  // K: dword of token t at t D4 + cg; V: the dwords of token group g at
  // ((r 4 + g) CL + m), r = 4 cg / CL, m = 4 cg % CL .. + 3
  uint4* rv = reinterpret_cast<uint4*>(rw) + (4 * cg / CL) * CL + (4 * cg % CL) / 4;  // group g: + g CL / 4
  const float s_old = t0 > 0 ? sc[kv] : 0.0f;
  uint2 x[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    const int t = tb + k;
    x[k] = make_uint2(0u, 0u);
    if (t >= t0 && t < t1) x[k] = *reinterpret_cast<const uint2*>(srow + t * tstride);
  }
  float amax = 0.0f;
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    amax = fmaxf(amax, fmaxf(fmaxf(fabsf(__uint_as_float(x[k].x << 16)),
                                   fabsf(__uint_as_float(x[k].x & 0xFFFF0000u))),
                             fmaxf(fabsf(__uint_as_float(x[k].y << 16)),
                                   fabsf(__uint_as_float(x[k].y & 0xFFFF0000u)))));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
  float s_new = s_old;
  bool requant = false;
  if (t0 == 0) {
    s_new = amax / 448.0f;
  } else if (!(amax <= 448.0f * s_old)) {
    s_new = amax / 448.0f;
    requant = true;
  }
  // four channels of token tb + k
  auto f4 = [&](int k, int b) {
    const uint32_t w = b < 2 ? x[k].x : x[k].y;
    return __uint_as_float(b & 1 ? w & 0xFFFF0000u : w << 16);
  };
  if (__builtin_amdgcn_readfirstlane(div_fast(s_new) && !requant)) {
    const float y = 1.0f / s_new;
    const bool whole = __builtin_amdgcn_readfirstlane(t0 == 0 && t1 == PAGE);
#pragma unroll
    for (int j = 0; j < NG; ++j) {
      const int ta = tb + 4 * j;  // the group's first token
      float q[4][4];              // [token][channel]
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int b = 0; b < 4; ++b) q[u][b] = div_by(f4(4 * j + u, b), s_new, y);
      // the group's dwords: K dword u = token ta + u, V dword b = channel 4 cg + b
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[i] = kv ? pack_e4m3(q[0][i], q[1][i], q[2][i], q[3][i]) : pack_e4m3(q[i][0], q[i][1], q[i][2], q[i][3]);
      if (kv) {
        uint4* dst = rv + (ta / 4) * (CL / 4);
        if (!whole) {  // bytes of tokens [t0, t1) are new; others old, or zero in a fresh page
          uint32_t m = 0;
#pragma unroll
          for (int u = 0; u < 4; ++u) m |= ta + u >= t0 && ta + u < t1 ? 0xFFu << (8 * u) : 0u;
          const uint4 o = t0 > 0 ? *dst : make_uint4(0u, 0u, 0u, 0u);
          w[0] = (w[0] & m) | (o.x & ~m);
          w[1] = (w[1] & m) | (o.y & ~m);
          w[2] = (w[2] & m) | (o.z & ~m);
          w[3] = (w[3] & m) | (o.w & ~m);
        }
        *dst = make_uint4(w[0], w[1], w[2], w[3]);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = ta + u;
          const bool nw = whole || (t >= t0 && t < t1);
          if (nw || t0 == 0) rw[t * D4 + cg] = nw ? w[u] : 0u;
        }
      }
    }
  } else {
    // old codes to re-round, or a scale without a fast division: rare, so one
    // body for the groups; group j is in x[0 .. 3], the later ones move down after it
#pragma unroll 1
    for (int j = 0; j < NG; ++j) {
      const int ta = tb + 4 * j;
      // the group's dwords: K dword u = token ta + u, V dword b = channel 4 cg + b
      uint32_t w[4] = {0u, 0u, 0u, 0u};
      if (t0 > 0) {  // old codes, re-rounded when the scale grew; none in a fresh page
        if (kv) {
          const uint4 o = rv[(ta / 4) * (CL / 4)];
          w[0] = o.x; w[1] = o.y; w[2] = o.z; w[3] = o.w;
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) w[u] = rw[(ta + u) * D4 + cg];
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t o = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int u = kv ? b : i, t = ta + u;  // token of byte b of dword i
          const float xv = kv ? f4(b, i) : f4(i, b);
          const uint32_t code = (w[i] >> (8 * b)) & 0xFFu;
          const bool nw = t >= t0 && t < t1, re = requant && t < t0;
          const uint32_t c = f32_to_e4m3((nw ? xv : e4m3_to_f32(code) * s_old) / s_new);
          o |= (re || (nw && s_new > 0.0f) ? c : nw ? 0u : code) << (8 * b);
        }
        w[i] = o;
      }
      if (kv) {
        rv[(ta / 4) * (CL / 4)] = make_uint4(w[0], w[1], w[2], w[3]);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) rw[(ta + u) * D4 + cg] = w[u];
      }
#pragma unroll
      for (int k = 0; k + 4 < NT; ++k) x[k] = x[k + 4];
    }
  }
  if (lane == 0) sc[kv] = s_new;
}

// One quantisation task = (listed page, layer, head, K or V); one wave each.
template <int D>
__device__ __forceinline__ void run_quant_task(const PoolView& P, int64_t task, int layer_sel,
                                               int n_lcall, const int32_t* sb, const int32_t* cu,
                                               int n_new_total, const uint16_t* k,
                                               const uint16_t* v, const int32_t* lst, int lane) {
  const int H = P.n_kv_heads;
  const int kv = (int)(task & 1);
  const int64_t item = task >> 1;
  const int e = (int)(item / (n_lcall * H));
  const int lh = (int)(item % (n_lcall * H));
  const int li = lh / H, h = lh % H;
  const int r = lst[4 * e], p = lst[4 * e + 1], id = lst[4 * e + 2];
  const int layer = layer_sel < 0 ? li : layer_sel;
  const int s0 = sb[r], n = cu[r + 1] - cu[r];
  const int t0 = max(0, s0 - p * PAGE), t1 = min(PAGE, s0 + n - p * PAGE);
  const int64_t ph = ((int64_t)layer * P.n_fp8 + id) * H + h;
  const int64_t row0 = (int64_t)cu[r] + p * PAGE - s0;  // input row of slot t is row0 + t
  const uint16_t* src = (kv ? v : k) + (int64_t)li * n_new_total * H * D;
  uint8_t* reg = P.fp8 + ph * fp8_region_bytes(D);
  float* sc = P.fp8_scales + ph * 2;
  if (kv)
    quant_task<D, true>(reg, sc, src, row0, t0, t1, H, h, lane);
  else
    quant_task<D, false>(reg, sc, src, row0, t0, t1, H, h, lane);
}

// Quantize every listed page-head of every requested layer (grid-stride over
// tasks, one wave per task).
template <int D>
__global__ __launch_bounds__(256) void append_quant_kernel(PoolView P, int layer_sel, int n_lcall,
                                                           const int32_t* sb, const int32_t* cu,
                                                           int n_new_total, const uint16_t* k,
                                                           const uint16_t* v) {
  if (P.ctrl[CTRL_ABORT]) return;
  const int64_t n_tasks = (int64_t)P.ctrl[CTRL_NLIST] * n_lcall * P.n_kv_heads * 2;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int64_t t = (int64_t)blockIdx.x * 4 + wid; t < n_tasks; t += (int64_t)gridDim.x * 4)
    run_quant_task<D>(P, t, layer_sel, n_lcall, sb, cu, n_new_total, k, v, P.list, lane);
}

// Small appends (decode steps: a few tokens per request): one wave per task
// (touched page, layer, head, K or V) and no barrier.  Every wave reads the
// whole call (rows and start positions, block-table entries and tags of the
// touched pages, the head of the FP8 free list) and so reaches the same
// validation and the same fresh-page ids; the wave that arrives last on a
// counter in the control block (by then every other wave has finished its
// reads) records the fresh pages in the block table, pops them off the free
// list and resets the counter.  Three dependent memory round trips: (1) rows,
// starts and the free-list top; (2) table entries, free-list head and the
// task's new rows; (3) the page-head's codes and scale when it already holds
// tokens.  A task assembles the page-head's code block in LDS (old codes,
// re-rounded through a 256-entry table when the scale grows; new codes; zeros
// past the new tokens of a fresh page) and stores it with whole-dword writes.
// Same validation, allocation order and arithmetic as the two-kernel path.
constexpr int STEP_APPEND_MAX_TOKENS = 256;  // also bounds the touched pages
constexpr int STEP_APPEND_MAX_REQ = 256;
constexpr int STEP_APPEND_MAX_WAVES = 4096;


template <int D>
__global__ __launch_bounds__(64) void append_step_kernel(PoolView P, int layer_sel, int n_lcall,
                                                         int n_req, int32_t* bt, uint8_t* tags,
                                                         int max_pages, const int32_t* sb,
                                                         const int32_t* cu, int n_new_total,
                                                         const uint16_t* k, const uint16_t* v) {
  constexpr int RQ = STEP_APPEND_MAX_REQ / 64, EQ = STEP_APPEND_MAX_TOKENS / 64;
  __shared__ int s_base[STEP_APPEND_MAX_REQ + 1];  // first list entry of request r
  __shared__ int s_cu[STEP_APPEND_MAX_REQ], s_n[STEP_APPEND_MAX_REQ], s_s0[STEP_APPEND_MAX_REQ];
  __shared__ __align__(16) uint32_t s_img[PAGE * D / 4];
  __shared__ uint8_t s_lut[256];
  const int lane = threadIdx.x;
  const int H = P.n_kv_heads;
  // ---- round trip 1: rows, starts, free-list top
  const int top = P.ctrl[CTRL_FP8_TOP];
  int bad = (cu[0] != 0 || cu[n_req] != n_new_total) ? (int)MKV_DEVERR_RANGE : 0;
  int run = 0;  // list entries of the requests before this group of 64
#pragma unroll
  for (int i = 0; i < RQ; ++i) {
    const int r = lane + 64 * i;
    int touch = 0;
    if (r < n_req) {
      const int c_r = cu[r], n = cu[r + 1] - c_r, s0 = sb[r];
      // rows outside the input stay unread: inputs are loaded before the call
      // as a whole is known to be valid
      if (n < 0 || s0 < 0 || c_r < 0 || c_r + n > n_new_total) {
        bad |= MKV_DEVERR_RANGE;
      } else if (n > 0) {
        const int p0 = s0 / PAGE, p1 = (s0 + n - 1) / PAGE;
        if (p1 >= max_pages) bad |= MKV_DEVERR_RANGE;
        else touch = p1 - p0 + 1;
      }
      s_cu[r] = c_r;
      s_n[r] = n;
      s_s0[r] = s0;
    }
    const int incl = wave_incl_scan(touch, lane);
    if (r < n_req) s_base[r] = run + incl - touch;
    run += __shfl(incl, 63, 64);
  }
  const int n_ent = run;
  if (lane == 0) s_base[n_req] = n_ent;
  __builtin_amdgcn_wave_barrier();
  // list entry e -> (request, page): the last request whose first entry is <= e
  auto locate = [&](int e, int& r, int& p) {
    int lo = 0, hi = n_req - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_base[mid] <= e) lo = mid;
      else hi = mid - 1;
    }
    r = lo;
    p = s_s0[lo] / PAGE + (e - s_base[lo]);
  };
  // ---- round trip 2: table entries of the list, the free-list head, the
  // task's new rows
  int ent_bt[EQ], ent_tag[EQ];
#pragma unroll
  for (int j = 0; j < EQ; ++j) {
    const int e = lane + 64 * j;
    ent_bt[j] = 0;
    ent_tag[j] = TAG_R;
    if (e < n_ent) {
      int r, p;
      locate(e, r, p);
      const int64_t i = (int64_t)r * max_pages + p;
      ent_bt[j] = bt[i];
      ent_tag[j] = tags[i];
    }
  }
  const int stk = lane < top ? P.fp8_stack[top - 1 - lane] : -1;  // ids handed out first
  const int64_t n_tasks = (int64_t)n_ent * n_lcall * H * 2;
  const int64_t task = blockIdx.x;
  SmallTask<D> T;
  int e_t = 0;
  if (task < n_tasks) {
    T.kv = (int)(task & 1);
    const int64_t item = task >> 1;
    e_t = (int)(item / (n_lcall * H));
    const int lh = (int)(item % (n_lcall * H));
    T.li = lh / H;
    T.h = lh % H;
    T.layer = layer_sel < 0 ? T.li : layer_sel;
    int r, p;
    locate(e_t, r, p);
    T.r = __builtin_amdgcn_readfirstlane(r);
    T.p = __builtin_amdgcn_readfirstlane(p);
    const int c_r = __builtin_amdgcn_readfirstlane(s_cu[T.r]);
    const int s0 = __builtin_amdgcn_readfirstlane(s_s0[T.r]);
    const int n = __builtin_amdgcn_readfirstlane(s_n[T.r]);
    T.row0 = c_r + T.p * PAGE - s0;  // input row of slot t is row0 + t
    T.t0 = max(0, s0 - T.p * PAGE);
    T.t1 = min(PAGE, s0 + n - T.p * PAGE);
    // a listed page belongs to a request whose rows passed the range checks
    small_task_load_x<D>(T, H, n_new_total, k, v, lane);
  }
  // ---- validation and fresh-page ranks (identical in every wave)
  int fresh[EQ], rank[EQ], n_fresh = 0;
#pragma unroll
  for (int j = 0; j < EQ; ++j) {
    const int e = lane + 64 * j;
    fresh[j] = (e < n_ent && ent_bt[j] < 0) ? 1 : 0;
    if (e < n_ent && !fresh[j]) {
      if (ent_tag[j] != TAG_R) bad |= MKV_DEVERR_NOT_RECENT;
      else if (ent_bt[j] >= P.n_fp8) bad |= MKV_DEVERR_RANGE;
    }
    const int incl = wave_incl_scan(fresh[j], lane);
    rank[j] = n_fresh + incl - fresh[j];
    n_fresh += __shfl(incl, 63, 64);
  }
  if (n_fresh > top) bad |= MKV_DEVERR_FP8_EXHAUSTED;
  bad = wave_or(bad);
  // id of each entry: its table entry, or the free-list element of its rank
  int ent_id[EQ];
#pragma unroll
  for (int j = 0; j < EQ; ++j) {
    ent_id[j] = ent_bt[j];
    const int sl = __shfl(stk, rank[j] & 63, 64);  // by every lane: one that sat out could not be read
    if (fresh[j] && bad == 0) ent_id[j] = rank[j] < 64 ? sl : P.fp8_stack[top - 1 - rank[j]];
  }
  if (bad == 0 && task < n_tasks) {
    // ---- round trip 3 and the task
    int idv = 0;
#pragma unroll
    for (int j = 0; j < EQ; ++j) idv = (e_t >> 6) == j ? ent_id[j] : idv;
    const int id = __builtin_amdgcn_readfirstlane(__shfl(idv, e_t & 63, 64));
    small_task_load_old<D>(T, P, id, lane);
    small_task_run<D>(T, P, id, s_img, s_lut, lane);
  }
  // ---- nothing to publish (no fresh page; every wave reached the same
  // verdict): the first wave reports an error, no wave waits for the others
  if (n_fresh == 0 || bad) {
    if (bad && blockIdx.x == 0 && lane == 0) atomicOr(&P.ctrl[CTRL_ERR], bad);
    return;
  }
  // ---- arrive; the last wave records the fresh pages.  Only the order of
  // every wave's table reads before the last wave's table writes matters:
  // a wave counts itself once all its loads have returned (no device-scope
  // fence, which would write back this die's L2).  The page codes and the
  // table are published to later kernels by the end of this kernel.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  int prev = 0;
  if (lane == 0) prev = atomicAdd(&P.ctrl[CTRL_APPEND_ARRIVE], 1);
  prev = __shfl(prev, 0, 64);
  if (prev != (int)gridDim.x - 1) return;
#pragma unroll
  for (int j = 0; j < EQ; ++j) {
    const int e = lane + 64 * j;
    if (e < n_ent && fresh[j]) {
      int r, p;
      locate(e, r, p);
      const int64_t i = (int64_t)r * max_pages + p;
      bt[i] = ent_id[j];
      tags[i] = TAG_R;
      P.rc8[ent_id[j]] = 1;
    }
  }
  if (lane == 0) P.ctrl[CTRL_FP8_TOP] = top - n_fresh;
  if (lane == 0) P.ctrl[CTRL_APPEND_ARRIVE] = 0;
}

// ===========================================================================
// Migrate (Retier to TQ3)
// ===========================================================================

// Plan of a migration, in two launches over nb <= MIG_BLOCKS workgroups; each
// workgroup owns a range of whole batches of the table taken as one run of
// (request, page) entries, MIG_KB consecutive entries per thread with every
// load of a batch in flight together.  The count launch validates its range
// (lengths, candidate ids) and counts the migrating pages; the list launch
// sums the counts of the ranges before its own, checks the whole call
// (errors, free-list room) so that a failing call changes nothing, ranks its
// migrating pages in (request, page) order with one block scan per batch,
// retags Anchors and writes the work list with the TQ3 ids popped in that
// order.  The table entries, Stale tags and FP8 releases are published by the
// publish kernel after the encode kernel has built the TQ3 pages (Alg. 1,
// copy before publish).
constexpr int MIG_KB = 8;
constexpr int MIG_NT = 1024;
constexpr int64_t MIG_BATCH = (int64_t)MIG_NT * MIG_KB;
struct MigBatch {
  uint8_t tg[MIG_KB], an[MIG_KB];
  int32_t id[MIG_KB], sl[MIG_KB], rq[MIG_KB], pg[MIG_KB], rc[MIG_KB];
};
// references of the entries' pages (shared pages are left alone by Retier and
// Promote); 0 where the tag or id names no page
struct RcView {
  const int32_t* rc8;
  const int32_t* rc3;
  int n_fp8, n_tq3;
};
__device__ __forceinline__ void mig_load_rc(MigBatch& m, const RcView& v) {
#pragma unroll
  for (int j = 0; j < MIG_KB; ++j) {
    const bool f8 = m.tg[j] == TAG_R || m.tg[j] == TAG_A, f3 = m.tg[j] == TAG_S;
    const int id = m.id[j];
    const bool ok = m.rq[j] >= 0 && id >= 0 && ((f8 && id < v.n_fp8) || (f3 && id < v.n_tq3));
    m.rc[j] = ok ? (f8 ? v.rc8 : v.rc3)[id] : 0;
  }
}
// entries f0 .. f0 + MIG_KB - 1: (request, page) stepped from one division
__device__ __forceinline__ void mig_load(MigBatch& m, int64_t f0, int64_t N, int max_pages,
                                         const int32_t* bt, const uint8_t* tags,
                                         const uint8_t* anchor, const int32_t* seq_lens) {
  int r = (int)(f0 / max_pages), p = (int)(f0 - (int64_t)r * max_pages);
#pragma unroll
  for (int j = 0; j < MIG_KB; ++j) {
    const bool in = f0 + j < N;
    const int64_t f = in ? f0 + j : 0;
    m.rq[j] = in ? r : -1;
    m.pg[j] = p;
    m.tg[j] = tags[f];
    m.an[j] = anchor ? anchor[f] : 0;
    m.id[j] = bt[f];
    m.sl[j] = seq_lens[in ? r : 0];
    if (++p == max_pages) { p = 0; ++r; }
  }
}
// The table as one batch of N <= MIG_BATCH entries, entry j MIG_NT + tid in slot j
// of thread tid: neighbouring threads load neighbouring entries (a single
// workgroup is bound by its CU's address unit, and slots past the table cost
// nothing).  Retier's list of one request's 128 and 1,030 pages takes 3.4 and 5.1 us,
// 5.2 and 9.8 with MIG_KB consecutive entries per thread; Promote's of 8 x 376 pages
// 8.4 us, 15.7.
__device__ __forceinline__ void mig_load_striped(MigBatch& m, int N, int max_pages, const int32_t* bt,
                                                 const uint8_t* tags, const uint8_t* anchor,
                                                 const int32_t* seq_lens) {
#pragma unroll
  for (int j = 0; j < MIG_KB; ++j) {
    m.rq[j] = -1;
    m.pg[j] = m.sl[j] = m.id[j] = 0;
    m.tg[j] = TAG_NONE;
    m.an[j] = 0;
    if (j * MIG_NT < N) {  // workgroup-uniform
      const bool in = j * MIG_NT + (int)threadIdx.x < N;
      const uint32_t f = in ? j * MIG_NT + threadIdx.x : 0;
      const uint32_t r = f / (uint32_t)max_pages;
      m.rq[j] = in ? (int)r : -1;
      m.pg[j] = (int)(f - r * (uint32_t)max_pages);
      m.tg[j] = tags[f];
      m.an[j] = anchor ? anchor[f] : 0;
      m.id[j] = bt[f];
      m.sl[j] = seq_lens[r];
    }
  }
}
// Exclusive sums, in entry order, of the counts that the 16 waves of a workgroup
// hold for their 64 entries of each slot: base[j] for this wave's slot j; returns
// the total.  s_cnt: 16 KB + 1 words; two barriers, whatever KB is.
template <int KB>
__device__ __forceinline__ int striped_bases(const int (&cnt)[KB], int (&base)[KB], int* s_cnt) {
  static_assert(16 * KB % 64 == 0, "a wave sums the counts");
  constexpr int PER = 16 * KB / 64;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < KB; ++j)
    if (lane == 0) s_cnt[16 * j + wid] = cnt[j];
  __syncthreads();
  if (wid == 0) {
    int v[PER], x = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) x += v[i] = s_cnt[PER * lane + i];
    const int incl = wave_incl_scan(x, lane);
    int e = incl - x;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      s_cnt[PER * lane + i] = e;
      e += v[i];
    }
    if (lane == 63) s_cnt[16 * KB] = incl;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < KB; ++j) base[j] = s_cnt[16 * j + wid];
  return s_cnt[16 * KB];
}
// The reference counts a migration plan needs: only a Recent page that has
// left the window and is not an anchor can migrate, and only then does its
// count decide (a shared page stays FP8); every other entry skips the gather.
__device__ __forceinline__ void mig_load_rc_candidates(MigBatch& m, const RcView& v, int W) {
#pragma unroll
  for (int j = 0; j < MIG_KB; ++j) {
    const int p = m.pg[j], S = m.sl[j], id = m.id[j];
    const bool cand = m.rq[j] >= 0 && m.tg[j] == TAG_R && !m.an[j] && p < (S + PAGE - 1) / PAGE &&
                      (p + 1) * PAGE <= S - W && id >= 0 && id < v.n_fp8;
    m.rc[j] = cand ? v.rc8[id] : 0;
  }
}
// 1: migrating page, 2: Anchor to retag, 0: neither
__device__ __forceinline__ int mig_kind(const MigBatch& m, int j, int W) {
  if (m.rq[j] < 0) return 0;
  const int p = m.pg[j], S = m.sl[j];
  if (m.tg[j] != TAG_R || p >= (S + PAGE - 1) / PAGE || (p + 1) * PAGE > S - W) return 0;
  if (m.an[j]) return 2;
  return m.rc[j] == 1 ? 1 : 0;  // a shared (sealed) page stays until it is private
}

// Count and validate the entries [e0, e1) (the whole workgroup); workgroup 0
// also checks every request's length.  Returns through s_cnt / s_err.
__device__ __forceinline__ void mig_count_range(int b, int n_req, const int32_t* bt,
                                                const uint8_t* tags, int max_pages,
                                                const uint8_t* anchor, const int32_t* seq_lens,
                                                int W, int64_t e0, int64_t e1, int n_fp8,
                                                int* s_cnt, int* s_err, const RcView& rv) {
  const int tid = threadIdx.x;
  int err = 0, cnt = 0;
  if (b == 0) {
    for (int r = tid; r < n_req; r += MIG_NT) {
      const int S = seq_lens[r];
      if (S < 0 || (S + PAGE - 1) / PAGE > max_pages) err |= MKV_DEVERR_RANGE;
    }
  }
  for (int64_t b0 = e0; b0 < e1; b0 += MIG_BATCH) {
    MigBatch m;
    mig_load(m, b0 + (int64_t)tid * MIG_KB, e1, max_pages, bt, tags, anchor, seq_lens);
    mig_load_rc_candidates(m, rv, W);
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      const int p = m.pg[j], S = m.sl[j];
      const bool old_r = m.rq[j] >= 0 && m.tg[j] == TAG_R && p < (S + PAGE - 1) / PAGE &&
                         (p + 1) * PAGE <= S - W && !m.an[j];
      if (old_r && (m.id[j] < 0 || m.id[j] >= n_fp8)) err |= MKV_DEVERR_RANGE;
      if (mig_kind(m, j, W) == 1) cnt++;
    }
  }
  if (cnt) atomicAdd(s_cnt, cnt);
  if (err) atomicOr(s_err, err);
}

__global__ __launch_bounds__(MIG_NT) void migrate_count_kernel(
    int n_req, const int32_t* bt, const uint8_t* tags, int max_pages, const uint8_t* anchor,
    const int32_t* seq_lens, int W, int32_t* ctrl, int32_t* mig, int64_t per_blk, int n_fp8,
    RcView rv) {
  __shared__ int s_err, s_cnt;
  const int tid = threadIdx.x, b = blockIdx.x;
  if (tid == 0) { s_err = 0; s_cnt = 0; }
  if (b == 0 && tid == 0) mig[2 * MIG_BLOCKS] = ctrl[CTRL_TQ3_TOP];  // read before the list launch moves it
  const int64_t N = (int64_t)n_req * max_pages;
  const int64_t e0 = (int64_t)b * per_blk, e1 = min(N, e0 + per_blk);
  __syncthreads();
  mig_count_range(b, n_req, bt, tags, max_pages, anchor, seq_lens, W, e0, e1, n_fp8, &s_cnt, &s_err,
                  rv);
  __syncthreads();
  if (tid == 0) {
    mig[b] = s_cnt;
    mig[MIG_BLOCKS + b] = s_err;
  }
}

// ONE: a single workgroup owns the whole table (at most one batch): it loads
// the batch once, counts and validates it, and lists it after one scan (one
// launch instead of two, one pass over the table instead of two).
template <bool ONE>
__global__ __launch_bounds__(MIG_NT) void migrate_list_kernel(
    int n_req, const int32_t* bt, uint8_t* tags, int max_pages, const uint8_t* anchor,
    const int32_t* seq_lens, int W, int32_t* ctrl, const int32_t* tq3_stack, int32_t* list,
    const int32_t* mig, int64_t per_blk, int nb, int n_fp8, RcView rv) {
  __shared__ int scratch[32];
  __shared__ int s_cnt[16 * MIG_KB + 1];
  __shared__ int s_err, s_tot, s_pre;
  const int tid = threadIdx.x, b = blockIdx.x;
  if (tid == 0) { s_err = 0; s_tot = 0; s_pre = 0; }
  __syncthreads();
  const int top3 = ONE ? ctrl[CTRL_TQ3_TOP] : mig[2 * MIG_BLOCKS];
  if constexpr (ONE) {
    MigBatch m;
    mig_load_striped(m, n_req * max_pages, max_pages, bt, tags, anchor, seq_lens);
    int err = 0, k[MIG_KB], cnt[MIG_KB], base[MIG_KB];
    for (int r = tid; r < n_req; r += MIG_NT) {
      const int S = seq_lens[r];
      if (S < 0 || (S + PAGE - 1) / PAGE > max_pages) err |= MKV_DEVERR_RANGE;
    }
    mig_load_rc_candidates(m, rv, W);
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      const int p = m.pg[j], S = m.sl[j];
      const bool old_r = m.rq[j] >= 0 && m.tg[j] == TAG_R && p < (S + PAGE - 1) / PAGE &&
                         (p + 1) * PAGE <= S - W && !m.an[j];
      if (old_r && (m.id[j] < 0 || m.id[j] >= n_fp8)) err |= MKV_DEVERR_RANGE;
      k[j] = mig_kind(m, j, W);
      cnt[j] = __popcll(__ballot(k[j] == 1));
    }
    if (err) atomicOr(&s_err, err);
    const int total = striped_bases<MIG_KB>(cnt, base, s_cnt);  // its barriers also publish s_err
    err = s_err;
    if (err == 0 && total > top3) err |= MKV_DEVERR_TQ3_EXHAUSTED;
    if (err == 0 && total > n_fp8) err |= MKV_DEVERR_RANGE;
    if (err) {
      if (tid == 0) {
        atomicOr(&ctrl[CTRL_ERR], err);
        ctrl[CTRL_ABORT] = 1;
        ctrl[CTRL_NLIST] = 0;
      }
      return;
    }
    const uint64_t below = (1ull << (tid & 63)) - 1ull;
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      const int e = base[j] + __popcll(__ballot(k[j] == 1) & below);
      if (k[j] == 2) tags[j * MIG_NT + tid] = TAG_A;  // Anchor: tag only, stays FP8
      if (k[j] == 1) {
        int32_t* le = list + 4LL * e;
        le[0] = m.rq[j];
        le[1] = m.pg[j];
        le[2] = m.id[j];
        le[3] = tq3_stack[top3 - 1 - e];
      }
    }
    if (tid == 0) {
      ctrl[CTRL_TQ3_TOP] = top3 - total;
      ctrl[CTRL_NLIST] = total;
      ctrl[CTRL_ABORT] = 0;
    }
    return;
  } else if (tid < nb) {
    const int c = mig[tid], e = mig[MIG_BLOCKS + tid];
    if (c) atomicAdd(&s_tot, c);
    if (c && tid < b) atomicAdd(&s_pre, c);
    if (e) atomicOr(&s_err, e);
  }
  __syncthreads();
  int err = s_err;
  const int total = s_tot;
  if (err == 0 && total > top3) err |= MKV_DEVERR_TQ3_EXHAUSTED;
  if (err == 0 && total > n_fp8) err |= MKV_DEVERR_RANGE;
  if (err) {
    if (b == 0 && tid == 0) {
      atomicOr(&ctrl[CTRL_ERR], err);
      ctrl[CTRL_ABORT] = 1;
      ctrl[CTRL_NLIST] = 0;
    }
    return;
  }
  const int64_t N = (int64_t)n_req * max_pages;
  const int64_t e0 = (int64_t)b * per_blk, e1 = min(N, e0 + per_blk);
  int base = s_pre;
  for (int64_t b0 = e0; b0 < e1; b0 += MIG_BATCH) {
    MigBatch m;
    mig_load(m, b0 + (int64_t)tid * MIG_KB, e1, max_pages, bt, tags, anchor, seq_lens);
    mig_load_rc_candidates(m, rv, W);
    int k[MIG_KB], c = 0;
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      k[j] = mig_kind(m, j, W);
      c += k[j] == 1;
    }
    int tot;
    int e = base + block_excl_scan(c, scratch, &tot);
    const int64_t f0 = b0 + (int64_t)tid * MIG_KB;
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      if (k[j] == 2) tags[f0 + j] = TAG_A;  // Anchor: tag only, stays FP8
      if (k[j] == 1) {
        int32_t* le = list + 4LL * e;
        le[0] = m.rq[j];
        le[1] = m.pg[j];
        le[2] = m.id[j];
        le[3] = tq3_stack[top3 - 1 - e];
        e++;
      }
    }
    base += tot;
  }
  if (b == 0 && tid == 0) {
    ctrl[CTRL_TQ3_TOP] = top3 - total;
    ctrl[CTRL_NLIST] = total;
    ctrl[CTRL_ABORT] = 0;
  }
}

// A chunk's dwords from its quads (the inverse of quad_sel, a whole chunk at once).
template <int NDW>
__device__ __forceinline__ void pack_quads(uint32_t* dw, const uint32_t* quad) {
#pragma unroll
  for (int j = 0; j < NDW; ++j) dw[j] = quad[2 * j] | quad[2 * j + 1] << 3;
#pragma unroll
  for (int p = 0; p < NDW / 3; ++p) {
    const uint32_t a = quad[2 * NDW + 2 * p], b = quad[2 * NDW + 2 * p + 1];
    dw[3 * p] |= (a & 0x03030303u) << 6;
    dw[3 * p + 1] |= (a & 0x04040404u) << 4 | (b & 0x01010101u) << 7;
    dw[3 * p + 2] |= (b & 0x06060606u) << 5;
  }
}
// NDW dwords to a chunk: 8-byte stores where the chunk size keeps them aligned
template <int NDW>
__device__ __forceinline__ void store_chunk(uint32_t* out, const uint32_t* dw) {
  if constexpr (NDW % 2 == 0) {
#pragma unroll
    for (int j = 0; j < NDW / 2; ++j) reinterpret_cast<uint2*>(out)[j] = make_uint2(dw[2 * j], dw[2 * j + 1]);
  } else {
#pragma unroll
    for (int j = 0; j < NDW; ++j) out[j] = dw[j];
  }
}
// dwords per row of the value quads in LDS (the chunk's quads, padded: 16-byte rows off one bank)
__host__ __device__ constexpr int enc_row(int d) { return d / 16 + 4; }

// Encode of one FP8 page-head into its TQ3 region by two independent waves, one
// for the keys and one for the values; no barrier, no LDS between them.
//
// Keys (enc_keys): lane 4 t + g owns channels D/4 g .. of token t, which is one
// K chunk of the region.  X = sigma * e4m3 * 2^9 (integers; kept doubled, X2 =
// 2 X, by the conversion's scale), the Sylvester Walsh-Hadamard transform in int32
// (exact): strides below D/4 inside the lane, the two others across the four lanes
// of a token.  The code of a rotated coordinate y is the codebook level nearest
// to z = y / sqrt(n2) (levels +-{0.25, 0.75, 1.375, 2.25}), ties to the lower level: the boundaries are 0 and
// +-{8, 17, 29} / 16, a positive y passes boundary b when 16 y > b sqrt(n2)
// strictly, y <= 0 when 16 |y| >= b sqrt(n2).  As y is an integer that is a
// comparison with f = floor(b sqrt(n2) / 16), found once per token and checked
// in 64-bit integers: with A = 2 |y| + (y <= 0) both signs read A >= 2 f + 2, or
// A >= 2 f + 1 where (16 f)^2 = b^2 n2 exactly.
template <int D>
__device__ __forceinline__ void enc_keys(const uint32_t* sgn, const uint8_t* f8, float sK, uint8_t* reg,
                                         int lane) {
  constexpr int QK = D / 4, NDW = 3 * D / 128, CB = 3 * D / 32;
  const int t = lane >> 2, g = lane & 3;
  uint4 raw[QK / 16];
#pragma unroll
  for (int i = 0; i < QK / 16; ++i) raw[i] = reinterpret_cast<const uint4*>(f8 + t * D + QK * g)[i];
  int y[QK];
  double nn = 0.0;  // sum of X2^2 (integers below 2^53: exact)
#pragma unroll
  for (int i = 0; i < QK / 4; ++i) {
    const uint4& r = raw[i / 4];
    const uint32_t w = (i % 4 == 0 ? r.x : i % 4 == 1 ? r.y : i % 4 == 2 ? r.z : r.w) ^ sgn[i];
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w, 1024.0f, false);
    const f2 hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w, 1024.0f, true);
    const float f[4] = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      nn = __builtin_fma((double)f[b], (double)f[b], nn);
      y[4 * i + b] = (int)f[b];
    }
  }
  auto sum4 = [](double v) {  // over the token's four lanes
    auto step = [](double x, auto ctl) {
      const uint64_t u = __builtin_bit_cast(uint64_t, x);
      constexpr int C = decltype(ctl)::value;
      const uint32_t a = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, C, 0xF, 0xF, false);
      const uint32_t b = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), C, 0xF, 0xF, false);
      return x + __builtin_bit_cast(double, (uint64_t)b << 32 | a);
    };
    v = step(v, std::integral_constant<int, 0xB1>{});
    return step(v, std::integral_constant<int, 0x4E>{});
  };
  const int64_t n2 = (int64_t)sum4(nn) >> 2;  // sum of X^2
  // With lane g's values offset by c = 1, 0, 0, -1 (an impulse at channel 0 of
  // the lane is that offset in all its outputs) those steps leave the lanes off
  // by beta = 0, 0, 1, -1 (see below), which the decision takes into account.
  const int beta = g == 2 ? 1 : g == 3 ? -1 : 0;
  y[0] += g == 0 ? 1 : g == 3 ? -1 : 0;
#pragma unroll
  for (int s = 1; s < QK; s <<= 1)
#pragma unroll
    for (int i = 0; i < QK; ++i)
      if (!(i & s)) {
        const int a = y[i], b = y[i + s];
        y[i] = a + b;
        y[i + s] = a - b;
      }
  // strides D/4 and D/2: lanes g ^ 1 and g ^ 2; the upper lane holds a - b, taken
  // as a + ~b (one instruction less than a - b), which is one too low
  const int m1 = (g & 1) ? -1 : 0, m2 = (g & 2) ? -1 : 0;
#pragma unroll
  for (int i = 0; i < QK; ++i) {
    y[i] = __builtin_amdgcn_mov_dpp(y[i], 0xB1, 0xF, 0xF, false) + (y[i] ^ m1);
    y[i] = __builtin_amdgcn_mov_dpp(y[i], 0x4E, 0xF, 0xF, false) + (y[i] ^ m2);
  }
  // with the lane's offset, A + beta = max(y2, 1 + 2 beta - y2) for the offset y2
  int th[3];  // A + beta >= th[k]: past boundary k
  {
    const int bnd[3] = {8, 17, 29};
    const double sq = sqrt((double)n2);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int64_t rhs = (int64_t)(bnd[k] * bnd[k]) * n2;
      int64_t f = (int64_t)(sq * (bnd[k] * 0.0625));
      if (256 * f * f > rhs) --f;
      if (256 * (f + 1) * (f + 1) <= rhs) ++f;
      th[k] = (int)(2 * f + 2) - (256 * f * f == rhs ? 1 : 0) + beta;
      if (n2 == 0) th[k] = 0x7FFFFFFF;  // a zero key: every code 3
    }
  }
  const int a0 = 1 + 2 * beta;
  const uint32_t flip = beta ? 0x07070707u : 0u;  // an odd offset turns A's parity round
  // codes, four to a word (quad q: channels 4 q .. of the chunk), and sum of 64 level^2
  uint32_t quad[QK / 4], ms = 0, mr = 0;
#pragma unroll
  for (int q = 0; q < QK / 4; ++q) {
    uint32_t c[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int y2 = y[4 * q + b];
      const int A = max(y2, a0 - y2);  // 2 |y| + (y <= 0) + beta
      const bool c1 = A >= th[1];
      const bool c2 = A >= (c1 ? th[2] : th[0]);
      const int cnt = (c1 ? 6 : 4) + (c2 ? 1 : 0);  // 4 + boundaries passed
      c[b] = (uint32_t)(cnt ^ -(A & 1));  // low three bits: 4 + n, or 3 - n where y <= 0
    }
    const uint32_t p01 = __builtin_amdgcn_perm(c[1], c[0], 0x0C0C0400u);
    const uint32_t p23 = __builtin_amdgcn_perm(c[3], c[2], 0x04000C0Cu);
    quad[q] = ((p01 | p23) & 0x07070707u) ^ flip;
    // 64 level^2 = 324, 121, 36, 4, 4, 36, 121, 324 = 4 * {81, 30, 9, 1, ...} + {0, 1, 0, 0, ...}
    ms = __builtin_amdgcn_sad_u8(__builtin_amdgcn_perm(0x511E0901u, 0x01091E51u, quad[q]), 0u, ms);
    mr = __builtin_amdgcn_sad_u8(__builtin_amdgcn_perm(0x00010000u, 0x00000100u, quad[q]), 0u, mr);
  }
  int M = (int)(4 * ms + mr);
  M += __builtin_amdgcn_mov_dpp(M, 0xB1, 0xF, 0xF, false);
  M += __builtin_amdgcn_mov_dpp(M, 0x4E, 0xF, 0xF, false);
  uint32_t dw[NDW];
  pack_quads<NDW>(dw, quad);
  uint32_t* out = reinterpret_cast<uint32_t*>(reg + (g * 16 + t) * CB);
  store_chunk<NDW>(out, dw);
  if (g == 0) {
    uint16_t g16 = 0;
    if (n2) {
      const double rr = (double)n2 / (double)M;
      const double root = sqrt(rr);
      g16 = f64_to_f16_rne_sat(root * ((double)sK * 0.015625));
    }
    reinterpret_cast<uint16_t*>(reg + 12 * D)[t] = g16;
  }
}

// Values (enc_values): lane l owns channel 64 i + l, i < D/64.  zero = fp16(min),
// scale = fp16((max - min) / 7) and code = clamp(rint((v - zero) / scale), 0, 7)
// are defined in fp64.  The code is computed as fma(e, sV / scale, -zero / scale)
// in fp32 (e the E4M3 value), whose error is below G = 2^-21 (|zero / scale| + 8)
// wherever the code is not clamped anyway: it is the fp64 one unless the
// result lies within G of a rounding boundary, and a wave with such a value
// (about one in a hundred) takes the fp64 division.  The quads meet in LDS, where
// lane 16 g + r builds chunk (r, g).
template <int D>
__device__ __forceinline__ void enc_values(const uint8_t* f8, float sV, uint8_t* reg, uint32_t* lds, int lane) {
  constexpr int CL = D / 16, NDW = 3 * D / 128, CB = 3 * D / 32, NI = D / 64, LP = enc_row(D);
  uint32_t w[NI][4];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int c = 64 * i + lane;
      w[i][g] = reinterpret_cast<const uint32_t*>(f8 + PAGE * D)[((c / CL) * 4 + g) * CL + c % CL];
    }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = 64 * i + lane;
    typedef float f2 __attribute__((ext_vector_type(2)));
    float e[PAGE];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f2 lo2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w[i][g], 1.0f, false);
      const f2 hi2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w[i][g], 1.0f, true);
      e[4 * g] = lo2[0], e[4 * g + 1] = lo2[1], e[4 * g + 2] = hi2[0], e[4 * g + 3] = hi2[1];
    }
    float emin = e[0], emax = e[0];
#pragma unroll
    for (int t = 1; t < PAGE; ++t) {
      emin = fminf(emin, e[t]);
      emax = fmaxf(emax, e[t]);
    }
    // (a page that holds an infinity has an infinite scale: a token whose code is zero is
    // then no number and counts for neither bound)
    if (sV == INFINITY) {
      emin = emin == 0.0f ? 1.0f : emin;
      emax = emax == 0.0f ? -1.0f : emax;
    }
    const double lo = (double)sV * (double)emin, hi = (double)sV * (double)emax;  // exact; sV >= 0
    const uint16_t z16 = f64_to_f16_rne_sat(lo);
    const uint16_t s16 = f64_to_f16_rne_sat((hi - lo) / 7.0);
    reinterpret_cast<uint16_t*>(reg + 12 * D + 32)[c] = s16;
    reinterpret_cast<uint16_t*>(reg + 14 * D + 32)[c] = z16;
    const float zf = (float)__builtin_bit_cast(_Float16, z16), sf = (float)__builtin_bit_cast(_Float16, s16);
    const float a = sf != 0.0f ? sV / sf : 0.0f, b = sf != 0.0f ? -zf / sf : 0.0f;
    const float lim = 0.5f - (fabsf(b) + 8.0f) * 0x1p-21f;
    uint32_t quad[4];
    float off = 0.0f;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      quad[g] = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float q = __builtin_fmaf(e[4 * g + u], a, b);
        const float rq = __builtin_rintf(q);
        off = fmaxf(off, fabsf(q - rq));
        quad[g] = __builtin_amdgcn_cvt_pk_u8_f32(fminf(fmaxf(rq, 0.0f), 7.0f), u, quad[g]);
      }
    }
    if (__any(!(off <= lim))) {
      const double z = f16_bits_to_f64(z16), s = f16_bits_to_f64(s16);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        quad[g] = 0;
#pragma unroll 1
        for (int u = 0; u < 4; ++u) {
          const double v = (double)sV * (double)e4m3_to_f32((w[i][g] >> (8 * u)) & 0xFFu);
          const double q = fmin(fmax(rint((v - z) / s), 0.0), 7.0);
          quad[g] |= (s != 0.0 ? (uint32_t)q : 0u) << (8 * u);
        }
      }
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) lds[((c / CL) * 4 + g) * LP + c % CL] = quad[g];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  {
    const int g = lane >> 4, r = lane & 15;
    uint32_t quad[CL], dw[NDW];
    const uint4* row = reinterpret_cast<const uint4*>(lds + (r * 4 + g) * LP);
#pragma unroll
    for (int q = 0; q < CL / 4; ++q) {
      const uint4 x = row[q];
      quad[4 * q] = x.x, quad[4 * q + 1] = x.y, quad[4 * q + 2] = x.z, quad[4 * q + 3] = x.w;
    }
    pack_quads<NDW>(dw, quad);
    store_chunk<NDW>(reinterpret_cast<uint32_t*>(reg + 6 * D + (g * 16 + r) * CB), dw);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();  // the rows are free for the wave's next page-head
}

// Encode every listed page-head (listed pages x layers x heads, grid-stride).
// Waves 2 j and 2 j + 1 of the launch take one page-head together, one its keys
// and one its values, and swap the roles from one page-head to the next (the key
// half has about 1.7 times the instructions).  Bound by VALU issue: about
// 1,700 + 1,000 instructions per page-head of d = 256.  The launch is what one
// round of resident workgroups holds: a decode step, which lists a page or two
// or none, pays for few workgroups.
constexpr int ENC_WG = 4;  // waves per workgroup
template <int D>
__global__ __launch_bounds__(64 * ENC_WG, 3) void migrate_encode_kernel(PoolView P) {
  if (P.ctrl[CTRL_ABORT]) return;
  __shared__ __align__(16) uint32_t s_quads[ENC_WG][64 * enc_row(D)];
  const int H = P.n_kv_heads, L = P.n_layers;
  const int64_t n_items = (int64_t)P.ctrl[CTRL_NLIST] * L * H;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t pair0 = (int64_t)blockIdx.x * (ENC_WG / 2) + (wid >> 1);
  if (pair0 >= n_items) return;
  // sign bits of the rotation's diagonal at the E4M3 bytes of this lane's key channels
  uint32_t sgn[D / 16];
  {
    const uint32_t* sg = reinterpret_cast<const uint32_t*>(P.sigma + (D / 4) * (lane & 3));
#pragma unroll
    for (int i = 0; i < D / 16; ++i) sgn[i] = sg[i] & 0x80808080u;
  }
  int role = (wid + blockIdx.x) & 1;
  for (int64_t item = pair0; item < n_items; item += (int64_t)gridDim.x * (ENC_WG / 2), role ^= 1) {
    const int e = (int)(item / (L * H));
    const int lh = (int)(item % (L * H));
    const int layer = lh / H, h = lh % H;
    const int src = P.list[4 * e + 2], dst = P.list[4 * e + 3];
    const int64_t sph = ((int64_t)layer * P.n_fp8 + src) * H + h;
    const uint8_t* f8 = P.fp8 + sph * fp8_region_bytes(D);
    uint8_t* reg = P.tq3 + (((int64_t)layer * P.n_tq3 + dst) * H + h) * tq3_region_bytes(D);
    if (role == 0)
      enc_keys<D>(sgn, f8, P.fp8_scales[sph * 2], reg, lane);
    else
      enc_values<D>(f8, P.fp8_scales[sph * 2 + 1], reg, s_quads[wid], lane);
  }
}

__global__ __launch_bounds__(1024) void migrate_publish_kernel(int32_t* bt, uint8_t* tags,
                                                               int max_pages, int32_t* ctrl,
                                                               int32_t* fp8_stack,
                                                               const int32_t* list, int32_t* rc8,
                                                               int32_t* rc3) {
  if (ctrl[CTRL_ABORT]) return;
  const int n = ctrl[CTRL_NLIST];
  const int top = ctrl[CTRL_FP8_TOP];
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    const int r = list[4 * k], p = list[4 * k + 1], src = list[4 * k + 2], dst = list[4 * k + 3];
    const int64_t i = (int64_t)r * max_pages + p;
    bt[i] = dst;
    tags[i] = TAG_S;
    rc3[dst] = 1;  // the request's reference moves to the new page
    rc8[src] = 0;
    fp8_stack[top + k] = src;
  }
  __syncthreads();
  if (threadIdx.x == 0) ctrl[CTRL_FP8_TOP] = top + n;
}

// ===========================================================================
// Promote (a Stale page back to FP8)
// ===========================================================================

// Plan of a promotion: one workgroup walks the table twice (count and
// validate, then list in (request, page) order with one block scan per batch), or
// once when the table is one batch (ONE: up to MIG_BATCH entries, kept in
// registers and ranked by wave ballots).
// A page is promoted when it is Stale, its mask entry is set and it lies below
// the request's length.  A failing call (bad length, out-of-range TQ3 id, FP8
// free list too short) sets the error word and the abort flag and lists
// nothing.  The FP8 ids are popped here; the pages are built by the build
// kernel and published after it (copy before publish).
__device__ __forceinline__ bool pro_hit(const MigBatch& m, int j) {
  if (m.rq[j] < 0 || m.tg[j] != TAG_S || !m.an[j] || m.rc[j] != 1) return false;
  return m.pg[j] < (m.sl[j] + PAGE - 1) / PAGE;
}

template <bool ONE>
__global__ __launch_bounds__(MIG_NT) void promote_plan_kernel(
    int n_req, const int32_t* bt, const uint8_t* tags, int max_pages, const uint8_t* mask,
    const int32_t* seq_lens, int32_t* ctrl, const int32_t* fp8_stack, int32_t* list, int n_tq3,
    RcView rv) {
  __shared__ int scratch[32];
  __shared__ int s_cnt[16 * MIG_KB + 1];
  __shared__ int s_err, s_tot;
  const int tid = threadIdx.x;
  if (tid == 0) { s_err = 0; s_tot = 0; }
  __syncthreads();
  if constexpr (ONE) {
    const int top8 = ctrl[CTRL_FP8_TOP];
    MigBatch m;
    mig_load_striped(m, n_req * max_pages, max_pages, bt, tags, mask, seq_lens);
    int err = 0, wcnt[MIG_KB], base[MIG_KB];
    for (int r = tid; r < n_req; r += MIG_NT) {
      const int S = seq_lens[r];
      if (S < 0 || (S + PAGE - 1) / PAGE > max_pages) err |= MKV_DEVERR_RANGE;
    }
    mig_load_rc(m, rv);
    bool hit[MIG_KB];
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      if (m.rq[j] >= 0 && m.tg[j] == TAG_S && m.an[j] && m.pg[j] < (m.sl[j] + PAGE - 1) / PAGE &&
          (m.id[j] < 0 || m.id[j] >= n_tq3))
        err |= MKV_DEVERR_RANGE;
      hit[j] = pro_hit(m, j);
      wcnt[j] = __popcll(__ballot(hit[j]));
    }
    if (err) atomicOr(&s_err, err);
    const int total = striped_bases<MIG_KB>(wcnt, base, s_cnt);  // its barriers also publish s_err
    err = s_err;
    if (err == 0 && total > top8) err |= MKV_DEVERR_FP8_EXHAUSTED;
    if (err) {
      if (tid == 0) {
        atomicOr(&ctrl[CTRL_ERR], err);
        ctrl[CTRL_ABORT] = 1;
        ctrl[CTRL_NLIST] = 0;
      }
      return;
    }
    const uint64_t below = (1ull << (tid & 63)) - 1ull;
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      const int e = base[j] + __popcll(__ballot(hit[j]) & below);
      if (hit[j]) {
        int32_t* le = list + 4LL * e;
        le[0] = m.rq[j];
        le[1] = m.pg[j];
        le[2] = m.id[j];                   // TQ3 source
        le[3] = fp8_stack[top8 - 1 - e];   // FP8 destination
      }
    }
    if (tid == 0) {
      ctrl[CTRL_FP8_TOP] = top8 - total;
      ctrl[CTRL_NLIST] = total;
      ctrl[CTRL_ABORT] = 0;
    }
    return;
  }
  const int64_t N = (int64_t)n_req * max_pages;
  int err = 0, cnt = 0;
  for (int r = tid; r < n_req; r += MIG_NT) {
    const int S = seq_lens[r];
    if (S < 0 || (S + PAGE - 1) / PAGE > max_pages) err |= MKV_DEVERR_RANGE;
  }
  for (int64_t b0 = 0; b0 < N; b0 += MIG_BATCH) {
    MigBatch m;
    mig_load(m, b0 + (int64_t)tid * MIG_KB, N, max_pages, bt, tags, mask, seq_lens);
    mig_load_rc(m, rv);
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      if (m.rq[j] >= 0 && m.tg[j] == TAG_S && m.an[j] && m.pg[j] < (m.sl[j] + PAGE - 1) / PAGE &&
          (m.id[j] < 0 || m.id[j] >= n_tq3))
        err |= MKV_DEVERR_RANGE;
      if (pro_hit(m, j)) {
        cnt++;
      }
    }
  }
  if (cnt) atomicAdd(&s_tot, cnt);
  if (err) atomicOr(&s_err, err);
  __syncthreads();
  const int total = s_tot;
  const int top8 = ctrl[CTRL_FP8_TOP];
  err = s_err;
  if (err == 0 && total > top8) err |= MKV_DEVERR_FP8_EXHAUSTED;
  if (err) {
    if (tid == 0) {
      atomicOr(&ctrl[CTRL_ERR], err);
      ctrl[CTRL_ABORT] = 1;
      ctrl[CTRL_NLIST] = 0;
    }
    return;
  }
  int base = 0;
  for (int64_t b0 = 0; b0 < N; b0 += MIG_BATCH) {
    MigBatch m;
    const int64_t f0 = b0 + (int64_t)tid * MIG_KB;
    mig_load(m, f0, N, max_pages, bt, tags, mask, seq_lens);
    mig_load_rc(m, rv);
    bool hit[MIG_KB];
    int c = 0;
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      hit[j] = pro_hit(m, j);
      c += hit[j];
    }
    int tot;
    int e = base + block_excl_scan(c, scratch, &tot);
#pragma unroll
    for (int j = 0; j < MIG_KB; ++j) {
      if (hit[j]) {
        int32_t* le = list + 4LL * e;
        le[0] = m.rq[j];
        le[1] = m.pg[j];
        le[2] = m.id[j];                   // TQ3 source
        le[3] = fp8_stack[top8 - 1 - e];   // FP8 destination
        e++;
      }
    }
    base += tot;
  }
  if (tid == 0) {
    ctrl[CTRL_FP8_TOP] = top8 - total;
    ctrl[CTRL_NLIST] = total;
    ctrl[CTRL_ABORT] = 0;
  }
}

// One half of a rebuilt page-head: the lane's D/4 values, neighbours in the FP8
// layout, and the page's scale.  s = amax / 448 over the 16 x D values, code =
// E4M3(x / s) (0 when s = 0).
template <int D>
__device__ __forceinline__ void dec_store(const float (&x)[D / 4], uint8_t* dst, float* scale, int lane) {
  float amax = 0.0f;
#pragma unroll
  for (int i = 0; i < D / 4; ++i) amax = fmaxf(amax, fabsf(x[i]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
  const float s = amax / 448.0f;
  uint32_t w[D / 16];
  if (__builtin_amdgcn_readfirstlane(div_fast(s))) {
    const float y = 1.0f / s;
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
      w[i] = pack_e4m3(div_by(x[4 * i], s, y), div_by(x[4 * i + 1], s, y), div_by(x[4 * i + 2], s, y),
                       div_by(x[4 * i + 3], s, y));
  } else {
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
      w[i] = s > 0.0f ? pack_e4m3(x[4 * i] / s, x[4 * i + 1] / s, x[4 * i + 2] / s, x[4 * i + 3] / s) : 0u;
  }
#pragma unroll
  for (int i = 0; i < D / 64; ++i)
    reinterpret_cast<uint4*>(dst)[i] = make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
  if (lane == 0) *scale = s;
}
// the quads of the chunk at c
template <int NDW>
__device__ __forceinline__ void load_chunk(uint32_t* dw, const uint8_t* c) {
  if constexpr (NDW % 2 == 0) {
#pragma unroll
    for (int j = 0; j < NDW / 2; ++j) {
      const uint2 v = reinterpret_cast<const uint2*>(c)[j];
      dw[2 * j] = v.x;
      dw[2 * j + 1] = v.y;
    }
  } else {
#pragma unroll
    for (int j = 0; j < NDW; ++j) dw[j] = reinterpret_cast<const uint32_t*>(c)[j];
  }
}
// Keys of a page-head: lane 4 t + g owns K chunk (t, g), channels D/4 g .. of token
// t.  codes -> 8 * codebook level (integers), the Walsh-Hadamard transform (sums of
// integers below 2^13, exact in fp32), then k = fp32((gamma * sigma_c * (y_c / 8)) /
// sqrt(D)): gamma (11 bits) times y is exact in fp32, so the division is the only
// rounding (D = 256: a power of two, none before the conversion).
template <int D>
__device__ __forceinline__ void dec_keys(const uint32_t* sgn, const uint8_t* reg, uint8_t* f8, float* scale,
                                         int lane) {
  constexpr int QK = D / 4, NDW = 3 * D / 128, CB = 3 * D / 32;
  const int t = lane >> 2, g = lane & 3;
  uint32_t dw[NDW];
  load_chunk<NDW>(dw, reg + (g * 16 + t) * CB);
  const float gam = (float)reinterpret_cast<const _Float16*>(reg + 12 * D)[t];
  float y[QK];
#pragma unroll
  for (int q = 0; q < QK / 4; ++q) {
    // levels -18, -11, -6, -2, 2, 6, 11, 18 by code
    const uint32_t l = __builtin_amdgcn_perm(0x120B0602u, 0xFEFAF5EEu, quad_sel<NDW>(dw, q));
#pragma unroll
    for (int b = 0; b < 4; ++b) y[4 * q + b] = (float)(int)(int8_t)(l >> (8 * b));
  }
#pragma unroll
  for (int st = 1; st < QK; st <<= 1)
#pragma unroll
    for (int i = 0; i < QK; ++i)
      if (!(i & st)) {
        const float a0 = y[i], a1 = y[i + st];
        y[i] = a0 + a1;
        y[i + st] = a0 - a1;
      }
  // strides D/4 and D/2: lanes g ^ 1 and g ^ 2
  const float m1 = (g & 1) ? -1.0f : 1.0f, m2 = (g & 2) ? -1.0f : 1.0f;
  auto dpp = [](float v, auto ctl) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctl)::value, 0xF, 0xF, false));
  };
#pragma unroll
  for (int i = 0; i < QK; ++i) {
    y[i] = __builtin_fmaf(m1, y[i], dpp(y[i], std::integral_constant<int, 0xB1>{}));
    y[i] = __builtin_fmaf(m2, y[i], dpp(y[i], std::integral_constant<int, 0x4E>{}));
  }
  const double rd = sqrt((double)D);
#pragma unroll
  for (int i = 0; i < QK; ++i) {
    const uint32_t flip = (sgn[i / 4] << (24 - 8 * (i % 4))) & 0x80000000u;
    const float a = __uint_as_float(__float_as_uint(gam) ^ flip) * (y[i] * 0.125f);  // exact
    if constexpr (D == 256) y[i] = a * 0.0625f;
    else y[i] = (float)((double)a / rd);
  }
  dec_store<D>(y, f8 + t * D + QK * g, scale, lane);
}
// Values: lane 16 g + r owns V chunk (r, g), whose quad m is the FP8 layout's dword
// m of lane-chunk (r, g) (tokens 4 g .. of channel CL r + m).  v = fp32(zero_c +
// scale_c * code): one fused multiply-add, the product and sum exact before its
// rounding.
template <int D>
__device__ __forceinline__ void dec_values(const uint8_t* reg, uint8_t* f8, float* scale, int lane) {
  constexpr int CL = D / 16, NDW = 3 * D / 128, CB = 3 * D / 32;
  const int g = lane >> 4, r = lane & 15;
  uint32_t dw[NDW];
  load_chunk<NDW>(dw, reg + 6 * D + (g * 16 + r) * CB);
  half8 sc[CL / 8], zr[CL / 8];
#pragma unroll
  for (int i = 0; i < CL / 8; ++i) {
    sc[i] = reinterpret_cast<const half8*>(reg + 12 * D + 32 + 2 * CL * r)[i];
    zr[i] = reinterpret_cast<const half8*>(reg + 14 * D + 32 + 2 * CL * r)[i];
  }
  float v[D / 4];
#pragma unroll
  for (int m = 0; m < CL; ++m) {
    const uint32_t q = quad_sel<NDW>(dw, m);
#pragma unroll
    for (int b = 0; b < 4; ++b)
      v[4 * m + b] = __builtin_fmaf((float)sc[m / 8][m % 8], (float)((q >> (8 * b)) & 0xFFu), (float)zr[m / 8][m % 8]);
  }
  dec_store<D>(v, f8 + PAGE * D + (r * 4 + g) * (D / 4), scale, lane);
}

// Rebuild every listed page-head (layer, KV head) from its TQ3 region into its new
// FP8 region, two waves to a page-head, one its keys and one its values, roles
// swapped from one page-head to the next (as in the encode).  Everything stays in
// registers and there is no barrier: 95 pages x 4 heads x 4 layers at d = 256 took
// 36 us with a workgroup and an LDS transform per page-head, now 16.5 us.
template <int D>
__global__ __launch_bounds__(64 * ENC_WG, 2) void promote_build_kernel(PoolView P) {
  if (P.ctrl[CTRL_ABORT]) return;
  const int H = P.n_kv_heads, L = P.n_layers;
  const int64_t n_items = (int64_t)P.ctrl[CTRL_NLIST] * L * H;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t pair0 = (int64_t)blockIdx.x * (ENC_WG / 2) + (wid >> 1);
  if (pair0 >= n_items) return;
  // sign bits of the rotation's diagonal at the bytes of this lane's key channels
  uint32_t sgn[D / 16];
  {
    const uint32_t* sg = reinterpret_cast<const uint32_t*>(P.sigma + (D / 4) * (lane & 3));
#pragma unroll
    for (int i = 0; i < D / 16; ++i) sgn[i] = sg[i] & 0x80808080u;
  }
  int role = (wid + blockIdx.x) & 1;
  for (int64_t item = pair0; item < n_items; item += (int64_t)gridDim.x * (ENC_WG / 2), role ^= 1) {
    const int e = (int)(item / (L * H));
    const int lh = (int)(item % (L * H));
    const int layer = lh / H, h = lh % H;
    const int src = P.list[4 * e + 2], dst = P.list[4 * e + 3];
    const uint8_t* reg = P.tq3 + (((int64_t)layer * P.n_tq3 + src) * H + h) * tq3_region_bytes(D);
    const int64_t ph = ((int64_t)layer * P.n_fp8 + dst) * H + h;
    uint8_t* f8 = P.fp8 + ph * fp8_region_bytes(D);
    if (role == 0)
      dec_keys<D>(sgn, reg, f8, P.fp8_scales + ph * 2, lane);
    else
      dec_values<D>(reg, f8, P.fp8_scales + ph * 2 + 1, lane);
  }
}

// Publish (Anchor, new FP8 id) and release the TQ3 ids, in list order.
__global__ __launch_bounds__(1024) void promote_publish_kernel(int32_t* bt, uint8_t* tags,
                                                               int max_pages, int32_t* ctrl,
                                                               int32_t* tq3_stack,
                                                               const int32_t* list, int32_t* rc8,
                                                               int32_t* rc3) {
  if (ctrl[CTRL_ABORT]) return;
  const int n = ctrl[CTRL_NLIST];
  const int top = ctrl[CTRL_TQ3_TOP];
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    const int32_t* le = list + 4LL * k;
    const int64_t i = (int64_t)le[0] * max_pages + le[1];
    bt[i] = le[3];
    tags[i] = TAG_A;
    rc8[le[3]] = 1;
    rc3[le[2]] = 0;
    tq3_stack[top + k] = le[2];
  }
  __syncthreads();
  if (threadIdx.x == 0) ctrl[CTRL_TQ3_TOP] = top + n;
}

// ===========================================================================
// Reference counts: SealPrefix / prefix attach (acquire), eviction and Finish
// (release)
// ===========================================================================

// (format, id) of a tagged entry: 0 FP8 (tags R, A), 1 TQ3 (tag S); false when
// the tag names no pool or the id is out of range.
__device__ __forceinline__ bool ref_of(uint8_t tag, int id, int n_fp8, int n_tq3, int& fmt) {
  fmt = tag == TAG_S ? 1 : 0;
  if (tag != TAG_R && tag != TAG_A && tag != TAG_S) return false;
  return id >= 0 && id < (fmt ? n_tq3 : n_fp8);
}

// One workgroup: every listed page must be live (one reference or more);
// otherwise nothing changes.  Then one more reference per entry.
__global__ __launch_bounds__(1024) void pages_acquire_kernel(int n, const int32_t* ids,
                                                             const uint8_t* tags, PoolView P) {
  __shared__ int s_err;
  const int tid = threadIdx.x;
  if (tid == 0) s_err = 0;
  __syncthreads();
  for (int k = tid; k < n; k += blockDim.x) {
    int fmt;
    const int id = ids[k];
    if (!ref_of(tags[k], id, P.n_fp8, P.n_tq3, fmt) || (fmt ? P.rc3 : P.rc8)[id] < 1)
      atomicOr(&s_err, (int)MKV_DEVERR_REFCOUNT);
  }
  __syncthreads();
  if (s_err) {
    if (tid == 0) atomicOr(&P.ctrl[CTRL_ERR], s_err);
    return;
  }
  for (int k = tid; k < n; k += blockDim.x) {
    int fmt;
    const int id = ids[k];
    (void)ref_of(tags[k], id, P.n_fp8, P.n_tq3, fmt);
    atomicAdd(&(fmt ? P.rc3 : P.rc8)[id], 1);
  }
}

// One workgroup.  Entries: an explicit list (reqs == nullptr: ids/tags[n]) or
// the rows of the listed requests (entry j * max_pages + p = row reqs[j], page
// p, mapped entries only).  Each entry drops one reference, in entry order: a
// page whose count reaches zero is pushed onto its free list at its last
// entry.  Pass 1 counts each page's entries and finds its last one; a page with
// more entries than references, a bad tag or id, or a bad request list fails the
// call (nothing changed).  Pass 2 ranks the freeing entries in order, applies the
// counts and unmaps the table rows.
// Bound by the pages' scattered words, one address a cycle for the workgroup's CU,
// and by memory round trips in a row.  So REL_KB entries per thread are in flight
// (entry b0 + j NT + tid in slot j), and a call of one batch (REL_BATCH entries)
// keeps its entries in registers and finds counts and last entries in an LDS hash
// table of the pages: only the reference counts are scattered.  A longer call
// does that in the pool's scratch (occ / last, 0 / -1 at rest, restored when the
// call fails) and loads its entries again in every pass.  16 rows of 214 pages take
// 8.8 us, 22 us with the scratch, and 28 us entry by entry.
constexpr int REL_NT = 1024, REL_KB = 4;
constexpr int64_t REL_BATCH = (int64_t)REL_NT * REL_KB;
constexpr int REL_SLOTS = (int)REL_BATCH * 3 / 2;  // hash slots: two thirds full at most
__global__ __launch_bounds__(REL_NT) void pages_release_kernel(int n, const int32_t* ids,
                                                               const uint8_t* tags, int n_fin,
                                                               const int32_t* reqs, int n_req,
                                                               int32_t* bt, uint8_t* bt_tags,
                                                               int max_pages, PoolView P) {
  __shared__ int s_cnt[16 * REL_KB + 1];
  __shared__ int s_err;
  __shared__ int s_key[REL_SLOTS], s_occ[REL_SLOTS];
  const int tid = threadIdx.x;
  const bool table = reqs != nullptr;
  const int64_t N = table ? (int64_t)n_fin * max_pages : n;
  const bool one = N <= REL_BATCH;
  const int top8 = P.ctrl[CTRL_FP8_TOP], top3 = P.ctrl[CTRL_TQ3_TOP];
  if (tid == 0) s_err = 0;
  if (one)
    for (int i = tid; i < REL_SLOTS; i += REL_NT) {
      s_key[i] = -1;
      s_occ[i] = 0;
    }
  __syncthreads();
  // a batch's entries: where they stand, page id, format; REL_NO: no entry or an
  // unmapped one, REL_BAD: names no page
  enum { REL_FP8 = 0, REL_TQ3 = 1, REL_NO = 2, REL_BAD = 3 };
  int id[REL_KB], fm[REL_KB];
  int64_t at[REL_KB];  // index of the table entry, -1: none
  auto load = [&](int64_t b0) {
    uint8_t tg[REL_KB];
#pragma unroll
    for (int j = 0; j < REL_KB; ++j) {
      const int64_t k = b0 + j * REL_NT + tid;
      at[j] = -1;
      id[j] = -1;
      tg[j] = TAG_NONE;
      fm[j] = REL_NO;
      if (b0 + j * REL_NT < N) {  // workgroup-uniform
        const bool in = k < N;
        if (table) {
          const int64_t kk = in ? k : 0;
          const int64_t q = N >> 32 ? kk / max_pages : (int64_t)((uint32_t)kk / (uint32_t)max_pages);
          const int r = reqs[q];
          // (a row out of range fails the call before anything is applied)
          if (in && r >= 0 && r < n_req) at[j] = (int64_t)r * max_pages + (kk - q * max_pages);
        } else if (in) {
          at[j] = k;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < REL_KB; ++j)
      if (b0 + j * REL_NT < N && at[j] >= 0) {
        id[j] = table ? bt[at[j]] : ids[at[j]];
        tg[j] = table ? bt_tags[at[j]] : tags[at[j]];
      }
#pragma unroll
    for (int j = 0; j < REL_KB; ++j)
      if (at[j] >= 0 && !(table && id[j] < 0)) {
        int f;
        fm[j] = ref_of(tg[j], id[j], P.n_fp8, P.n_tq3, f) ? f : REL_BAD;
      }
  };
  load(0);
  if (table) {
    for (int j = tid; j < n_fin; j += REL_NT) {
      const int r = reqs[j];
      if (r < 0 || r >= n_req || (j > 0 && reqs[j - 1] >= r)) atomicOr(&s_err, (int)MKV_DEVERR_RANGE);
    }
    __syncthreads();
    const int err = s_err;
    __syncthreads();  // read by every wave before one finds a bad entry below
    if (err) {
      if (tid == 0) atomicOr(&P.ctrl[CTRL_ERR], err);
      return;
    }
  }
  int occ[REL_KB], rc[REL_KB], lst[REL_KB];
  if (one) {
    int slot[REL_KB];
#pragma unroll
    for (int j = 0; j < REL_KB; ++j) {
      occ[j] = rc[j] = slot[j] = 0;
      lst[j] = -1;
      if (fm[j] < REL_NO) rc[j] = (fm[j] ? P.rc3 : P.rc8)[id[j]];
      if (fm[j] == REL_BAD) atomicOr(&s_err, (int)MKV_DEVERR_REFCOUNT);
    }
#pragma unroll
    for (int j = 0; j < REL_KB; ++j)
      if (fm[j] < REL_NO) {  // the page's slot: there are more slots than entries, so one is found
        const int key = (int)((uint32_t)id[j] << 1) | fm[j];
        int h = (int)__umulhi((uint32_t)key * 2654435761u, (uint32_t)REL_SLOTS);
        for (int old; (old = atomicCAS(&s_key[h], -1, key)) != -1 && old != key;) h = h + 1 == REL_SLOTS ? 0 : h + 1;
        atomicAdd(&s_occ[h], 1);
        slot[j] = h;
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < REL_KB; ++j)
      if (fm[j] < REL_NO) {
        occ[j] = s_occ[slot[j]];
        s_key[slot[j]] = 0;  // from here on the slot's largest entry index
        if (occ[j] > rc[j]) atomicOr(&s_err, (int)MKV_DEVERR_REFCOUNT);
      }
    __syncthreads();
    if (s_err) {
      if (tid == 0) atomicOr(&P.ctrl[CTRL_ERR], s_err);
      return;
    }
#pragma unroll
    for (int j = 0; j < REL_KB; ++j)
      if (fm[j] < REL_NO) atomicMax(&s_key[slot[j]], j * REL_NT + tid);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < REL_KB; ++j)
      if (fm[j] < REL_NO) lst[j] = s_key[slot[j]];
  } else {
    for (int64_t b0 = 0; b0 < N; b0 += REL_BATCH) {
      if (b0 > 0) load(b0);
#pragma unroll
      for (int j = 0; j < REL_KB; ++j) {
        if (fm[j] == REL_BAD) atomicOr(&s_err, (int)MKV_DEVERR_REFCOUNT);
        if (fm[j] < REL_NO) {
          atomicAdd(&(fm[j] ? P.occ3 : P.occ8)[id[j]], 1);
          atomicMax(&(fm[j] ? P.last3 : P.last8)[id[j]], (int)(b0 + j * REL_NT + tid));
        }
      }
    }
    __syncthreads();
  }
  auto counts = [&]() {
#pragma unroll
    for (int j = 0; j < REL_KB; ++j) {
      occ[j] = rc[j] = 0;
      lst[j] = -1;
      if (fm[j] < REL_NO) {
        occ[j] = (fm[j] ? P.occ3 : P.occ8)[id[j]];
        rc[j] = (fm[j] ? P.rc3 : P.rc8)[id[j]];
        lst[j] = (fm[j] ? P.last3 : P.last8)[id[j]];
      }
    }
  };
  if (!one) {
    for (int64_t b0 = 0; b0 < N; b0 += REL_BATCH) {
      load(b0);
      counts();
#pragma unroll
      for (int j = 0; j < REL_KB; ++j)
        if (occ[j] > rc[j]) atomicOr(&s_err, (int)MKV_DEVERR_REFCOUNT);
    }
    __syncthreads();
    const int err = s_err;
    if (err) {
      for (int64_t b0 = 0; b0 < N; b0 += REL_BATCH) {
        load(b0);
#pragma unroll
        for (int j = 0; j < REL_KB; ++j)
          if (fm[j] < REL_NO) {
            (fm[j] ? P.occ3 : P.occ8)[id[j]] = 0;
            (fm[j] ? P.last3 : P.last8)[id[j]] = -1;
          }
      }
      if (tid == 0) atomicOr(&P.ctrl[CTRL_ERR], err);
      return;
    }
  }
  const uint64_t below = (1ull << (tid & 63)) - 1ull;
  int base8 = 0, base3 = 0;
  for (int64_t b0 = 0; b0 < N; b0 += REL_BATCH) {
    if (!one) {
      load(b0);
      counts();
    }
    // waves' counts of the freeing entries, FP8 in the low and TQ3 in the high half
    bool freed[REL_KB];
    int cnt[REL_KB], base[REL_KB];
#pragma unroll
    for (int j = 0; j < REL_KB; ++j) {
      const bool last = fm[j] < REL_NO && lst[j] == (int)(b0 + j * REL_NT + tid);
      freed[j] = last && rc[j] == occ[j];
      cnt[j] = __popcll(__ballot(freed[j] && fm[j] == REL_FP8)) | __popcll(__ballot(freed[j] && fm[j] == REL_TQ3)) << 16;
      if (last) {
        (fm[j] ? P.rc3 : P.rc8)[id[j]] = rc[j] - occ[j];
        if (!one) {
          (fm[j] ? P.occ3 : P.occ8)[id[j]] = 0;
          (fm[j] ? P.last3 : P.last8)[id[j]] = -1;
        }
      }
      if (table && at[j] >= 0) {
        bt[at[j]] = -1;
        bt_tags[at[j]] = TAG_NONE;
      }
    }
    const int tot = striped_bases<REL_KB>(cnt, base, s_cnt);
#pragma unroll
    for (int j = 0; j < REL_KB; ++j) {
      const uint64_t m8 = __ballot(freed[j] && fm[j] == REL_FP8), m3 = __ballot(freed[j] && fm[j] == REL_TQ3);
      if (freed[j]) {
        if (fm[j]) P.tq3_stack[top3 + base3 + (base[j] >> 16) + __popcll(m3 & below)] = id[j];
        else P.fp8_stack[top8 + base8 + (base[j] & 0xFFFF) + __popcll(m8 & below)] = id[j];
      }
    }
    base8 += tot & 0xFFFF;
    base3 += tot >> 16;
    __syncthreads();  // s_cnt is free for the next batch
  }
  if (tid == 0) {
    P.ctrl[CTRL_FP8_TOP] = top8 + base8;
    P.ctrl[CTRL_TQ3_TOP] = top3 + base3;
  }
}

hipError_t launch_pages_acquire(const PoolView& P, int n, const int32_t* ids, const uint8_t* tags,
                                hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(pages_acquire_kernel, dim3(1), dim3(1024), 0, s, n, ids, tags, P);
  return hipGetLastError();
}

hipError_t launch_pages_release(const PoolView& P, int n, const int32_t* ids, const uint8_t* tags,
                                int n_fin, const int32_t* reqs, int n_req, int32_t* bt,
                                uint8_t* bt_tags, int max_pages, hipStream_t s) {
  if ((reqs ? n_fin : n) == 0) return hipSuccess;
  hipLaunchKernelGGL(pages_release_kernel, dim3(1), dim3(REL_NT), 0, s, n, ids, tags, n_fin, reqs,
                     n_req, bt, bt_tags, max_pages, P);
  return hipGetLastError();
}

// ===========================================================================
// Compact per-format page lists
// ===========================================================================
__global__ __launch_bounds__(1024) void partition_kernel(const int32_t* bt, const uint8_t* tags,
                                                         int max_pages, const int32_t* seq_lens,
                                                         int32_t* list8, int32_t* list3,
                                                         int32_t* counts, int32_t* err) {
  __shared__ int scratch[32];
  const int r = blockIdx.x, tid = threadIdx.x;
  const int S = seq_lens[r];
  const int np = (S + PAGE - 1) / PAGE;
  if (S < 1 || np > max_pages) {
    if (tid == 0) {
      counts[2 * r] = 0;
      counts[2 * r + 1] = 0;
      if (err) atomicOr(err, (int)MKV_DEVERR_RANGE);
    }
    return;
  }
  int b8 = 0, b3 = 0, bad = 0;
  for (int c0 = 0; c0 < np; c0 += blockDim.x) {
    const int p = c0 + tid;
    const int64_t i = (int64_t)r * max_pages + p;
    const int tg = p < np ? tags[i] : TAG_NONE;
    const int is8 = (p < np && (tg == TAG_R || tg == TAG_A)) ? 1 : 0;
    const int is3 = (p < np && tg == TAG_S) ? 1 : 0;
    if (p < np && !is8 && !is3) bad = 1;
    int t8, t3;
    const int r8 = block_excl_scan(is8, scratch, &t8);
    const int r3 = block_excl_scan(is3, scratch, &t3);
    if (is8) {
      list8[((int64_t)r * max_pages + b8 + r8) * 2] = p;
      list8[((int64_t)r * max_pages + b8 + r8) * 2 + 1] = bt[i];
    }
    if (is3) {
      list3[((int64_t)r * max_pages + b3 + r3) * 2] = p;
      list3[((int64_t)r * max_pages + b3 + r3) * 2 + 1] = bt[i];
    }
    b8 += t8;
    b3 += t3;
  }
  if (bad && err) atomicOr(err, (int)MKV_DEVERR_BAD_TAG);
  if (tid == 0) {
    counts[2 * r] = b8;
    counts[2 * r + 1] = b3;
  }
}

__global__ void fill_zero_kernel(uint32_t* p, int64_t n_words) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// ===========================================================================
// Launchers
// ===========================================================================

hipError_t launch_append(const PoolView& P, int layer, int n_req, int32_t* bt, uint8_t* tags,
                         int max_pages, const int32_t* sb, const int32_t* cu, int n_new_total,
                         const uint16_t* k, const uint16_t* v, hipStream_t s) {
  const int n_lcall = layer < 0 ? P.n_layers : 1;
  // decode-step appends: one wave per task, as many waves as the call can have
  // tasks (every touched page receives at least one token)
  const int64_t step_waves = (int64_t)n_new_total * n_lcall * P.n_kv_heads * 2;
  if (n_new_total <= STEP_APPEND_MAX_TOKENS && n_req <= STEP_APPEND_MAX_REQ &&
      step_waves <= STEP_APPEND_MAX_WAVES) {
    const int grid = step_waves < 1 ? 1 : (int)step_waves;
    if (P.d == 256)
      hipLaunchKernelGGL(append_step_kernel<256>, dim3(grid), dim3(64), 0, s, P, layer, n_lcall,
                         n_req, bt, tags, max_pages, sb, cu, n_new_total, k, v);
    else
      hipLaunchKernelGGL(append_step_kernel<128>, dim3(grid), dim3(64), 0, s, P, layer, n_lcall,
                         n_req, bt, tags, max_pages, sb, cu, n_new_total, k, v);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(append_plan_kernel, dim3(1), dim3(1024), 0, s, n_req, bt, tags, max_pages, sb,
                     cu, P.ctrl, P.fp8_stack, P.list, P.n_fp8, n_new_total, P.rc8);
  // upper bound on listed pages: new tokens / 16 + one partial page per request
  const int64_t pages_bound = (int64_t)n_new_total / PAGE + n_req + 1;
  const int grid = grid_for((pages_bound * n_lcall * P.n_kv_heads * 2 + 3) / 4, 8192);
  if (P.d == 256)
    hipLaunchKernelGGL(append_quant_kernel<256>, dim3(grid), dim3(256), 0, s, P, layer, n_lcall, sb,
                       cu, n_new_total, k, v);
  else
    hipLaunchKernelGGL(append_quant_kernel<128>, dim3(grid), dim3(256), 0, s, P, layer, n_lcall, sb,
                       cu, n_new_total, k, v);
  return hipGetLastError();
}

hipError_t launch_migrate(const PoolView& P, int n_req, int32_t* bt, uint8_t* tags, int max_pages,
                          const uint8_t* anchor, const int32_t* seq_lens, hipStream_t s) {
  // whole batches per workgroup, at most MIG_BLOCKS workgroups
  const int64_t n_ent = (int64_t)n_req * max_pages;
  const int64_t n_bat = (n_ent + MIG_BATCH - 1) / MIG_BATCH;
  const int64_t bat_per = (n_bat + MIG_BLOCKS - 1) / MIG_BLOCKS;
  const int nb = (int)((n_bat + bat_per - 1) / bat_per);
  const int64_t per_blk = bat_per * MIG_BATCH;
  int32_t* mig = P.ctrl + ctrl_layout(P.n_fp8, P.n_tq3, P.d).mig;
  const RcView rv = {P.rc8, P.rc3, P.n_fp8, P.n_tq3};
  if (nb == 1) {
    hipLaunchKernelGGL(migrate_list_kernel<true>, dim3(1), dim3(MIG_NT), 0, s, n_req, bt, tags,
                       max_pages, anchor, seq_lens, P.recent, P.ctrl, P.tq3_stack, P.list, mig,
                       per_blk, nb, P.n_fp8, rv);
  } else {
    hipLaunchKernelGGL(migrate_count_kernel, dim3(nb), dim3(MIG_NT), 0, s, n_req, bt, tags,
                       max_pages, anchor, seq_lens, P.recent, P.ctrl, mig, per_blk, P.n_fp8, rv);
    hipLaunchKernelGGL(migrate_list_kernel<false>, dim3(nb), dim3(MIG_NT), 0, s, n_req, bt, tags,
                       max_pages, anchor, seq_lens, P.recent, P.ctrl, P.tq3_stack, P.list, mig,
                       per_blk, nb, P.n_fp8, rv);
  }
  int64_t bound = (int64_t)n_req * max_pages;
  if (bound > P.n_fp8) bound = P.n_fp8;
  const int grid = grid_for((bound * P.n_layers * P.n_kv_heads + ENC_WG / 2 - 1) / (ENC_WG / 2), 1024);
  if (P.d == 256)
    hipLaunchKernelGGL(migrate_encode_kernel<256>, dim3(grid), dim3(64 * ENC_WG), 0, s, P);
  else
    hipLaunchKernelGGL(migrate_encode_kernel<128>, dim3(grid), dim3(64 * ENC_WG), 0, s, P);
  hipLaunchKernelGGL(migrate_publish_kernel, dim3(1), dim3(1024), 0, s, bt, tags, max_pages, P.ctrl,
                     P.fp8_stack, P.list, P.rc8, P.rc3);
  return hipGetLastError();
}

hipError_t launch_promote(const PoolView& P, int n_req, int32_t* bt, uint8_t* tags, int max_pages,
                          const uint8_t* mask, const int32_t* seq_lens, hipStream_t s) {
  const auto plan = (int64_t)n_req * max_pages <= MIG_BATCH ? promote_plan_kernel<true> : promote_plan_kernel<false>;
  hipLaunchKernelGGL(plan, dim3(1), dim3(MIG_NT), 0, s, n_req, bt, tags, max_pages, mask, seq_lens, P.ctrl,
                     P.fp8_stack, P.list, P.n_tq3, RcView{P.rc8, P.rc3, P.n_fp8, P.n_tq3});
  int64_t bound = (int64_t)n_req * max_pages;
  if (bound > P.n_fp8) bound = P.n_fp8;
  if (bound > P.n_tq3) bound = P.n_tq3;
  const int grid = grid_for((bound * P.n_layers * P.n_kv_heads + ENC_WG / 2 - 1) / (ENC_WG / 2), 1024);
  if (P.d == 256)
    hipLaunchKernelGGL(promote_build_kernel<256>, dim3(grid), dim3(64 * ENC_WG), 0, s, P);
  else
    hipLaunchKernelGGL(promote_build_kernel<128>, dim3(grid), dim3(64 * ENC_WG), 0, s, P);
  hipLaunchKernelGGL(promote_publish_kernel, dim3(1), dim3(1024), 0, s, bt, tags, max_pages, P.ctrl,
                     P.tq3_stack, P.list, P.rc8, P.rc3);
  return hipGetLastError();
}

// Arithmetic conformance probe: the fp64 division, square root and binary16
// rounding of this translation unit (the ones gamma and the V scale/zero rest
// on), element by element.
__global__ __launch_bounds__(256) void fp64_probe_kernel(const double* a, const double* b, int64_t n,
                                                         double* quot, double* root,
                                                         uint16_t* half) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double x = a[i], y = b[i];
    quot[i] = x / y;
    root[i] = sqrt(x);
    half[i] = f64_to_f16_rne_sat(x);
  }
}

hipError_t launch_fp64_probe(const double* a, const double* b, int64_t n, double* quot,
                             double* root, uint16_t* half, hipStream_t s) {
  hipLaunchKernelGGL(fp64_probe_kernel, dim3(grid_for((n + 255) / 256, 4096)), dim3(256), 0, s, a, b,
                     n, quot, root, half);
  return hipGetLastError();
}

hipError_t launch_partition(int n_req, const int32_t* bt, const uint8_t* tags, int max_pages,
                            const int32_t* seq_lens, int32_t* list8, int32_t* list3,
                            int32_t* counts, int32_t* err, hipStream_t s) {
  hipLaunchKernelGGL(partition_kernel, dim3(n_req), dim3(1024), 0, s, bt, tags, max_pages, seq_lens,
                     list8, list3, counts, err);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  const int64_t words = (int64_t)(bytes / 4);
  if (words == 0) return hipSuccess;
  const int grid = grid_for((words + 255) / 256, 1024);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, s, (uint32_t*)p, words);
  return hipGetLastError();
}

}  // namespace mkv
