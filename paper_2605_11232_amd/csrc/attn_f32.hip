// float32 paged attention, the exact-precision path for float32 caches: row
// tiles on the float32 matrix instruction, and one wavefront per (token, head)
// for many short sequences of one or two rows.
//
// Same definition as the bf16 path (paper: Section 2 PagedAttention / APC;
// Section 3, cached prefixes give the recomputed result): causal softmax over
// keys 0..a of the request's logical sequence, read through its block table.
// All arithmetic is float32 with fused multiply-adds (v_mfma_f32_16x16x4_f32 multiplies and
// accumulates in float32); exp/log are the device library's float32 functions.
//
// Row tiles: a workgroup computes 16 NC rows ((query, head-in-group) pairs of one
// sequence and kv-head, so all of them read the same keys); its wavefronts
// take the sequence's 16-key blocks in turn, each with its own running
// softmax, and combine through LDS at the end.  Both products run on operands
// as the cache holds them, 16 bytes per lane straight from memory: the score
// tile is computed transposed (S^T = K Q^T), so a lane's four scores are four
// keys of one query row, which is the layout of the B operand of
// O^T += V^T P^T.  No key, value or probability goes through LDS.
//
// Bound: the float32 matrix rate.  A block of 16 keys costs a wavefront
// 64 NC instructions of 32 cycles (D = 128) against 16 KB of loads, so loads
// one block ahead and two or three wavefronts per SIMD cover the memory
// latency; what is left is each workgroup's start (sequence, table, keys: a
// chain of loads), its combine and the last wave of workgroups (1.4 of 2
// wavefronts resident on average, matrix units busy 49 % of the call).
// Append and attention, 8 requests of 64-256 new tokens on 512 cached ones,
// 32/8 heads of 128: 0.163 ms (80 TFLOP/s), against 2.0 ms with one wavefront
// per (token, head) on vector instructions; 4 requests of 32-64 tokens, 8/2
// heads of 64, alone: 30 us against 41.
#include <hip/hip_ext.h>

#include "device_common.h"
#include "plan_format.h"

namespace pa {
namespace dev {
namespace {

constexpr int W = 4;  // wavefronts of a workgroup

// q, out: any 4-byte aligned address
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bool is_finite(float x) { return fabsf(x) < __builtin_huge_valf(); }

// max over the four lane groups (lanes l, l ^ 16, l ^ 32, l ^ 48)
__device__ __forceinline__ float max_groups(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Tiles of R rows: sequence r's first tile has index first_tile(r), at least
// cdiv(rows of r, R) below first_tile(r + 1); the excess tiles are empty.
template <int R>
__device__ __forceinline__ uint32_t first_tile(int cu, int G, int r) {
  return uint32_t(cu) * uint32_t(G) / R + uint32_t(r);
}

template <int D, int NC>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2))) void attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ kc, const float* __restrict__ vc,
    const int32_t* __restrict__ bt, int32_t max_blocks, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ cu_q, int32_t n_seqs, int32_t hq, int32_t hkv, int32_t num_blocks,
    float scale, float* __restrict__ out, float* __restrict__ lse) {
  constexpr int R = 16 * NC;  // rows per workgroup
  constexpr int CH = NC == 2 && D == 128 ? 2 : 4;  // as the registers allow
  constexpr int DT = D / 16;  // 16-dim pieces: 16-byte loads per lane, for each of K and V^T
  // + 4: the rows of a store fall in different banks
  __shared__ float acc_sh[W][R][D + 4];
  __shared__ float m_sh[W][R], l_sh[W][R];
  __shared__ int odd_sh[W];
  const int lane = threadIdx.x & 63, j = lane & 15, g4 = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = hq / hkv;
  // kv-heads innermost (a head's workgroups share an XCD's L2 when there are
  // eight), a sequence's last, longest tiles first
  const int g = blockIdx.x % hkv;
  const uint32_t tile = gridDim.x / hkv - 1 - blockIdx.x / hkv;
  // sequence of the tile: the last r with first_tile(r) <= tile, 64 probes a round
  int lo = 0, hi = n_seqs;
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) / 64, i = lo + lane * step;
    const bool le = i < hi && first_tile<R>(cu_q[i < hi ? i : lo], G, i) <= tile;
    lo += (__popcll(__ballot(le)) - 1) * step;
    hi = min(hi, lo + step);
  }
  const int r = __builtin_amdgcn_readfirstlane(lo);
  const int qs = cu_q[r], n = cu_q[r + 1] - qs, L = seq_lens[r];
  const int row0 = int(tile - first_tile<R>(qs, G, r)) * R;
  const int nrows = min(R, n * G - row0);
  if (nrows <= 0) return;  // an empty tile

  // column j of 16-row tile c is row 16 c + j
  bool valid[NC];
  int apos[NC];  // the row's position: keys 0..apos are visible
  int64_t orow[NC];
  f32x4 qf[NC][DT];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int rho = row0 + 16 * c + j, qi = rho / G;
    valid[c] = 16 * c + j < nrows;
    apos[c] = valid[c] ? L - n + qi : -1;
    orow[c] = (int64_t)(qs + qi) * hq + g * G + (rho - qi * G);
    // dims 16 i + 4 g4 .. + 3
#pragma unroll
    for (int i = 0; i < DT; ++i)
      qf[c][i] = valid[c] ? f32x4(*reinterpret_cast<const f32x4u*>(q + orow[c] * D + 16 * i + 4 * g4))
                          : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int amin = L - n + row0 / G;                // first row's position
  const int amax = L - n + (row0 + nrows - 1) / G;  // last row's
  const int nblk = amax / kBlock + 1;

  // Row p of a block's score tile is slot position p; lane group g4 holds
  // positions 4 g4 .. + 3, which are offsets voff .. + 3 (bits 2 and 3 swapped).
  const int voff = key_slot_pos(4 * g4);
  const int32_t* row = bt + (int64_t)r * max_blocks;
  // this wavefront's blocks w, w + W, ..: 64 table entries at a time, clamped,
  // one per lane
  auto fetch_ids = [&](int it0) {
    const int b = w + W * (it0 + lane);
    return clamp_block(row[min(min(b, nblk - 1), max_blocks - 1)], num_blocks);
  };
  f32x4 kreg[DT], vreg[DT];
  auto load_k = [&](int id) {
    const float* p = kc + ((int64_t)id * hkv + g) * (kBlock * D) + j * kKeyGroup + 4 * g4;
#pragma unroll
    for (int i = 0; i < DT; ++i)
      kreg[i] = *reinterpret_cast<const f32x4*>(p + (i / 2) * (kBlock * kKeyGroup) + (i % 2) * 16);
  };
  auto load_v = [&](int id) {
    const float* p = vc + ((int64_t)id * hkv + g) * (kBlock * D) + j * kBlock + voff;
#pragma unroll
    for (int i = 0; i < DT; ++i) vreg[i] = *reinterpret_cast<const f32x4*>(p + 16 * kBlock * i);
  };

  f32x4 acc[NC][DT];
  float m[NC], l[NC];
  bool odd = false;  // this lane left out a value that is not finite
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    m[c] = kNegInf;
    l[c] = 0.f;
#pragma unroll
    for (int i = 0; i < DT; ++i) acc[c][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  int ids = fetch_ids(0);
  int next = __builtin_amdgcn_readlane(ids, 0);
  if (w < nblk) {
    load_k(next);
    load_v(next);
  }
  for (int blk = w, it = 0; blk < nblk; blk += W, ++it) {
    const bool more = blk + W < nblk;
    // past the last block: that block again (fetch_ids)
    if (((it + 1) & 63) == 0) ids = fetch_ids(it + 1);
    next = __builtin_amdgcn_readlane(ids, (it + 1) & 63);
    // scores, CH partial sums over the dims
    f32x4 sp[NC][CH];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < CH; ++e) sp[c][e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < NC; ++c) sp[c][e % CH] = mfma_f32(kreg[i][e], qf[c][i][e], sp[c][e % CH]);
    // Unconditional, so that the values' wait below does not wait for these
    // loads too (the last block's keys are read once more).
    load_k(next);
    const int key0 = blk * kBlock + voff;  // the key of this lane's element 0
    const bool masked = blk * kBlock + kBlock - 1 > amin;  // wave-uniform
    f32x4 p[NC];
    float mx[NC];
    bool higher = false;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      f32x4 s = sp[c][0] + sp[c][1];
      if constexpr (CH == 4) s += sp[c][2] + sp[c][3];
      s *= scale;
#pragma unroll
      for (int e = 0; e < 4; ++e) p[c][e] = key0 + e <= apos[c] ? s[e] : kNegInf;
      mx[c] = max_groups(fmaxf(fmaxf(p[c][0], p[c][1]), fmaxf(p[c][2], p[c][3])));
      higher = higher || mx[c] > m[c];
    }
    if (__any(higher)) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const float mnew = fmaxf(m[c], mx[c]);
        const float alpha = m[c] == kNegInf ? 0.f : expf(m[c] - mnew);
        l[c] *= alpha;
#pragma unroll
        for (int i = 0; i < DT; ++i) acc[c][i] *= alpha;
        m[c] = mnew;
      }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const float ref = m[c] == kNegInf ? 0.f : m[c];
#pragma unroll
      for (int e = 0; e < 4; ++e) p[c][e] = expf(p[c][e] - ref);
      l[c] += (p[c][0] + p[c][1]) + (p[c][2] + p[c][3]);
    }
    if (masked) {
      // Values past the last visible key may never have been written: zero.  A
      // visible value that is not finite would reach rows that must not see
      // it (0 * inf): it is left out here and added row by row at the end.
#pragma unroll
      for (int i = 0; i < DT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in = key0 + e <= amax, fin = is_finite(vreg[i][e]);
          odd = odd || (in && !fin);
          vreg[i][e] = in && fin ? vreg[i][e] : 0.f;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < DT; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c][i] = mfma_f32(vreg[i][e], p[c][e], acc[c][i]);
    if (!more) break;
    load_v(next);
  }

  // combine the wavefronts' parts
  const bool any_odd = __any(odd);
  if (lane == 0) odd_sh[w] = any_odd;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    l[c] += wave_xor(l[c], 16);
    l[c] += wave_xor(l[c], 32);
#pragma unroll
    for (int i = 0; i < DT; ++i)
      *reinterpret_cast<f32x4*>(&acc_sh[w][16 * c + j][16 * i + 4 * g4]) = acc[c][i];
    if (g4 == 0) {
      m_sh[w][16 * c + j] = m[c];
      l_sh[w][16 * c + j] = l[c];
    }
  }
  __syncthreads();
  for (int u = threadIdx.x; u < nrows * (D / 4); u += 64 * W) {
    const int rr = u / (D / 4), d = u % (D / 4) * 4;
    float mm = m_sh[0][rr];
#pragma unroll
    for (int x = 1; x < W; ++x) mm = fmaxf(mm, m_sh[x][rr]);
    float ls = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < W; ++x) {
      const float f = m_sh[x][rr] == kNegInf ? 0.f : expf(m_sh[x][rr] - mm);
      ls = fmaf(f, l_sh[x][rr], ls);
      const f32x4 a = *reinterpret_cast<const f32x4*>(&acc_sh[x][rr][d]);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = fmaf(f, a[e], o[e]);
    }
    const int rho = row0 + rr, qi = rho / G;
    const int64_t at = (int64_t)(qs + qi) * hq + g * G + (rho - qi * G);
    int left_out = 0;
#pragma unroll
    for (int x = 0; x < W; ++x) left_out |= odd_sh[x];
    if (left_out) {
      // the masked blocks' visible values that are not finite
      for (int key = (amin + 1) / kBlock * kBlock; key <= L - n + qi; ++key) {
        const int off = key % kBlock;
        const int64_t at_blk =
            ((int64_t)clamp_block(row[min(key / kBlock, max_blocks - 1)], num_blocks) * hkv + g) * (kBlock * D);
        float v[4], s = 0.f;
        bool fin = true;
        for (int e = 0; e < 4; ++e) {
          v[e] = vc[at_blk + (d + e) * kBlock + off];
          fin = fin && is_finite(v[e]);
        }
        if (fin) continue;
        for (int x = 0; x < D; ++x) s = fmaf(q[at * D + x], kc[at_blk + key_elem(off, x)], s);
        const float p = expf(s * scale - mm);
        for (int e = 0; e < 4; ++e) o[e] += is_finite(v[e]) ? 0.f : p * v[e];
      }
    }
    *reinterpret_cast<f32x4u*>(out + at * D + d) = o * (1.f / ls);
    if (lse && d == 0) lse[at] = mm + logf(ls);
  }
}

template <int D, int NC>
void launch_t(hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop, const float* q,
              const float* kc, const float* vc, const int32_t* bt, int32_t max_blocks,
              const int32_t* seq_lens, const int32_t* cu_q, int32_t n_seqs, int32_t total_q,
              int32_t hq, int32_t hkv, int32_t num_blocks, float scale, float* out, float* lse) {
  const int64_t grid = f32_tile_grid(total_q, n_seqs, hq, hkv);
  // the caller's timing events ride on the dispatch (no event packets)
  hipExtLaunchKernelGGL((attn_f32_kernel<D, NC>), dim3(static_cast<unsigned>(grid)),
                        dim3(64 * W), 0, stream, ev_start, ev_stop, 0, q, kc, vc, bt,
                        max_blocks, seq_lens, cu_q, n_seqs, hq, hkv, num_blocks, scale, out, lse);
}

// One wavefront per (query token, q-head), on vector instructions: a 64-key
// chunk puts one key in each lane for the scores (16-byte loads of the key's
// 32-dim runs, eight partial sums), then the lanes switch to owning head
// dimensions for the weighted value sum: each lane reads one dimension's 16
// offsets of a block as four 16-byte loads and takes the probabilities from
// LDS, in four partial sums.  A workgroup of the tile kernel costs about as much for
// one row as for sixteen, and a chain of loads before its first key; where
// sequences have one row or two and few keys, that is most of it.  The planner
// chooses (f32_by_row).
template <int D>
__global__ __launch_bounds__(64) void attn_f32_row_kernel(
    const float* __restrict__ q, const float* __restrict__ kc, const float* __restrict__ vc,
    const int32_t* __restrict__ bt, int32_t max_blocks, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ cu_q, int32_t n_seqs, int32_t hq, int32_t hkv, int32_t num_blocks,
    float scale, float* __restrict__ out, float* __restrict__ lse) {
  constexpr int DL = D / 64;  // value dimensions per lane
  static_assert(D % 64 == 0, "head_dim 64 or 128");
  __shared__ float qsh[D];
  __shared__ float psh[64];
  __shared__ int bsh[64 / kBlock];
  const int token = blockIdx.x / hq, h = blockIdx.x % hq;
  const int lane = threadIdx.x;
  // sequence r: the last r with cu_q[r] <= token (empty sequences are skipped)
  int lo = 0, hi = n_seqs;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu_q[mid] <= token) lo = mid; else hi = mid;
  }
  const int r = lo;
  const int L = seq_lens[r];
  const int n = cu_q[r + 1] - cu_q[r];
  const int a = L - n + (token - cu_q[r]);
  const int g = h / (hq / hkv);
  const int32_t* row = bt + (int64_t)r * max_blocks;
  for (int d = lane; d < D; d += 64) qsh[d] = q[((int64_t)token * hq + h) * D + d];
  __syncthreads();

  float od[DL][4];  // sums over every fourth key
#pragma unroll
  for (int k = 0; k < DL; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) od[k][e] = 0.f;
  float m = kNegInf, l = 0.f;
  for (int c0 = 0; c0 <= a; c0 += 64) {
    const int key = c0 + lane;
    const bool vis = key <= a;
    // every lane's block id is a clamped table entry, so each address below
    // is inside the cache
    const int blk = clamp_block(row[min(key / kBlock, max_blocks - 1)], num_blocks);
    float s = kNegInf;
    if (vis) {
      // the key's 32-dim runs in the grouped key layout, 32 floats each
      const float* kp = kc + ((int64_t)blk * hkv + g) * kBlock * D + key_elem(key % kBlock, 0);
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int gd = 0; gd < D; gd += kKeyGroup) {
        const f32x4* k4 = reinterpret_cast<const f32x4*>(kp + gd * kBlock);
#pragma unroll
        for (int j = 0; j < kKeyGroup / 4; ++j) {
          const f32x4 kv = k4[j];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[j % 8] = fmaf(qsh[gd + 4 * j + e], kv[e], acc[j % 8]);
        }
      }
      s = (((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]))) * scale;
    }
    float cm = s;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cm = fmaxf(cm, __shfl_xor(cm, o, 64));
    const float mnew = fmaxf(m, cm);
    const float alpha = m == kNegInf ? 0.f : expf(m - mnew);
    const float p = vis ? expf(s - mnew) : 0.f;
    float ps = p;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) ps += __shfl_xor(ps, o, 64);
    l = l * alpha + ps;
    m = mnew;
#pragma unroll
    for (int k = 0; k < DL; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) od[k][e] *= alpha;
    psh[lane] = p;
    if (lane % kBlock == 0) bsh[lane / kBlock] = blk;
    __syncthreads();
    // keys c0 .. c0 + nk - 1 are visible; the chunk starts on a block boundary
    const int nk = min(64, a + 1 - c0);
    for (int b = 0; b * kBlock < nk; ++b) {
      const float* vb = vc + ((int64_t)bsh[b] * hkv + g) * D * kBlock;
      const int kb = b * kBlock, nb = min(kBlock, nk - kb);
#pragma unroll
      for (int k = 0; k < DL; ++k) {
        const f32x4* v4 = reinterpret_cast<const f32x4*>(vb + (lane + 64 * k) * kBlock);
        f32x4 vv[kBlock / 4];
#pragma unroll
        for (int j = 0; j < kBlock / 4; ++j) vv[j] = v4[j];
        if (nb == kBlock) {
#pragma unroll
          for (int j = 0; j < kBlock; ++j) od[k][j % 4] = fmaf(psh[kb + j], vv[j / 4][j % 4], od[k][j % 4]);
        } else {
          // keys past the last visible one: slots that may never have been written
#pragma unroll
          for (int j = 0; j < kBlock; ++j)
            if (j < nb) od[k][j % 4] = fmaf(psh[kb + j], vv[j / 4][j % 4], od[k][j % 4]);
        }
      }
    }
    __syncthreads();  // psh and bsh are rewritten by the next chunk
  }
  const float inv = 1.f / l;
#pragma unroll
  for (int k = 0; k < DL; ++k)
    out[((int64_t)token * hq + h) * D + lane + 64 * k] = ((od[k][0] + od[k][1]) + (od[k][2] + od[k][3])) * inv;
  if (lse && lane == 0) lse[(int64_t)token * hq + h] = m + logf(l);
}

}  // namespace

int launch_attn_f32(const void* q, const void* kc, const void* vc, int32_t num_blocks,
                    const int32_t* bt, int32_t max_blocks, const int32_t* seq_lens,
                    const int32_t* cu_q, int32_t n_seqs, int32_t total_q, int32_t hq, int32_t hkv,
                    int32_t d, bool by_row, float scale, void* out, float* lse,
                    hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (total_q == 0 || n_seqs == 0) {
    // nothing launched: the events still mark this point of the stream
    for (hipEvent_t ev : {ev_start, ev_stop}) {
      const hipError_t e = ev ? hipEventRecord(ev, stream) : hipSuccess;
      if (e != hipSuccess) return static_cast<int>(e);
    }
    return 0;
  }
  if (by_row) {
    const int64_t grid = int64_t(total_q) * hq;
    auto row = d == 128 ? attn_f32_row_kernel<128> : attn_f32_row_kernel<64>;
    hipExtLaunchKernelGGL(row, dim3(static_cast<unsigned>(grid)), dim3(64), 0, stream, ev_start,
                          ev_stop, 0, static_cast<const float*>(q), static_cast<const float*>(kc),
                          static_cast<const float*>(vc), bt, max_blocks, seq_lens, cu_q, n_seqs,
                          hq, hkv, num_blocks, scale, static_cast<float*>(out), lse);
    return static_cast<int>(hipGetLastError());
  }
  const bool wide = f32_wide_tiles(total_q, n_seqs, hq, hkv);
  auto launch = d == 128 ? (wide ? launch_t<128, 2> : launch_t<128, 1>)
                         : (wide ? launch_t<64, 2> : launch_t<64, 1>);
  launch(stream, ev_start, ev_stop, static_cast<const float*>(q), static_cast<const float*>(kc),
         static_cast<const float*>(vc), bt, max_blocks, seq_lens, cu_q, n_seqs, total_q, hq, hkv,
         num_blocks, scale, static_cast<float*>(out), lse);
  return static_cast<int>(hipGetLastError());
}

}  // namespace dev
}  // namespace pa
