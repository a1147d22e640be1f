// fp32 routed attention for gfx950: the exact-precision path (small layers, 1e-5 parity).
// Inputs and outputs are fp32; everything in between is fp64, so the result is the correctly
// computed softmax(scale Q K^T) V rounded once to fp32, whatever the number of keys: a product
// of two fp32 values is exact in fp64, and the sums (head_dim terms per score, all keys per
// output element) carry fp64 rounding only.  (An all-fp32 version of this kernel drifted past
// 1e-5 from about three thousand keys on: sequential fp32 accumulation over the key stream.)
//
// Both contractions run on v_mfma_f64_16x16x4_f64 and are computed transposed, as in the bf16
// kernels:  S^T = K Q^T,  O^T += V^T P^T  -- lane (m = lane & 15, g = lane >> 4) owns query m.
// The instruction's operands are one double per lane (row or column m, k index g) and its
// accumulator register v holds row 4 v + g, so with key 4 v + g in register v the probabilities
// are already the B operand of the second product's step v.  The k index of the first product and
// the row index of the second one are permutations of the head dimension chosen so that K, V and
// O move as 16-byte pieces: step (c, i) contracts dim 16 c + 4 g + i, and accumulator row m of
// tile (h, i) is dim 64 h + 4 m + i.
//
// What bounds it: the fp64 matrix instruction (64 cycles, 77.9 TFLOP/s over the chip in a
// register-only loop) shares its execution unit with the vector ALU -- in the same loop eight
// fp32 fused multiply-adds behind each matrix instruction cost their full issue time, 32 cycles --
// so what is not a matrix instruction is paid for.  Per 16 keys x 16 queries x 128 dims that is
// 64 matrix instructions = 4,096 cycles and about 64 widenings of K and V, four exponentials and the
// addresses; counters of eight dense heads of 3,072 tokens: 3.2 other vector instructions a matrix instruction, the matrix unit
// busy in 74 % of the CU's busy cycles, at 2.18 GHz where the register-only loop has 2.38 (profiles/fp32_attention_counters.txt).  Hence no LDS staging and no running maximum: a wavefront owns 16 query rows and reads
// its K and V rows straight from L2 into operand registers (16 B/clk and CU, a quarter of what a CU's
// cache port moves), K of the next block while the softmax and the second product run, V of this block
// under the first product.  The row reference is a lagging maximum, raised only when a score exceeds it
// by more than 2^512: fp64 has the range, and the accumulators are then touched by matrix
// instructions only.
//
// Split: the NW wavefronts of a workgroup share 16 query rows and take every NW-th 16-key block;
// their (reference, sum, accumulator) triples are merged through LDS at the end, each wavefront a part of
// the channels, in a fixed order.  A
// full head of 3,072 tokens is then 192 items of 48 blocks per wavefront instead of one long
// stream per 64 rows.
//
// Measured (attention launch and whole layer; the vector-ALU kernel before it in brackets): eight dense
// heads of 3,072 tokens x 128 run at 57 TFLOP/s, 73 % of the matrix instruction's rate, without the
// exponentials at 59; the 3,072-token layer with 2 full, 3 window and 3 core-set heads 440 us
// [1,701 us], two heads of 256 tokens x 64 16 us [140 us, four of its launches reorder passes].
#include <hip/hip_runtime.h>

#include <algorithm>

#include "vorta_attn_common.h"

namespace vorta {

typedef double f64x4 __attribute__((ext_vector_type(4)));
#define MFMA64(a_, b_, c_) __builtin_amdgcn_mfma_f64_16x16x4f64(a_, b_, c_, 0, 0, 0)

template <int D, int NW>
__global__ __launch_bounds__(64 * NW, 8 / NW) void attn_f32_kernel(const AttnArgs a) {
  constexpr int BM = 16, KB = 16;            // query rows per item, keys per block
  constexpr int NC = D / 16;                 // 16-byte pieces of a K row per lane
  constexpr int NH = D / 64;                 // 16-byte pieces of a V row per lane and k step
  constexpr int NT = 4 * NH;                 // accumulator tiles of O^T
  constexpr double REF_SLACK = 512.0;        // log2 units a score may exceed the row reference by
  __shared__ double s_ref[NW][BM], s_sum[NW][BM];
  __shared__ f64x4 s_acc[NW][NT][64];
  read_together(a);
  const WorkItem w = decode_item<BM, D>(a, blockIdx.x);
  if (w.n_rows <= 0) return;       // q-block past the end of a clipped tile
  // window heads without tile-ordered copies: rows of the caller's tensors through the tile permutation
  const bool gather = w.seg == 2 && a.win_gather;
  const float* Q = (const float*)(w.seg == 0 || gather ? a.q0 : w.seg == 1 ? a.qc : a.qt) + w.q_off;
  const float* K = (const float*)(w.seg == 0 || gather ? a.k0 : w.seg == 1 ? a.kc : a.kt) + w.kv_off;
  const float* V = (const float*)(w.seg == 0 || gather ? a.v0 : w.seg == 1 ? a.vc : a.vt) + w.kv_off;
  const bool unpool = w.seg == 1 && a.keep_idx;
  float* O = unpool ? (float*)a.o0 + a.core_heads[w.head] * a.head_stride0
                    : (float*)(w.seg == 0 || gather ? a.o0 : w.seg == 1 ? a.oc : a.ot) + w.o_off;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int m = lane & 15, g = lane >> 4;

  // rows are addressed by their element offset: row times stride is below 2^31, checked on the host
  auto row_off = [&](int row) { return (unsigned)row * (unsigned)w.row_stride; };
  unsigned my_off;
  {
    int row = w.row0 + min(m, w.n_rows - 1);
    if (gather) row = a.tok_of[row];
    my_off = row_off(row);
  }
  // scores come out in log2 units: scale and log2(e) go into Q (fp64: a rounding of 2^-53)
  double q[4 * NC];
  {
    const double qs = (double)a.scale * 1.4426950408889634074;
    const float* qp = Q + my_off + 4 * g;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const float4 x = *(const float4*)(qp + 16 * c);
      q[4 * c] = (double)x.x * qs; q[4 * c + 1] = (double)x.y * qs;
      q[4 * c + 2] = (double)x.z * qs; q[4 * c + 3] = (double)x.w * qs;
    }
  }

  const RunList rl(w);
  int n_keys = 0;
  for (int r = 0; r < w.n_runs; ++r) n_keys += rl.len(r);
  // cursor of this wavefront's next block: run, keys into it, its first row and length
  int fr = 0, fpos = 0, fstart = rl.start(0), flen = rl.len(0);
  auto advance = [&](int keys) {
    fpos += keys;
    while (fpos >= flen && fr + 1 < w.n_runs) {
      fpos -= flen;
      ++fr;
      fstart = rl.start(fr);
      flen = rl.len(fr);
    }
  };
  unsigned koff = 0;               // row offset of key m of the block
  float4 kf[NC];
  auto load_k = [&]() {            // rows of the block under the cursor, then on to this wavefront's next one
    int key[1] = {m}, rows[1];
    block_rows(rl, fr, fpos, fstart, flen, KB, key, rows);
    koff = row_off(gather ? a.tok_of[rows[0]] : rows[0]);
    const float* kp = K + koff + 4 * g;
#pragma unroll
    for (int c = 0; c < NC; ++c) kf[c] = *(const float4*)(kp + 16 * c);
    advance(NW * KB);
  };

  f64x4 o[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) o[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  double ref = -INFINITY, sum = 0.0;         // row reference of query m, this lane's share of the row sum

  int left = n_keys - KB * wave;             // keys from this wavefront's next block on
  advance(KB * wave);
  if (left > 0) load_k();
  for (; left > 0; left -= NW * KB) {
    float4 vf[4][NH];                        // V rows of keys 4 v + g
    unsigned voff[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) voff[v] = __shfl(koff, 4 * v + g, 64);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float* vp = V + voff[v] + 4 * m;
#pragma unroll
      for (int h = 0; h < NH; ++h) vf[v][h] = *(const float4*)(vp + 64 * h);
    }
    f64x4 s = {0.0, 0.0, 0.0, 0.0}, s2 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      s = MFMA64((double)kf[c].x, q[4 * c], s);
      s2 = MFMA64((double)kf[c].y, q[4 * c + 1], s2);
      s = MFMA64((double)kf[c].z, q[4 * c + 2], s);
      s2 = MFMA64((double)kf[c].w, q[4 * c + 3], s2);
    }
    s += s2;
    if (left < KB) {                         // last block: register v is key 4 v + g
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (4 * v + g >= left) s[v] = -INFINITY;
    }
    if (left > NW * KB) load_k();            // rows of the next block arrive under the softmax and the second product

    double mx = fmax(fmax(s[0], s[1]), fmax(s[2], s[3]));
    if (__any(mx - ref > REF_SLACK)) {       // always for the first block
      mx = fmax(mx, __shfl_xor(mx, 16, 64));
      mx = fmax(mx, __shfl_xor(mx, 32, 64));
      const double ref_new = fmax(ref, mx);
      const double alpha = ref == ref_new ? 1.0 : exp2(ref - ref_new);   // 0 for the first block
      ref = ref_new;
      sum *= alpha;
#pragma unroll
      for (int t = 0; t < NT; ++t) o[t] *= alpha;
    }
    const double base = ref == -INFINITY ? 0.0 : ref;    // only scores of -inf so far: probabilities 0
    f64x4 p;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      p[v] = exp2(s[v] - base);
      sum += p[v];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        o[4 * h] = MFMA64((double)vf[v][h].x, p[v], o[4 * h]);
        o[4 * h + 1] = MFMA64((double)vf[v][h].y, p[v], o[4 * h + 1]);
        o[4 * h + 2] = MFMA64((double)vf[v][h].z, p[v], o[4 * h + 2]);
        o[4 * h + 3] = MFMA64((double)vf[v][h].w, p[v], o[4 * h + 3]);
      }
  }

  // ---- merge of the NW shares of the key stream: a wavefront sums and stores every NW-th 16-byte piece of the rows.  What
  // others sum goes through LDS with the references and sums, unscaled, so that one barrier does.  (A tree of additions, the first
  // wavefront storing: 3 heads of 1,024 tokens x 64 32.1 -> 31.3 us, one dense head of 3,072 x 128 121.6 -> 119.9.)
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  if (g == 0) {
    s_ref[wave][m] = ref;
    s_sum[wave][m] = sum;
  }
  // piece u = 4 h + v: register v of the four tiles of channels 64 h on
  auto piece = [&](int u) { return f64x4{o[u & ~3][u & 3], o[(u & ~3) + 1][u & 3], o[(u & ~3) + 2][u & 3], o[(u & ~3) + 3][u & 3]}; };
#pragma unroll
  for (int u = 0; u < NT; ++u)
    if (u % NW != wave) s_acc[wave][u][lane] = piece(u);
  __syncthreads();
  if (wave >= NT || m >= w.n_rows) return;
  double top = -INFINITY, total = 0.0, weight[NW];
#pragma unroll
  for (int i = 0; i < NW; ++i) top = fmax(top, s_ref[i][m]);
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const double r = s_ref[i][m];
    weight[i] = r == -INFINITY ? 0.0 : exp2(r - top);
    total += s_sum[i][m] * weight[i];
  }
  const double inv = 1.0 / total;
  constexpr int MINE = (NT + NW - 1) / NW;
  float4 out[MINE];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    if (u % NW != wave) continue;
    f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < NW; ++i) x += (i == wave ? piece(u) : s_acc[i][u][lane]) * weight[i];
    out[u / NW] = make_float4((float)(x[0] * inv), (float)(x[1] * inv), (float)(x[2] * inv), (float)(x[3] * inv));
  }
  {
    auto store = [&](unsigned off) {
      float* op = O + off + 4 * g;
#pragma unroll
      for (int j = 0; j < MINE; ++j) {
        const int u = NW * j + wave;
        *(float4*)(op + 64 * (u / 4) + 16 * (u % 4)) = out[j];
      }
    };
    if (!unpool) {
      store(my_off);
    } else {                                   // to every token that reads this slot
      const unsigned stride = (unsigned)a.row_stride0;
      const int slot = w.row0 + m;
      if (slot >= a.Lc) {
        store((unsigned)(a.L + slot - a.Lc) * stride);
      } else {
        const int tok = a.keep_idx[(long)w.head * a.Lc + slot];
        const int2 bucket = a.slot_bucket[slot];
        store((unsigned)tok * stride);
        if (tok == bucket.x)                   // the bucket's centre: the tokens pruned into it.  Each is looked up by one of the row's four
          // lanes, 16 in one memory latency (four by every lane: one head of 750 tokens 18.7 -> 17.2 us, 8 of 5,200 128 -> 121)
          for (int j0 = 0; j0 < a.bucket_max; j0 += 16) {
            int t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              t[u] = slot_bucket_token(a, bucket, j0 + 4 * u + g);
              if (t[u] == tok || (t[u] >= 0 && a.assign[(long)w.head * a.L + t[u]] != slot)) t[u] = -1;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
              for (int from = 0; from < 4; ++from) {
                const int to = __shfl(t[u], 16 * from + m, 64);
                if (to >= 0) store((unsigned)to * stride);
              }
          }
      }
    }
  }
}

// Wavefronts of a workgroup.  Four let two workgroups share a CU; with no more items than CUs the second one is missing, and
// eight hide more of the latency if the longest item's key stream pays for the longer merge.  340 layers of 196 to 4,056 tokens, 1 to 8
// heads, each timed both ways: from 32 key blocks on eight are 2 to 11 % faster (3,456 keys 167 -> 135 us, 1,120 keys 56.0 -> 53.4, 588
// keys level), with fewer 1 to 11 % slower (two heads of 256 tokens 16.9 -> 17.6 us).  They also keep a CU for themselves, where four
// wavefronts of two items now and then meet on one CU although others are idle (3 heads of 802 tokens 45 us, 69 then).  With
// more items than CUs four are faster by 5 to 12 % more often than not.  The choice is 0.5 to 1.2 % slower than the faster of the two on average; by
// the number of rows (1,024 and more, as the tree of additions at the end of an item had it) it was 0.7 to 2.8 %.
static int f32_wavefronts(const vorta_plan* p, const RouteLists& rl, const AttnArgs& a, int units) {
  int keys = 0;
  if (rl.count[0] || (rl.count[1] && a.n_text)) keys = a.N;
  if (rl.count[1]) keys = std::max(keys, p->win_most_keys);
  if (rl.count[2]) keys = std::max(keys, a.Nc);
  return a.end_tile <= units && (keys + 15) / 16 >= 32 ? 8 : 4;
}

int launch_attention_f32(vorta_plan* p, const RouteLists& rl, const vorta_attn_io* io, const CoreIndex* core, void* stream) {
  AttnArgs a;
  if (int rc = fill_attn_args(p, rl, io, core, 16, WIN_ALL, &a)) return rc;
  if (a.end_tile == 0) return VORTA_OK;
  const dim3 grid(a.end_tile);
  hipStream_t st = (hipStream_t)stream;
  const bool few = f32_wavefronts(p, rl, a, p->n_cus) == 8;
  if (p->d.head_dim == 64) {
    if (few) hipLaunchKernelGGL((attn_f32_kernel<64, 8>), grid, dim3(512), 0, st, a);
    else hipLaunchKernelGGL((attn_f32_kernel<64, 4>), grid, dim3(256), 0, st, a);
  } else {
    if (few) hipLaunchKernelGGL((attn_f32_kernel<128, 8>), grid, dim3(512), 0, st, a);
    else hipLaunchKernelGGL((attn_f32_kernel<128, 4>), grid, dim3(256), 0, st, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(VORTA_EHIP, "launch of attn_f32_kernel: %s", hipGetErrorString(e));
  return VORTA_OK;
}

}  // namespace vorta

// For the tests, not part of the ABI: wavefronts of a workgroup of an fp32 layer call with these routes on a device of `units` CUs.
extern "C" int vorta_test_f32_wavefronts(vorta_plan* p, const uint8_t* routes_host, int32_t units, int32_t* out) {
  using namespace vorta;
  RouteLists rl;
  if (int rc = split_routes(p, routes_host, &rl)) return rc;
  AttnArgs a;
  const vorta_attn_io io = {};
  if (int rc = fill_attn_args(p, rl, &io, nullptr, 16, WIN_ALL, &a)) return rc;
  *out = f32_wavefronts(p, rl, a, units);
  return VORTA_OK;
}
