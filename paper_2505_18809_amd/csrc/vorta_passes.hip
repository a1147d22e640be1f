// Memory-bound passes of the routed attention layer for gfx950: token reorder to / from
// 3-D tile order, bucketed core-set selection (index build), pool / merge, unpool, and the
// gate-weighted blend of Eq. 5.  All of them move 16-byte chunks of token rows (a 256-byte
// bf16 row of head_dim 128 is one fully coalesced segment whatever order rows are visited in);
// the index arithmetic is done once per row chunk and amortised over the heads of a route.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <new>
#include <type_traits>

#include "vorta_internal.h"

namespace vorta {

#define VORTA_HIP(call)                                                                    \
  do {                                                                                     \
    hipError_t e_ = (call);                                                                \
    if (e_ != hipSuccess) return fail(VORTA_EHIP, "%s: %s", #call, hipGetErrorString(e_)); \
  } while (0)

static int launch_status(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(VORTA_EHIP, "launch of %s: %s", what, hipGetErrorString(e));
  return VORTA_OK;
}

static void release_device_tables(vorta_plan* p) {
  if (p->d_tables) (void)hipFree(p->d_tables);
  p->d_tables = nullptr;
}
// vorta_plan_destroy lives with the host code; it frees the device tables through this hook
static const bool release_hook_set = (g_release_device_tables = release_device_tables, true);

// All tables of the plan in one allocation and one copy, each 256-byte aligned.  The tables that exist on the
// device only are written where they lie in the image that is copied (1,048,576 tokens: 6.4 -> 2.0 ms), and only the
// tables that the kernels of the plan's type read are among them (75,600 tokens: bf16 183 -> 141 us, fp32 182 -> 72).
static int upload_device_tables(vorta_plan* p, int dev) {
  struct Table {
    const void* host;      // null: device only
    size_t bytes;
    void** slot;
    size_t at;
  };
  auto table = [](const auto& v, auto** slot) { return Table{v.data(), v.size() * sizeof(v[0]), (void**)slot, 0}; };
  auto made = [](int64_t n, int32_t** slot) { return Table{nullptr, (size_t)n * sizeof(int32_t), (void**)slot, 0}; };
  const bool bf16 = p->d.dtype == VORTA_BF16;      // the attention kernels of the two types read different tables
  const std::vector<int32_t> none;
  const auto &runs = bf16 ? none : p->runs, &n_runs = bf16 ? none : p->n_runs;
  Table tables[] = {made(p->N, &p->d_tok_of), made(bf16 ? p->N : 0, &p->d_row_of), made(bf16 ? p->L : 0, &p->d_win_rows),
                    made(bf16 ? p->L : 0, &p->d_win_tok), made(2 * p->Lc, &p->d_slot_bucket),
                    table(runs, &p->d_runs), table(n_runs, &p->d_n_runs), table(p->slot_base, &p->d_slot_base),
                    table(p->tile_row0, &p->d_tile_row0), table(p->win_list[0], &p->d_win_list[0]),
                    table(p->win_list[1], &p->d_win_list[1]), table(p->win_list[2], &p->d_win_list[2]),
                    table(p->win_list[3], &p->d_win_list[3]), table(p->win_keys, &p->d_win_keys),
                    table(p->rope_cs, &p->d_rope_cs)};
  size_t total = 0;
  for (Table& t : tables) {
    t.at = total;
    total += (t.bytes + 255) & ~(size_t)255;
  }
  const std::unique_ptr<char[]> image(new (std::nothrow) char[total]);
  if (!image) return fail(VORTA_EHIP, "no host memory for %zu bytes of tables", total);
  auto place = [&](int i) { return (int32_t*)(image.get() + tables[i].at); };
  int32_t *tok_of = place(0), *row_of = place(1), *win_rows = place(2), *win_tok = place(3), *slot_bucket = place(4);
  // the inverse tile permutation; text rows keep their place
  const vorta_layer_desc& d = p->d;
  int32_t* row = tok_of;
  for (int f0 = 0; f0 < d.F; f0 += d.tile[0])
    for (int h0 = 0; h0 < d.H; h0 += d.tile[1])
      for (int w0 = 0; w0 < d.W; w0 += d.tile[2])
        for (int f = f0; f < std::min(f0 + d.tile[0], d.F); ++f)
          for (int h = h0; h < std::min(h0 + d.tile[1], d.H); ++h) {
            const int32_t first = (f * d.H + h) * d.W + w0, n = std::min(d.tile[2], d.W - w0), r = (int32_t)(row - tok_of);
            for (int32_t i = 0; i < n; ++i) *row++ = first + i;
            for (int32_t i = 0; bf16 && i < n; ++i) row_of[first + i] = r + i;
          }
  for (int64_t i = p->L; i < p->N; ++i) tok_of[i] = (int32_t)i;
  if (bf16) {
    for (int64_t i = p->L; i < p->N; ++i) row_of[i] = (int32_t)i;
    for (int32_t t : p->win_tiles)
      for (int32_t r = p->tile_row0[t]; r < p->tile_row0[t + 1]; ++r) {
        *win_rows++ = r;
        *win_tok++ = tok_of[r];
      }
  }
  const int32_t* base = p->slot_base.data();
  for (int f0 = 0; f0 < d.F; f0 += d.bucket[0])
    for (int h0 = 0; h0 < d.H; h0 += d.bucket[1])
      for (int w0 = 0; w0 < d.W; w0 += d.bucket[2], ++base) {
        const int df = std::min(d.bucket[0], d.F - f0), dh = std::min(d.bucket[1], d.H - h0), dw = std::min(d.bucket[2], d.W - w0);
        const int32_t centre = ((f0 + df / 2) * d.H + h0 + dh / 2) * d.W + w0 + dw / 2, extents = df | dh << 8 | dw << 16;
        for (int32_t s = base[0]; s < base[1]; ++s) {
          *slot_bucket++ = centre;
          *slot_bucket++ = extents;
        }
      }
  for (const Table& t : tables)
    if (t.host && t.bytes) std::memcpy(image.get() + t.at, t.host, t.bytes);
  VORTA_HIP(hipMalloc(&p->d_tables, total));
  VORTA_HIP(hipMemcpy(p->d_tables, image.get(), total, hipMemcpyHostToDevice));
  for (const Table& t : tables) *t.slot = (char*)p->d_tables + t.at;
  int cus = 0;
  VORTA_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  if (cus > 0) p->n_cus = cus;
  return VORTA_OK;
}

int ensure_device_tables(vorta_plan* p) {
  std::lock_guard<std::mutex> lock(p->mu);
  int dev = -1;
  VORTA_HIP(hipGetDevice(&dev));
  if (p->on_device) {
    // the tables live on the device that was current at the plan's first device call
    if (dev != p->device)
      return fail(VORTA_EINVAL, "plan belongs to device %d, current device is %d: one plan per device", p->device, dev);
    return VORTA_OK;
  }
  if (int rc = upload_device_tables(p, dev)) {
    release_device_tables(p);      // nothing half-built is kept; the next call starts over
    return rc;
  }
  p->device = dev;
  p->on_device = true;
  return VORTA_OK;
}

struct HeadList {
  int n;
  HeadIds id;
};

static HeadList head_list(const RouteLists& rl, int route) {
  HeadList h;
  h.n = rl.count[route];
  for (int i = 0; i < h.n; ++i) h.id.set(i, rl.heads[route][i]);
  return h;
}

struct Geo {
  int F, H, W;
  int L, N;
  int bF, bH, bW;   // bucket
  int nbH, nbW;     // bucket grid along H, W
  int keep_num, keep_den;
};

static Geo make_geo(const vorta_plan* p) {
  Geo g;
  g.F = p->d.F; g.H = p->d.H; g.W = p->d.W;
  g.L = (int)p->L; g.N = (int)p->N;
  g.bF = p->d.bucket[0]; g.bH = p->d.bucket[1]; g.bW = p->d.bucket[2];
  g.nbH = p->nb[1]; g.nbW = p->nb[2];
  g.keep_num = p->d.keep_num; g.keep_den = p->d.keep_den;
  return g;
}

// Rotary embedding: the table holds (cos, sin) per position and channel pair, axis after axis.
struct Rope {
  const float2* cs;     // [F][pF], [H][pH], [W][pW]
  int pF, pH, pW;       // channel pairs that turn with the frame index, the row, the column
  int baseH, baseW;     // first table entry of the H and W axes
  int H, W;             // grid extents, to decode a token index
  bool all;             // the spans cover every channel of a head
};

static Rope make_rope(const vorta_plan* p) {
  Rope r;
  r.cs = (const float2*)p->d_rope_cs;
  r.pF = p->d.rope_dims[0] / 2; r.pH = p->d.rope_dims[1] / 2; r.pW = p->d.rope_dims[2] / 2;
  r.baseH = p->d.F * r.pF;
  r.baseW = r.baseH + p->d.H * r.pH;
  r.H = p->d.H; r.W = p->d.W;
  r.all = 2 * (r.pF + r.pH + r.pW) == p->d.head_dim;
  return r;
}

// What of the table a lane needs for its NP channel pairs, whatever the token: pair i's entry is
// base[i] + the token's row of the table of axis[i]; a pair past the spans is left alone, and takes the first
// entry so that the read stays inside.  Spans that cover the head (rope.all, the same for every lane) need no
// such test, a fifth of the instructions of a turn; a token's three table rows are multiplied out once, not
// once per pair (an integer product costs four additions).
template <int NP>
struct RopeLane {
  int base[NP], axis[NP];
  bool past[NP], all;
  __device__ __forceinline__ RopeLane(const Rope& r, int pair0) : all(r.all) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int j = pair0 + i, jh = j - r.pF, jw = jh - r.pH;
      axis[i] = j < r.pF ? 0 : jh < r.pH ? 1 : 2;
      base[i] = j < r.pF ? j : jh < r.pH ? r.baseH + jh : r.baseW + jw;
      past[i] = jw >= r.pW;
    }
  }
  __device__ __forceinline__ void load(const Rope& r, int f, int h, int w, float2 (&cs)[NP]) const {
    const int of = f * r.pF, oh = h * r.pH, ow = w * r.pW;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      int at = base[i] + (axis[i] == 0 ? of : axis[i] == 1 ? oh : ow);
      if (!all) at = past[i] ? 0 : at;
      cs[i] = r.cs[at];
    }
  }
  // Turns x[2i], x[2i+1].  fp64; for rows as given (bf16 or fp32 elements times fp32 table entries) the
  // products are exact, so the fused form changes no bit there.
  __device__ __forceinline__ void turn(const float2 (&cs)[NP], double* x) const {
    if (all) turn_pairs<true>(cs, x);
    else turn_pairs<false>(cs, x);
  }
  template <bool ALL>
  __device__ __forceinline__ void turn_pairs(const float2 (&cs)[NP], double* x) const {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const double c = (double)cs[i].x, sn = (double)cs[i].y, u = x[2 * i], v = x[2 * i + 1];
      const double x0 = __builtin_fma(u, c, -(v * sn)), x1 = __builtin_fma(u, sn, v * c);
      x[2 * i] = !ALL && past[i] ? u : x0;
      x[2 * i + 1] = !ALL && past[i] ? v : x1;
    }
  }
};

// ------------------------------------------------------------------------------------------
// reorder: one thread per (tile-order row, 16-byte chunk), looping over the heads of route 1
// ------------------------------------------------------------------------------------------
template <bool TO_TILES>
__global__ __launch_bounds__(256) void reorder_kernel(uint4* __restrict__ user, uint4* __restrict__ tiled,
                                                      const int* __restrict__ tok_of, HeadList hl, int N,
                                                      long head_stride_c, long row_stride_c, int cshift) {
  const long gid = (long)blockIdx.x * 256 + threadIdx.x;
  const int pos = (int)(gid >> cshift);
  const int c = (int)(gid & ((1 << cshift) - 1));
  if (pos >= N) return;
  const int i = tok_of[pos];   // tile-order row -> token (text rows keep their place)
  const long u0 = (long)i * row_stride_c + c;
  const long t0 = ((long)pos << cshift) + c;
  const long tiled_head = (long)N << cshift;
#pragma unroll 4
  for (int s = 0; s < hl.n; ++s) {
    const long u = u0 + hl.id[s] * head_stride_c, t = t0 + s * tiled_head;
    if (TO_TILES) tiled[t] = user[u];
    else user[u] = tiled[t];
  }
}

static int chunk_shift(const vorta_plan* p) {
  const int chunks = p->d.head_dim * p->elem_bytes / 16;   // 16 or 32
  return chunks == 32 ? 5 : 4;
}

int launch_reorder(vorta_plan* p, const RouteLists& rl, const void* user, void* tiled, bool to_tiles,
                   void* stream) {
  if (rl.count[1] == 0) return VORTA_OK;
  const UserTensor ut = user_tensor(p, user);
  const int cs = chunk_shift(p);
  const int epc = 16 / p->elem_bytes;   // elements per chunk
  const long total = (long)p->N << cs;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  const HeadList hl = head_list(rl, 1);
  hipStream_t st = (hipStream_t)stream;
  if (to_tiles)
    hipLaunchKernelGGL(reorder_kernel<true>, dim3(blocks), dim3(256), 0, st, (uint4*)user, (uint4*)tiled,
                       p->d_tok_of, hl, (int)p->N, ut.head_stride / epc, ut.row_stride / epc, cs);
  else
    hipLaunchKernelGGL(reorder_kernel<false>, dim3(blocks), dim3(256), 0, st, (uint4*)user, (uint4*)tiled,
                       p->d_tok_of, hl, (int)p->N, ut.head_stride / epc, ut.row_stride / epc, cs);
  return launch_status("reorder_kernel");
}

// ------------------------------------------------------------------------------------------
// unpool: out[i] = o_c[assign[i]] for the heads of route 2 (text rows: o_c[L_c + t])
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void unpool_kernel(uint4* __restrict__ out, const uint4* __restrict__ o_c,
                                                     const int* __restrict__ assign, HeadList hl, int L,
                                                     int N, int Lc, long head_stride_c, long row_stride_c,
                                                     int cshift) {
  const long gid = (long)blockIdx.x * 256 + threadIdx.x;
  const int i = (int)(gid >> cshift);
  const int c = (int)(gid & ((1 << cshift) - 1));
  if (i >= N) return;
  const long u0 = (long)i * row_stride_c + c;
  const long core_head = (long)(Lc + N - L) << cshift;
#pragma unroll 4
  for (int s = 0; s < hl.n; ++s) {
    const int slot = i < L ? assign[(long)s * L + i] : Lc + (i - L);
    out[u0 + hl.id[s] * head_stride_c] = o_c[s * core_head + ((long)slot << cshift) + c];
  }
}

int launch_unpool(vorta_plan* p, const RouteLists& rl, const void* o_c, const int32_t* assign, void* out,
                  void* stream) {
  if (rl.count[2] == 0) return VORTA_OK;
  const UserTensor ut = user_tensor(p, out);
  const int cs = chunk_shift(p);
  const int epc = 16 / p->elem_bytes;
  const long total = (long)p->N << cs;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  hipLaunchKernelGGL(unpool_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, (uint4*)out,
                     (const uint4*)o_c, assign, head_list(rl, 2), (int)p->L, (int)p->N, (int)p->Lc,
                     ut.head_stride / epc, ut.row_stride / epc, cs);
  return launch_status("unpool_kernel");
}

// ------------------------------------------------------------------------------------------
// Bucketed core-set selection (helpers; the kernels follow).
// ------------------------------------------------------------------------------------------
template <typename T> struct Elem;
template <> struct Elem<float> {
  __device__ static double load(const float* p) { return (double)*p; }
  __device__ static void store(float* p, double v) { *p = (float)v; }
};
template <> struct Elem<uint16_t> {   // bf16 bits
  __device__ static double load(const uint16_t* p) { return (double)__uint_as_float((unsigned)*p << 16); }
  __device__ static void store(uint16_t* p, double v) {
    const unsigned u = __float_as_uint((float)v);      // round-to-nearest-even on the upper 16 bits
    *p = (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
  }
};

struct Bucket {
  int f0, h0, w0;   // origin
  int df, dh, dw;   // clipped extent
  int size, centre;
  float inv_hw, inv_dw;
};

__device__ __forceinline__ Bucket bucket_of(const Geo& g, int b) {
  Bucket k;
  const int per_f = g.nbH * g.nbW;
  const int bf = b / per_f, r = b - bf * per_f;
  const int bh = r / g.nbW, bw = r - bh * g.nbW;
  k.f0 = bf * g.bF; k.h0 = bh * g.bH; k.w0 = bw * g.bW;
  k.df = min(g.bF, g.F - k.f0); k.dh = min(g.bH, g.H - k.h0); k.dw = min(g.bW, g.W - k.w0);
  k.size = k.df * k.dh * k.dw;
  k.centre = ((k.df / 2) * k.dh + k.dh / 2) * k.dw + k.dw / 2;
  k.inv_hw = __builtin_amdgcn_rcpf((float)(k.dh * k.dw));
  k.inv_dw = __builtin_amdgcn_rcpf((float)k.dw);
  return k;
}

// Grid position and raster index of token j (0 <= j < 64) of a bucket.  The quotients are taken in
// fp32: (j + 1/2) / n is at least 1 / 128 away from an integer, far more than the reciprocal is off.
struct BucketToken {
  int f, h, w, tok;
};
__device__ __forceinline__ BucketToken bucket_token(const Geo& g, const Bucket& k, int j) {
  BucketToken t;
  const int a = (int)(((float)j + 0.5f) * k.inv_hw), r = j - a * (k.dh * k.dw);
  const int b = (int)(((float)r + 0.5f) * k.inv_dw), c = r - b * k.dw;
  t.f = k.f0 + a; t.h = k.h0 + b; t.w = k.w0 + c;
  t.tok = (t.f * g.H + t.h) * g.W + t.w;
  return t;
}

// 16-byte chunk of a row (8 bf16 or 4 fp32 elements): raw load, and widening to fp64
template <typename T> struct Chunk;
template <> struct Chunk<uint16_t> {
  static constexpr int N = 8;
  __device__ static uint4 raw(const uint16_t* p) { return *(const uint4*)p; }
  __device__ static void widen(const uint4& u, double* x) {
    const unsigned w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = (double)__uint_as_float(w[i] << 16);
      x[2 * i + 1] = (double)__uint_as_float(w[i] & 0xffff0000u);
    }
  }
  __device__ static void load(const uint16_t* p, double* x) { widen(raw(p), x); }
};
template <> struct Chunk<float> {
  static constexpr int N = 4;
  __device__ static uint4 raw(const float* p) { return *(const uint4*)p; }
  __device__ static void widen(const uint4& u, double* x) {
    x[0] = __uint_as_float(u.x); x[1] = __uint_as_float(u.y); x[2] = __uint_as_float(u.z); x[3] = __uint_as_float(u.w);
  }
  __device__ static void load(const float* p, double* x) { widen(raw(p), x); }
};

// A 16-byte chunk from fp64 values, each rounded to the element type through fp32 (round to nearest even).
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
template <typename T> __device__ __forceinline__ uint4 pack_chunk(const double* x);
template <> __device__ __forceinline__ uint4 pack_chunk<uint16_t>(const double* x) {
  unsigned u[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x2_t f = {(float)x[2 * i], (float)x[2 * i + 1]};
    u[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2_t));
  }
  return make_uint4(u[0], u[1], u[2], u[3]);
}
template <> __device__ __forceinline__ uint4 pack_chunk<float>(const double* x) {
  return make_uint4(__float_as_uint((float)x[0]), __float_as_uint((float)x[1]), __float_as_uint((float)x[2]),
                    __float_as_uint((float)x[3]));
}

// x / m for a small whole m with r = 1 / m (both correctly rounded): the quotient's error is removed by
// one residual step, three operations where a division takes ten times that.  A sum that is infinite
// or NaN has no residual and keeps the plain product.
__device__ __forceinline__ double div_by(double x, double m, double r) {
  const double q = x * r, e = __builtin_fma(-q, m, x);
  return e == e ? __builtin_fma(e, r, q) : q;
}

// ---- cross-lane sums of fp64 values.  The 16 lanes of a DPP row by rotations, the rows by half-row and
// half-wavefront swaps: all in the vector ALU, and every lane ends up with the same bits.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)u, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xf, 0xf, true);
  return v + __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double row16_sum(double v) {
  v = dpp_add<0x128>(v);      // row_ror:8
  v = dpp_add<0x124>(v);
  v = dpp_add<0x122>(v);
  return dpp_add<0x121>(v);
}
template <bool HALF>          // HALF: lanes l and l ^ 32, else l and l ^ 16
__device__ __forceinline__ double swap_add(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
  unsigned l0, l1, h0, h1;
  if constexpr (HALF) {
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
  } else {
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
  }
  return __builtin_bit_cast(double, ((unsigned long long)h0 << 32) | l0) +
         __builtin_bit_cast(double, ((unsigned long long)h1 << 32) | l1);
}
template <int CPR>            // sum over the CPR lanes that hold one row
__device__ __forceinline__ double row_sum(double v) {
  v = row16_sum(v);
  return CPR == 32 ? swap_add<false>(v) : v;
}
// Sums of a and of b over lanes l and l ^ 16 (HALF: l ^ 32), each in one lane of the two: rows 0 and 2 (HALF: the lower
// half) have a's, rows 1 and 3 (the upper half) b's.  The swap that brings a's other half brings b's too.
template <bool HALF>
__device__ __forceinline__ double scatter_add(double a, double b) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, a), w = __builtin_bit_cast(unsigned long long, b);
  unsigned l0, l1, h0, h1;
  if constexpr (HALF) {
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)w, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(w >> 32), false, false);
    l0 = l[0]; l1 = l[1]; h0 = h[0]; h1 = h[1];
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)w, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(w >> 32), false, false);
    l0 = l[0]; l1 = l[1]; h0 = h[0]; h1 = h[1];
  }
  return __builtin_bit_cast(double, ((unsigned long long)h0 << 32) | l0) +
         __builtin_bit_cast(double, ((unsigned long long)h1 << 32) | l1);
}
__device__ __forceinline__ double read_lane(double v, int lane) {
  const long long u = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)u, lane), hi = __builtin_amdgcn_readlane((int)(u >> 32), lane);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// The merged row of a bucket, from every lane's sums over the tokens it has seen (chunk c of its group's tokens): the
// groups' sums are added so that each group is left with one channel pair of the chunk, which it divides, turns and
// stores: 18 instead of 112 instructions for eight channels over four groups, and a quarter of the rest.  (Every group
// with the whole sums, one of them storing: selection of 16 heads of 75,600 tokens 265 -> 253 us, with rotation 326 -> 285
// at that time.)
template <typename T, int CPR>
struct MergedRow {
  static constexpr int PAIRS = Chunk<T>::N / 2, G = 64 / CPR;
  static_assert((G == 4 && (PAIRS == 4 || PAIRS == 2)) || (G == 2 && PAIRS == 2), "groups and channel pairs of a chunk");
  static __device__ __forceinline__ int pair_of(int grp) { return grp % PAIRS; }
  static __device__ __forceinline__ bool stores(int grp) { return grp < PAIRS; }
  static __device__ __forceinline__ void sum(const double (&x)[2 * PAIRS], double (&z)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (G == 2) {
        z[j] = scatter_add<true>(x[j], x[2 + j]);
      } else if constexpr (PAIRS == 2) {
        z[j] = swap_add<true>(scatter_add<false>(x[j], x[2 + j]));
      } else {
        z[j] = scatter_add<true>(scatter_add<false>(x[j], x[2 + j]), scatter_add<false>(x[4 + j], x[6 + j]));
      }
    }
  }
};
template <typename T> __device__ __forceinline__ void store_pair(T* to, const double (&z)[2]);
template <> __device__ __forceinline__ void store_pair<uint16_t>(uint16_t* to, const double (&z)[2]) {
  const f32x2_t f = {(float)z[0], (float)z[1]};
  *(unsigned*)to = __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2_t));
}
template <> __device__ __forceinline__ void store_pair<float>(float* to, const double (&z)[2]) {
  *(float2*)to = make_float2((float)z[0], (float)z[1]);
}

// ---- shared by the index pass, the pool pass and the two in one.  One wavefront per (bucket, head), or three
// where the one-pass kernel has few of them (its template parameter APART).  A row is CPR 16-byte chunks (16 or
// 32) and lies across CPR lanes, lane (c = lane % CPR, group = lane / CPR) holding chunk c of token G pass + group
// (G = 64 / CPR tokens a pass): every load and store instruction moves whole rows, and index and pool read the bucket
// in the same form.

// Dot product with the centre row (chunk craw) and squared norm of the row whose chunk is xraw, summed over
// the row's lanes.  fp64; a product of two bf16 (or fp32) values is exact in it, so forming
// it inside a fused multiply-add changes no bit.
template <typename T, int CPR>
__device__ __forceinline__ void row_dots(const uint4& craw, const uint4& xraw, double& dot, double& norm) {
  double c[Chunk<T>::N], x[Chunk<T>::N];
  Chunk<T>::widen(craw, c);
  Chunk<T>::widen(xraw, x);
  double d = 0.0, n = 0.0;
#pragma unroll
  for (int e = 0; e < Chunk<T>::N; ++e) {
    d = __builtin_fma(c[e], x[e], d);
    n = __builtin_fma(x[e], x[e], n);
  }
  dot = row_sum<CPR>(d);
  norm = row_sum<CPR>(n);
}

// Value of token `lane` (lanes below the bucket size), given pass p's value spread over the token's row.
template <int CPR>
__device__ __forceinline__ void to_token_lane(double v, int pass, int lane, double& mine) {
  constexpr int G = 64 / CPR;
  const double x = __shfl(v, CPR * (lane & (G - 1)), 64);
  if (lane / G == pass) mine = x;
}

// Cosine similarity from the sums; 0 for a zero norm or a non-finite result (keeps the ranking a total order).
__device__ __forceinline__ double similarity(double dot, double nc, double nj) {
#pragma clang fp contract(off)
  double sim = 0.0;
  if (nc != 0.0 && nj != 0.0) sim = dot / sqrt(nc * nj);
  return sim == sim ? sim : 0.0;
}

// Lane j holds the similarity of token j.  Ranks the non-centre tokens (larger similarity first,
// ties by index), prunes the first `prune` of them and numbers the kept tokens in raster order.
// Returns the slot token `lane` reads its output from (its own if kept, else the centre's);
// kept / centre_slot say whether the lane's token owns a slot and which slot the centre has.
__device__ __forceinline__ int rank_and_assign(const Bucket& k, int prune, int lane, double my_sim, int base_slot,
                                               bool& kept, int& centre_slot) {
  int rank = 0;
  for (int m = 0; m < k.size; ++m) {
    if (m == k.centre) continue;
    const double sm = read_lane(my_sim, m);
    if (sm > my_sim || (sm == my_sim && m < lane)) ++rank;
  }
  const bool in_bucket = lane < k.size;
  kept = in_bucket && (lane == k.centre || rank >= prune);
  const unsigned long long kept_mask = __ballot(kept);
  const int my_slot = base_slot + __popcll(kept_mask & ((1ull << lane) - 1ull));
  centre_slot = base_slot + __popcll(kept_mask & ((1ull << k.centre) - 1ull));
  return kept ? my_slot : centre_slot;
}

template <typename T, int D>   // D = head_dim
__global__ __launch_bounds__(256) void bcs_index_kernel(const T* __restrict__ feat, HeadList hl, Geo g,
                                                        int n_buckets, const int* __restrict__ slot_base,
                                                        long head_stride, long row_stride, int Lc,
                                                        int* __restrict__ keep_idx, int* __restrict__ assign) {
  constexpr int CN = Chunk<T>::N, CPR = D / CN, G = 64 / CPR;
  const int lane = threadIdx.x & 63;
  const int b = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int s = blockIdx.y;
  if (b >= n_buckets) return;
  const Bucket k = bucket_of(g, b);
  const int base_slot = slot_base[b], prune = k.size - (slot_base[b + 1] - base_slot);
  const int c = lane % CPR, grp = lane / CPR;
  const T* base = feat + hl.id[s] * head_stride + c * CN;
  const uint4 craw = Chunk<T>::raw(base + (long)bucket_token(g, k, k.centre).tok * row_stride);
  double my_dot = 0.0, my_norm = 0.0;
  // Rows of 32 chunks, two tokens a pass: four passes at a time, so that their loads go out together and their sums
  // run in each other's latency (64-token buckets of 3,072 tokens, 8 heads, 18.7 -> 15.3 us; a large grid 4 to 11 %
  // faster).  With 16 chunks the registers cost more than the latency (75,600 tokens, 94 -> 100 us).
  constexpr int U = CPR == 32 ? 4 : 1;
  int pass = 0;
  auto row = [&](int p) { return Chunk<T>::raw(base + (long)bucket_token(g, k, min(G * p + grp, k.size - 1)).tok * row_stride); };
  auto take = [&](int p, const uint4& raw) {
    double dot, norm;
    row_dots<T, CPR>(craw, raw, dot, norm);
    to_token_lane<CPR>(dot, p, lane, my_dot);
    to_token_lane<CPR>(norm, p, lane, my_norm);
  };
  for (; (pass + U - 1) * G < k.size; pass += U) {
    uint4 raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u] = row(pass + u);
#pragma unroll
    for (int u = 0; u < U; ++u) take(pass + u, raw[u]);
  }
  for (; pass * G < k.size; ++pass) take(pass, row(pass));
  const double nc = read_lane(my_norm, k.centre);
  bool kept;
  int centre_slot;
  const int slot = rank_and_assign(k, prune, lane, similarity(my_dot, nc, my_norm), base_slot, kept, centre_slot);
  if (lane < k.size) {
    const int tok = bucket_token(g, k, lane).tok;
    if (kept) keep_idx[(long)s * Lc + slot] = tok;
    assign[(long)s * g.L + tok] = slot;
  }
}

int launch_bcs_index(vorta_plan* p, const RouteLists& rl, const UserTensor& ut, int32_t* keep_idx,
                     int32_t* assign, void* stream) {
  if (rl.count[2] == 0) return VORTA_OK;
  const void* feat = ut.base;
  const dim3 grid((p->n_buckets + 3) / 4, rl.count[2]);
  const HeadList hl = head_list(rl, 2);
  const Geo g = make_geo(p);
  hipStream_t st = (hipStream_t)stream;
  if (p->d.dtype == VORTA_BF16)
    hipLaunchKernelGGL((bcs_index_kernel<uint16_t, 128>), grid, dim3(256), 0, st, (const uint16_t*)feat, hl, g,
                       p->n_buckets, p->d_slot_base, ut.head_stride, ut.row_stride, (int)p->Lc, keep_idx, assign);
  else if (p->d.head_dim == 64)
    hipLaunchKernelGGL((bcs_index_kernel<float, 64>), grid, dim3(256), 0, st, (const float*)feat, hl, g,
                       p->n_buckets, p->d_slot_base, ut.head_stride, ut.row_stride, (int)p->Lc, keep_idx, assign);
  else
    hipLaunchKernelGGL((bcs_index_kernel<float, 128>), grid, dim3(256), 0, st, (const float*)feat, hl, g,
                       p->n_buckets, p->d_slot_base, ut.head_stride, ut.row_stride, (int)p->Lc, keep_idx, assign);
  return launch_status("bcs_index_kernel");
}

// ------------------------------------------------------------------------------------------
// pool / merge.  A kept token's chunk is copied to its slot; the chunks of the centre and of the
// tokens pruned into it are summed in fp64, the G partial sums are added across the groups, and
// the groups write the mean to the centre's slot, a channel pair of every chunk each.
// ROPE: every pooled row is turned by the rotary embedding at the position of the token that owns
// its slot (the kept token itself; for a merged row the bucket's centre) before it is stored.
// ------------------------------------------------------------------------------------------
template <typename T, int D, bool ROPE>
__global__ __launch_bounds__(256) void bcs_pool_kernel(const T* __restrict__ src, HeadList hl, Geo g,
                                                       int n_buckets, long head_stride, long row_stride,
                                                       int n_core_rows, const int* __restrict__ assign,
                                                       T* __restrict__ dst, Rope rope) {
  constexpr int CN = Chunk<T>::N, CPR = D / CN, G = 64 / CPR;
  const int lane = threadIdx.x & 63;
  const int b = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int s = blockIdx.y;
  if (b >= n_buckets) return;
  const Bucket k = bucket_of(g, b);
  const int c = lane % CPR, grp = lane / CPR;
  const T* base = src + hl.id[s] * head_stride + c * CN;
  T* out = dst + (long)s * n_core_rows * D + c * CN;
  const RopeLane<CN / 2> rl(rope, c * (CN / 2));

  int my_slot = 0;
  if (lane < k.size) my_slot = assign[(long)s * g.L + bucket_token(g, k, lane).tok];
  const int centre_slot = __shfl(my_slot, k.centre, 64);
  const int members = __popcll(__ballot(lane < k.size && my_slot == centre_slot));
  double acc[CN];
#pragma unroll
  for (int e = 0; e < CN; ++e) acc[e] = 0.0;
  for (int j0 = 0; j0 < k.size; j0 += G) {
    const int j = j0 + grp;
    const int slot = __shfl(my_slot, min(j, k.size - 1), 64);
    if (j >= k.size) continue;
    const BucketToken t = bucket_token(g, k, j);
    const uint4 raw = Chunk<T>::raw(base + (long)t.tok * row_stride);
    if (slot == centre_slot) {
      double x[CN];
      Chunk<T>::widen(raw, x);
#pragma unroll
      for (int e = 0; e < CN; ++e) acc[e] += x[e];
    } else if (ROPE) {
      double x[CN];
      float2 cs[CN / 2];
      Chunk<T>::widen(raw, x);
      rl.load(rope, t.f, t.h, t.w, cs);
      rl.turn(cs, x);
      *(uint4*)(out + (long)slot * D) = pack_chunk<T>(x);
    } else {
      *(uint4*)(out + (long)slot * D) = raw;
    }
  }
  using Merged = MergedRow<T, CPR>;
  const double m = (double)members, r = 1.0 / m;
  const int pair = Merged::pair_of(grp);
  double z[2];
  Merged::sum(acc, z);
#pragma unroll
  for (int e = 0; e < 2; ++e) z[e] = div_by(z[e], m, r);
  if (ROPE) {
    const BucketToken t = bucket_token(g, k, k.centre);
    const RopeLane<1> rl_pair(rope, c * (CN / 2) + pair);
    float2 cs[1];
    rl_pair.load(rope, t.f, t.h, t.w, cs);
    rl_pair.turn(cs, z);
  }
  if (Merged::stores(grp)) store_pair<T>(out + (long)centre_slot * D + 2 * pair, z);
}

// text rows ride along unchanged behind the L_c pooled rows
__global__ __launch_bounds__(256) void copy_text_rows_kernel(const uint4* __restrict__ user,
                                                             uint4* __restrict__ core, HeadList hl, int L,
                                                             int n_text, int Lc, long head_stride_c,
                                                             long row_stride_c, int cshift) {
  const long gid = (long)blockIdx.x * 256 + threadIdx.x;
  const int t = (int)(gid >> cshift);
  const int c = (int)(gid & ((1 << cshift) - 1));
  if (t >= n_text) return;
  const long core_head = (long)(Lc + n_text) << cshift;
  for (int s = 0; s < hl.n; ++s)
    core[s * core_head + ((long)(Lc + t) << cshift) + c] =
        user[hl.id[s] * head_stride_c + (long)(L + t) * row_stride_c + c];
}

int launch_bcs_pool(vorta_plan* p, const RouteLists& rl, const void* src, const int32_t* keep_idx,
                    const int32_t* assign, bool rotate, void* dst, void* stream) {
  (void)keep_idx;   // the slot of every token is in `assign`; kept for a symmetric interface
  if (rl.count[2] == 0) return VORTA_OK;
  const UserTensor ut = user_tensor(p, src);
  const dim3 grid((p->n_buckets + 3) / 4, rl.count[2]);
  const HeadList hl = head_list(rl, 2);
  const Geo g = make_geo(p);
  const int rows = (int)(p->Lc + p->d.n_text);
  hipStream_t st = (hipStream_t)stream;
  const bool rope_on = rotate && p->rope;
  const Rope rope = make_rope(p);
#define VORTA_POOL(T_, D_, R_)                                                                                  \
  hipLaunchKernelGGL((bcs_pool_kernel<T_, D_, R_>), grid, dim3(256), 0, st, (const T_*)src, hl, g, p->n_buckets, \
                     ut.head_stride, ut.row_stride, rows, assign, (T_*)dst, rope)
  if (p->d.dtype == VORTA_BF16) {
    if (rope_on) VORTA_POOL(uint16_t, 128, true); else VORTA_POOL(uint16_t, 128, false);
  } else if (p->d.head_dim == 64) {
    if (rope_on) VORTA_POOL(float, 64, true); else VORTA_POOL(float, 64, false);
  } else {
    if (rope_on) VORTA_POOL(float, 128, true); else VORTA_POOL(float, 128, false);
  }
#undef VORTA_POOL
  if (int rc = launch_status("bcs_pool_kernel")) return rc;
  if (p->d.n_text > 0) {
    const int cs = chunk_shift(p);
    const int epc = 16 / p->elem_bytes;
    const long total = (long)p->d.n_text << cs;
    hipLaunchKernelGGL(copy_text_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       (const uint4*)src, (uint4*)dst, hl, (int)p->L, p->d.n_text, (int)p->Lc,
                       ut.head_stride / epc, ut.row_stride / epc, cs);
    return launch_status("copy_text_rows_kernel");
  }
  return VORTA_OK;
}

// ------------------------------------------------------------------------------------------
// Rotary embedding of whole rows, heads of routes 0 and 1: one thread per (row, 16-byte chunk) looks its
// table entries up once and loops over the heads, four at a time so that four loads are in flight; dst
// has the caller's layout.  One or two tensors (the layer call turns Q and K).  Text rows
// are copied.  Bound: HBM: Q and K of 14 heads x 119,056 tokens (1.7 GB) 339 us = 5.0 TB/s; with the table
// read again for every head and a launch for each tensor 578 us.
// ------------------------------------------------------------------------------------------
template <typename T>
struct RopeRows {
  const T* src[2];
  T* dst[2];
  HeadList hl;
  int L, N, cshift;
  long head_stride, row_stride;
  int blocks;          // workgroups per tensor
  int tensors;
};
template <typename T>
__device__ __forceinline__ void rope_rows_block(const RopeRows<T>& job, const Rope& rope, int block) {
  constexpr int CN = Chunk<T>::N;
  const bool second = block >= job.blocks;
  const T* __restrict__ src = second ? job.src[1] : job.src[0];
  T* __restrict__ dst = second ? job.dst[1] : job.dst[0];
  const HeadList& hl = job.hl;
  const long gid = (long)(second ? block - job.blocks : block) * 256 + threadIdx.x;
  const int i = (int)(gid >> job.cshift);
  const int c = (int)(gid & ((1 << job.cshift) - 1));
  if (i >= job.N) return;
  const long off0 = (long)i * job.row_stride + c * CN;
  if (i >= job.L) {
    for (int s = 0; s < hl.n; ++s) {
      const long off = off0 + hl.id[s] * job.head_stride;
      *(uint4*)(dst + off) = *(const uint4*)(src + off);
    }
    return;
  }
  const RopeLane<CN / 2> rl(rope, c * (CN / 2));
  float2 cs[CN / 2];
  const int f = i / (rope.H * rope.W), rem = i - f * (rope.H * rope.W), h = rem / rope.W;
  rl.load(rope, f, h, rem - h * rope.W, cs);
  for (int s0 = 0; s0 < hl.n; s0 += 4) {
    uint4 raw[4];
    long off[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (s0 + u >= hl.n) break;
      off[u] = off0 + hl.id[s0 + u] * job.head_stride;
      raw[u] = Chunk<T>::raw(src + off[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (s0 + u >= hl.n) break;
      double x[CN];
      Chunk<T>::widen(raw[u], x);
      rl.turn(cs, x);
      *(uint4*)(dst + off[u]) = pack_chunk<T>(x);
    }
  }
}

static int rope_rows_blocks(const vorta_plan* p) { return (int)((((long)p->N << chunk_shift(p)) + 255) / 256); }

template <typename T>
static RopeRows<T> rope_rows_job(const vorta_plan* p, const RouteLists& rl, const RopeCopies& r) {
  RopeRows<T> job;
  job.src[0] = (const T*)r.src[0]; job.src[1] = (const T*)r.src[1];
  job.dst[0] = (T*)r.dst[0]; job.dst[1] = (T*)r.dst[1];
  job.hl.n = 0;
  for (int route = 0; route < 2; ++route)
    for (int i = 0; i < rl.count[route]; ++i) job.hl.id.set(job.hl.n++, rl.heads[route][i]);
  const UserTensor ut = user_tensor(p, r.src[0]);
  job.L = (int)p->L; job.N = (int)p->N; job.cshift = chunk_shift(p);
  job.head_stride = ut.head_stride; job.row_stride = ut.row_stride;
  job.blocks = rope_rows_blocks(p);
  job.tensors = r.src[1] ? 2 : 1;
  return job;
}

// ------------------------------------------------------------------------------------------
// Select and pool in one pass (what the layer call runs): one wavefront per (bucket, head), where there are few of
// them one for each of its three tensors, requests the
// bucket's K, Q and V rows before it computes anything, P passes of G tokens each, so one memory round
// trip covers them all and every row comes from HBM once; then it ranks as bcs_index_kernel does, writes
// keep_idx / assign, and merges and stores the three tensors as bcs_pool_kernel does (same operations in
// the same order: the results of the two forms are identical bit for bit).  Further workgroups of a
// head copy its text rows behind the pooled ones, and the last ones turn the rows of the heads on
// routes 0 and 1 where the layer call asks for that too (a launch of its own costs a small layer 4 us).
//
// Rows of 12 tokens in bf16 without rotation take 74 vector registers, six wavefronts a SIMD (72 and seven while head ids were single bytes):
// 3 heads of 32,760 tokens 21.6 to 22.3 us then, 22.1 to 22.7 now, 16 of 75,600 level.  32-bit offsets of the output rows bring 72 back and up to
// 1.5 % there, but cost launches of less than 10 us 1 to 3 % and the 16-token instance a wavefront; a launch bound spills (8 to 12 % slower).
//
// Bound: HBM.  On 16 heads of 75,600 tokens (1.40 GB with the index) 253 us = 5.5 TB/s, more than a large copy
// reaches (4.9); with the rotary embedding 281 us, bound by vector instructions (the fp64 turn of every pooled Q and K
// row and its look-ups).  Buckets of 27 tokens with 2/3 of them kept (1.57 GB) 290 us = 5.4 TB/s, with rotation 360.  An earlier form
// that read K a second time as quarter rows, divided in fp64, took 64-bit integer quotients and stored
// element by element: 397 us and 718 us.
// ------------------------------------------------------------------------------------------
constexpr int HOLD_PASSES = 4;     // up to so many passes the rotation of a bucket's tokens fits in registers
template <typename T, int D, int P, bool ROPE, bool APART>
__global__ __launch_bounds__(256) void bcs_select_pool_kernel(const T* __restrict__ q, const T* __restrict__ k,
                                                              const T* __restrict__ v, HeadList hl, Geo g, int n_buckets,
                                                              int bucket_blocks, const int* __restrict__ slot_base,
                                                              long head_stride, long row_stride, int Lc, int n_core_rows,
                                                              int* __restrict__ keep_idx, int* __restrict__ assign,
                                                              T* __restrict__ qc, T* __restrict__ kc, T* __restrict__ vc,
                                                              Rope rope, int text_blocks, RopeRows<T> rows_job) {
  constexpr int CN = Chunk<T>::N, CPR = D / CN, G = 64 / CPR;
  // A head's workgroups: its buckets, its text rows, its share of the rotation.  APART: planes 0, 1 and 2 of the grid are the
  // buckets' K (and the index), Q and V, and the other workgroups of the launch fill planes behind them.  (Behind each of the
  // three, where they let Q's and V's start late: 1 core-set head of 4,096 tokens, 16 to a bucket, with 2 heads turned 11.0 us,
  // one wavefront for all three 9.4, now 8.4.)
  const int z = APART ? (int)blockIdx.z : 0;
  const bool does_k = !APART || z == 0, does_q = !APART || z == 1, does_v = !APART || z == 2;
  int s = blockIdx.y, x = blockIdx.x;              // x: place among the head's workgroups
  if constexpr (APART) {
    if (z >= 3) {
      const int other = ((z - 3) * (int)gridDim.y + s) * (int)gridDim.x + x, turn = other - text_blocks * (int)gridDim.y;
      if (turn >= 0) {
        if constexpr (ROPE)
          if (turn < rows_job.blocks * rows_job.tensors) rope_rows_block(rows_job, rope, turn);
        return;
      }
      s = other / text_blocks;
      x = bucket_blocks + other - s * text_blocks;
    }
  }
  if (ROPE && !APART && x >= bucket_blocks + text_blocks) {
    const int block = (x - bucket_blocks - text_blocks) * gridDim.y + s;
    if (block < rows_job.blocks * rows_job.tensors) rope_rows_block(rows_job, rope, block);
    return;
  }
  const long head_off = hl.id[s] * head_stride;
  if (x >= bucket_blocks) {          // text rows
    const int i = (x - bucket_blocks) * 256 + threadIdx.x;
    const int t = i / CPR, c = i % CPR;
    if (t >= g.N - g.L) return;
    const long from = head_off + (long)(g.L + t) * row_stride + c * CN, to = ((long)s * n_core_rows + Lc + t) * D + c * CN;
    *(uint4*)(qc + to) = Chunk<T>::raw(q + from);
    *(uint4*)(kc + to) = Chunk<T>::raw(k + from);
    *(uint4*)(vc + to) = Chunk<T>::raw(v + from);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int b = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (b >= n_buckets) return;
  const Bucket kb = bucket_of(g, b);               // kb.size <= P G: checked on the host
  const int c = lane % CPR, grp = lane / CPR;

  // ---- every load of the wavefront.  With a rotation the pointers of Q and V are made new here: known to be read only, the
  // compiler moves their loads down to where the rows are merged, a memory round trip behind K's.  (16 heads of 75,600 tokens:
  // buckets of 27 tokens 433 -> 396 us, of 8 tokens 344 -> 335, of 12 level.  Without a rotation more wavefronts, which the
  // registers of the early loads cost, hide more: 8 tokens 251 us as it is, 264 that way.)
  typedef const __attribute__((address_space(1))) T* global_ptr;
  global_ptr q_now = (global_ptr)q, v_now = (global_ptr)v;
  if constexpr (ROPE) asm volatile("" : "+s"(q_now), "+s"(v_now));
  const BucketToken centre = bucket_token(g, kb, kb.centre);
  const uint4 craw = Chunk<T>::raw(k + head_off + (long)centre.tok * row_stride + c * CN);
  uint4 rq[P], rk[P], rv[P];
  BucketToken tok_p[P];
  long off[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    tok_p[p] = bucket_token(g, kb, min(G * p + grp, kb.size - 1));
    off[p] = head_off + (long)tok_p[p].tok * row_stride + c * CN;
  }
#pragma unroll
  for (int p = 0; p < P; ++p) rk[p] = Chunk<T>::raw(k + off[p]);
  if constexpr (APART) {           // the one tensor that is pooled here, in rq's place
    if (does_q)
#pragma unroll
      for (int p = 0; p < P; ++p) rq[p] = Chunk<T>::raw((const T*)(q_now + off[p]));
    if (does_v)
#pragma unroll
      for (int p = 0; p < P; ++p) rq[p] = Chunk<T>::raw((const T*)(v_now + off[p]));
  } else {
#pragma unroll
    for (int p = 0; p < P; ++p) rq[p] = Chunk<T>::raw((const T*)(q_now + off[p]));
#pragma unroll
    for (int p = 0; p < P; ++p) rv[p] = Chunk<T>::raw((const T*)(v_now + off[p]));
  }
  const int base_slot = slot_base[b], prune = kb.size - (slot_base[b + 1] - base_slot);
  if constexpr (ROPE) __builtin_amdgcn_sched_barrier(0);
  const RopeLane<CN / 2> rl(rope, c * (CN / 2));

  // ---- select
  double my_dot = 0.0, my_norm = 0.0;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    double dot, norm;
    row_dots<T, CPR>(craw, rk[p], dot, norm);
    to_token_lane<CPR>(dot, p, lane, my_dot);
    to_token_lane<CPR>(norm, p, lane, my_norm);
  }
  const double nc = read_lane(my_norm, kb.centre);
  bool kept;
  int centre_slot;
  const int slot_of_lane = rank_and_assign(kb, prune, lane, similarity(my_dot, nc, my_norm), base_slot, kept, centre_slot);
  if (does_k && lane < kb.size) {
    const int tok = bucket_token(g, kb, lane).tok;
    if (kept) keep_idx[(long)s * Lc + slot_of_lane] = tok;
    assign[(long)s * g.L + tok] = slot_of_lane;
  }

  // ---- pool
  const double m = (double)(prune + 1), r = 1.0 / m;
  int slot_p[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    slot_p[p] = __shfl(slot_of_lane, min(G * p + grp, kb.size - 1), 64);
    // widen K again below instead of keeping its fp64 form in registers across the ranking
    asm volatile("" : "+v"(rk[p].x), "+v"(rk[p].y), "+v"(rk[p].z), "+v"(rk[p].w));
  }
  // rotation of the bucket's tokens, looked up once for K and Q where it fits in registers (V's wavefront looks it up too where it has one
  // of its own: pooling V ahead of that is level to 3 % slower)
  constexpr bool HOLD = ROPE && P <= HOLD_PASSES;
  float2 cs[HOLD ? P : 1][CN / 2], cs_centre[1];
  using Merged = MergedRow<T, CPR>;
  const int pair = Merged::pair_of(grp);
  const RopeLane<1> rl_pair(rope, c * (CN / 2) + pair);
  if (HOLD) {
#pragma unroll
    for (int p = 0; p < P; ++p) rl.load(rope, tok_p[p].f, tok_p[p].h, tok_p[p].w, cs[HOLD ? p : 0]);
  }
  if (ROPE) rl_pair.load(rope, centre.f, centre.h, centre.w, cs_centre);
  // NT tensors at once: K and Q share the look-ups of their rotation where those are not kept (16 heads of 75,600 tokens, buckets
  // of 27: 396 -> 360 us, fp32 buckets of 12 9.6 -> 8.8 us for 3 heads of 3,072; where they are kept, the registers of the second
  // sum cost a wavefront of four: buckets of 12 281 -> 316 us)
  auto pool = [&](auto tensors, const uint4 (&rows0)[P], T* dst0, const uint4 (&rows1)[P], T* dst1, auto rotate) {
    constexpr int NT = decltype(tensors)::value;
    T* const out[2] = {dst0 + (long)s * n_core_rows * D + c * CN, dst1 + (long)s * n_core_rows * D + c * CN};
    double acc[NT][CN];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < CN; ++e) acc[t][e] = 0.0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      if (G * p + grp >= kb.size) continue;
      if (slot_p[p] == centre_slot) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          double x[CN];
          Chunk<T>::widen(t ? rows1[p] : rows0[p], x);
#pragma unroll
          for (int e = 0; e < CN; ++e) acc[t][e] += x[e];
        }
      } else {
        if constexpr (rotate.value && !HOLD) rl.load(rope, tok_p[p].f, tok_p[p].h, tok_p[p].w, cs[0]);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          uint4 row = t ? rows1[p] : rows0[p];
          if constexpr (rotate.value) {
            double x[CN];
            Chunk<T>::widen(row, x);
            rl.turn(cs[HOLD ? p : 0], x);
            row = pack_chunk<T>(x);
          }
          *(uint4*)(out[t] + (long)slot_p[p] * D) = row;
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      double z[2];
      Merged::sum(acc[t], z);
#pragma unroll
      for (int e = 0; e < 2; ++e) z[e] = div_by(z[e], m, r);
      if constexpr (rotate.value) rl_pair.turn(cs_centre, z);
      if (Merged::stores(grp)) store_pair<T>(out[t] + (long)centre_slot * D + 2 * pair, z);
    }
  };
  const std::integral_constant<int, 1> one;
  const std::integral_constant<int, 2> two;
  const std::integral_constant<bool, true> turned;
  const std::integral_constant<bool, false> as_given;
  if constexpr (APART) {
    const std::integral_constant<bool, ROPE> rotate;
    if (does_k) pool(one, rk, kc, rk, kc, rotate);
    if (does_q) pool(one, rq, qc, rq, qc, rotate);
    if (does_v) pool(one, rq, vc, rq, vc, as_given);
    return;
  }
  if constexpr (ROPE && !HOLD) {
    pool(two, rk, kc, rq, qc, turned);
  } else {
    const std::integral_constant<bool, ROPE> rotate;
    pool(one, rk, kc, rk, kc, rotate);
    pool(one, rq, qc, rq, qc, rotate);
  }
  pool(one, rv, vc, rv, vc, as_given);
}

// True when one of the fused instances holds the plan's buckets: 12, 16 or 32 tokens in rows of 16 chunks,
// 12 or 16 in rows of 32 (the rows of a bucket live in registers).
static int fused_tokens(const vorta_plan* p) {
  const int tokens = p->d.bucket[0] * p->d.bucket[1] * p->d.bucket[2];   // <= 64
  const int chunks = p->d.head_dim * p->elem_bytes / 16;
  return tokens <= 12 ? 12 : tokens <= 16 ? 16 : tokens <= 32 && chunks == 16 ? 32 : 0;
}
bool bcs_fused_applies(const vorta_plan* p) { return fused_tokens(p) > 0; }

// How the launch of the selection in one pass is cut.
struct SelectForm {
  bool apart;                       // a wavefront for each tensor of a bucket, not one for all three
  int bucket_blocks, text_blocks;   // workgroups of a head
  int turn_blocks;                  // workgroups of the launch that turn rows of the heads on routes 0 and 1
};

// A wavefront for each tensor (APART) while those are no more than the SIMDs, one for all three beyond: the three rank the
// bucket each, so what is saved is time only while SIMDs are idle.  256 CUs, 64 to 336 (bucket, head) pairs: 1.07 to 1.19 times as
// fast (buckets of 12 of one head of 256 tokens 5.4 -> 4.5 us), 400 to 640 level or up to 4 % slower, 768 9 to 15 % slower.
// Rotated rows in more than four passes, which look the rotation up pass by pass (HOLD is false), gain up to 512 pairs (400 to 512:
// buckets of 27 tokens 13.3 -> 11.6 us, 12 and 16 tokens in fp32 rows of 128 channels 9.0 -> 8.3 and 11.0 -> 10.0), are level up to
// 576 and slower from 600.
// Where the launch turns rows too, the more wavefronts must not delay those: its workgroups (blocks below) are at most 4 a CU, and
// times the heads that each of the turning ones goes through at most 24 a CU, 64 with rotated buckets in more than four passes,
// which take longer themselves.  349 such launches of 256 to 9,216 tokens with 1 to 39 turned heads: 0.3 % over the faster form on
// average, ten by more than 1.5 %, the worst 6 %; by the number of pairs alone, with the order of the workgroups then, 1.0 %, 45 of them slower than
// one wavefront for all by more than 1 % and up to 20 % (1 core-set head of 3,072 tokens, 24 turned: 15.8 us, 17.6 apart).
// tensors: that are turned, 0 = none.
static SelectForm select_form(const vorta_plan* p, const RouteLists& rl, int tensors, int units) {
  SelectForm f;
  f.bucket_blocks = (p->n_buckets + 3) / 4;
  f.text_blocks = (int)((((long)p->d.n_text << chunk_shift(p)) + 255) / 256);
  const int passes = (fused_tokens(p) << chunk_shift(p)) / 64;
  const bool by_pass = p->rope && passes > HOLD_PASSES;
  f.turn_blocks = p->rope ? rope_rows_blocks(p) * tensors : 0;
  const long pairs = (long)p->n_buckets * rl.count[2];
  const long blocks = (3L * f.bucket_blocks + f.text_blocks) * rl.count[2] + f.turn_blocks;
  const int turned = f.turn_blocks ? rl.count[0] + rl.count[1] : 0;
  f.apart = pairs <= (by_pass ? 9L * units / 4 : 4L * units / 3) && blocks <= 4L * units &&
            blocks * turned <= (by_pass ? 64L : 24L) * units;
  return f;
}

// Index on K, then Q, K, V pooled (Q and K rotated if the plan has a rotary embedding) into
// qc, kc, vc, and the text rows copied behind them.
int launch_bcs_select_pool(vorta_plan* p, const RouteLists& rl, const void* q, const void* k, const void* v,
                           int32_t* keep_idx, int32_t* assign, void* qc, void* kc, void* vc, const RopeCopies* copies,
                           void* stream) {
  if (rl.count[2] == 0) return VORTA_OK;
  const UserTensor ut = user_tensor(p, k);
  const SelectForm f = select_form(p, rl, !copies ? 0 : copies->src[1] ? 2 : 1, p->n_cus);
  const HeadList hl = head_list(rl, 2);
  const Geo g = make_geo(p);
  const int rows = (int)(p->Lc + p->d.n_text), fused = fused_tokens(p);
  const int n = rl.count[2], per_plane = f.bucket_blocks * n;
  const dim3 grid = f.apart ? dim3(f.bucket_blocks, n, 3 + (f.text_blocks * n + f.turn_blocks + per_plane - 1) / per_plane)
                            : dim3(f.bucket_blocks + f.text_blocks + (f.turn_blocks + n - 1) / n, n);
  const Rope rope = make_rope(p);
  hipStream_t st = (hipStream_t)stream;
#define VORTA_FUSED(T_, D_, P_, R_, A_)                                                                                 \
  {                                                                                                                     \
    RopeRows<T_> job{};                                                                                                 \
    if (R_ && copies) job = rope_rows_job<T_>(p, rl, *copies);                                                          \
    hipLaunchKernelGGL((bcs_select_pool_kernel<T_, D_, P_, R_, A_>), grid, dim3(256), 0, st, (const T_*)q, (const T_*)k, \
                       (const T_*)v, hl, g, p->n_buckets, f.bucket_blocks, p->d_slot_base, ut.head_stride, ut.row_stride, \
                       (int)p->Lc, rows, keep_idx, assign, (T_*)qc, (T_*)kc, (T_*)vc, rope, f.text_blocks, job);        \
  }
#define VORTA_FUSED_R(T_, D_, P_) \
  if (p->rope) VORTA_FUSED_A(T_, D_, P_, true) else VORTA_FUSED_A(T_, D_, P_, false)
#define VORTA_FUSED_A(T_, D_, P_, R_) \
  { if (f.apart) VORTA_FUSED(T_, D_, P_, R_, true) else VORTA_FUSED(T_, D_, P_, R_, false) }
  if (p->d.dtype == VORTA_BF16) {
    if (fused == 12) { VORTA_FUSED_R(uint16_t, 128, 3); }
    else if (fused == 16) { VORTA_FUSED_R(uint16_t, 128, 4); }
    else { VORTA_FUSED_R(uint16_t, 128, 8); }
  } else if (p->d.head_dim == 64) {
    if (fused == 12) { VORTA_FUSED_R(float, 64, 3); }
    else if (fused == 16) { VORTA_FUSED_R(float, 64, 4); }
    else { VORTA_FUSED_R(float, 64, 8); }
  } else {
    if (fused == 12) { VORTA_FUSED_R(float, 128, 6); }
    else { VORTA_FUSED_R(float, 128, 8); }
  }
#undef VORTA_FUSED_R
#undef VORTA_FUSED_A
#undef VORTA_FUSED
  return launch_status("bcs_select_pool_kernel");
}

template <typename T>
__global__ __launch_bounds__(256) void rope_rows_kernel(RopeRows<T> job, Rope rope) {
  rope_rows_block(job, rope, blockIdx.x);
}

int launch_rope_rows(vorta_plan* p, const RouteLists& rl, const RopeCopies& copies, void* stream) {
  if (rl.count[0] + rl.count[1] == 0 || !p->rope) return VORTA_OK;
  const Rope rope = make_rope(p);
  hipStream_t st = (hipStream_t)stream;
#define VORTA_ROPE(T_)                                                                                          \
  {                                                                                                             \
    const RopeRows<T_> job = rope_rows_job<T_>(p, rl, copies);                                                  \
    hipLaunchKernelGGL(rope_rows_kernel<T_>, dim3(job.blocks * job.tensors), dim3(256), 0, st, job, rope);      \
  }
  if (p->d.dtype == VORTA_BF16) VORTA_ROPE(uint16_t) else VORTA_ROPE(float)
#undef VORTA_ROPE
  return launch_status("rope_rows_kernel");
}

// ------------------------------------------------------------------------------------------
// Router (Eq. 3) and hard selection (Eq. 4) for a whole sampling schedule: one wavefront per
// (step, head).  The gates depend on the timestep embedding only, so every step's routes can be
// had before sampling starts, in one launch.  The three logits are fp64 sums (lanes stride over
// d_t, then a fixed xor tree), the softmax is fp64, the gates are stored as fp32; Eq. 4 is
// decided on the fp64 gates, every tie going to full attention.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void router_kernel(const float* __restrict__ t_emb, const float* __restrict__ w_r,
                                                    int d_t, int heads, float* __restrict__ alpha,
                                                    uint8_t* __restrict__ routes) {
#pragma clang fp contract(off)
  const int h = blockIdx.x, step = blockIdx.y, lane = threadIdx.x;
  const float* t = t_emb + (long)step * d_t;
  const float* w = w_r + (long)h * d_t * 3;
  double z[3] = {0.0, 0.0, 0.0};
  for (int i = lane; i < d_t; i += 64) {
    const double ti = (double)t[i];
#pragma unroll
    for (int k = 0; k < 3; ++k) z[k] += ti * (double)w[3 * i + k];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) z[k] += __shfl_xor(z[k], off, 64);
  if (lane == 0) {
    const double m = fmax(z[0], fmax(z[1], z[2]));
    const double e0 = exp(z[0] - m), e1 = exp(z[1] - m), e2 = exp(z[2] - m);
    const double sum = e0 + e1 + e2;
    const double a1 = e0 / sum, a2 = e1 / sum, a3 = e2 / sum;
    float* out = alpha + ((long)step * heads + h) * 3;
    out[0] = (float)a1; out[1] = (float)a2; out[2] = (float)a3;
    uint8_t r = VORTA_ROUTE_FULL;
    if (a2 > a1 && a2 > a3) r = VORTA_ROUTE_WINDOW;
    else if (a3 > a1 && a3 > a2) r = VORTA_ROUTE_CORESET;
    routes[(long)step * heads + h] = r;
  }
}

int launch_router(const float* t_emb, const float* w_r, int n_steps, int d_t, int heads, float* alpha,
                  uint8_t* routes, void* stream) {
  hipLaunchKernelGGL(router_kernel, dim3(heads, n_steps), dim3(64), 0, (hipStream_t)stream, t_emb, w_r, d_t, heads,
                     alpha, routes);
  return launch_status("router_kernel");
}

// ------------------------------------------------------------------------------------------
// Eq. 5 blend: out = a1 o_full + a2 o_sliding + a3 o_coreset, gates per head
// ------------------------------------------------------------------------------------------
struct Gates {
  float a[VORTA_MAX_HEADS][3];
};

template <typename T>
__global__ __launch_bounds__(256) void blend_kernel(const T* __restrict__ o0, const T* __restrict__ o1,
                                                    const T* __restrict__ o2, T* __restrict__ out, Gates gt,
                                                    long total, int head_dim, int heads, long N, int layout) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const long row = i / head_dim;
  const int h = layout == VORTA_LAYOUT_NHD ? (int)(row % heads) : (int)(row / N);
  const double v = (double)gt.a[h][0] * Elem<T>::load(o0 + i) + (double)gt.a[h][1] * Elem<T>::load(o1 + i) +
                   (double)gt.a[h][2] * Elem<T>::load(o2 + i);
  Elem<T>::store(out + i, v);
}

int launch_blend3(vorta_plan* p, const void* o0, const void* o1, const void* o2, const float* alpha_host,
                  void* out, void* stream) {
  Gates gt;
  std::memset(&gt, 0, sizeof(gt));
  for (int h = 0; h < p->d.heads; ++h)
    for (int r = 0; r < 3; ++r) gt.a[h][r] = alpha_host[3 * h + r];
  const long total = (long)p->d.heads * p->N * p->d.head_dim;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  hipStream_t st = (hipStream_t)stream;
  if (p->d.dtype == VORTA_BF16)
    hipLaunchKernelGGL(blend_kernel<uint16_t>, dim3(blocks), dim3(256), 0, st, (const uint16_t*)o0,
                       (const uint16_t*)o1, (const uint16_t*)o2, (uint16_t*)out, gt, total, p->d.head_dim,
                       p->d.heads, (long)p->N, p->d.layout);
  else
    hipLaunchKernelGGL(blend_kernel<float>, dim3(blocks), dim3(256), 0, st, (const float*)o0, (const float*)o1,
                       (const float*)o2, (float*)out, gt, total, p->d.head_dim, p->d.heads, (long)p->N,
                       p->d.layout);
  return launch_status("blend_kernel");
}

}  // namespace vorta

// For the tests, not part of the ABI: how vorta_bcs_select_pool (layer = 0) or the selection launch of a layer call is cut with these
// routes on a device of `units` CUs: {apart, bucket_blocks, text_blocks, turn_blocks}, all 0 where no instance of the
// one-pass kernel holds the plan's buckets.
extern "C" int vorta_test_select_form(const vorta_plan* p, const uint8_t* routes_host, int32_t layer, int32_t units, int32_t out[4]) {
  using namespace vorta;
  RouteLists rl;
  if (int rc = split_routes(p, routes_host, &rl)) return rc;
  const int tensors = layer && rl.count[0] + rl.count[1] ? 2 : 0;
  const SelectForm f = bcs_fused_applies(p) ? select_form(p, rl, tensors, units) : SelectForm{};
  out[0] = f.apart; out[1] = f.bucket_blocks; out[2] = f.text_blocks; out[3] = f.turn_blocks;
  return VORTA_OK;
}
