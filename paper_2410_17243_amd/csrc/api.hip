// C ABI of the tiled contrastive loss: argument validation, workspace layout,
// grid selection and launches on the caller's stream.  No allocation, no host
// synchronisation, no global mutable state.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "bwd.hpp"
#include "infcl.h"

namespace infcl {
int launch_fwd(const void* img, const void* txt, int64_t b, int64_t d, int dtype, const float* scale, float* loss,
               double* loss64, float* lse_r, float* lse_c, float* aux, hipStream_t stream, float* pairs, float* udiag,
               float* ref2, double* partial);
int launch_fwd_shard(const void* img, const void* txt, int64_t b, int64_t d, int dtype, int64_t r0, int64_t nrows,
                     const float* scale, float* colpair, hipStream_t stream, float* pairs, float* udiag, float* ref2);
int launch_fwd_shard_finish(int64_t b, int64_t d, int dtype, int64_t r0, int64_t nrows, int64_t nparts,
                            const float* colpairs, const float* scale, float* lse_r, float* lse_c, float* aux,
                            double* loss_part, hipStream_t stream, float* pairs, const float* udiag, double* partial);
int fwd1_pairs(int64_t b);
int fwd2_pairs(int64_t b, int64_t d);
bool fwd2_supported(int64_t d, int dtype);
int launch_bwd(const void* img, const void* txt, int64_t b, int64_t d, int dtype, int64_t r0, int64_t nrows,
               const float* scale, const float* lse_r, const float* lse_c, const float* aux, const float* dloss,
               void* dimg, void* dtxt, int gdt, float* dscale, double* dscale64, float* lse2, double* ds_part,
               float* g16, float* part, size_t part_cap, hipStream_t stream);
BwdPlan plan_bwd(int64_t b, int64_t nrows, int64_t d, int dtype, size_t cap);
bool bwd_supported(int64_t d, int dtype);
}  // namespace infcl

namespace {

constexpr int64_t kMaxB = (int64_t)1 << 30;

// Widths: the interface takes 16-bit rows of any multiple of 8 features up to
// 1024 and fp32 rows of any multiple of 4 up to 512 (16-byte rows); the sweeps
// are built for multiples of 128 (16-bit) and 64 (fp32), and other widths run
// on zero-padded copies of the inputs in the workspace, the gradients going
// through padded buffers there too.  Zero features add nothing to any dot
// product, so every output is that of the unpadded problem; the padding's
// gradients are zero and are dropped.
int64_t kernel_width(int64_t d, int dtype) {
  const int64_t q = dtype == INFCL_F32 ? 64 : 128;
  return (d + q - 1) / q * q;
}
bool width_ok(int64_t d, int dtype) { return dtype == INFCL_F32 ? d % 4 == 0 && d <= 512 : d % 8 == 0 && d <= 1024; }
size_t elem_size(int dtype) { return dtype == INFCL_F32 ? 4 : 2; }

struct Layout {
  int64_t dk;  // the width the sweeps run at
  size_t pad, pairs, udiag, ref2, fwd_part;
  size_t fwd_total;  // the forward's share, from the start
  size_t lse2, bwd_part, g16, gpad;
  size_t base;   // least workspace the calls accept
  size_t total;  // infcl_workspace_size: with the room for partial sums
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace regions, sized for the sweeps that (b, d, dtype) launches.  The
// forward's: the padded copies of the inputs, the partial pairs of its grid,
// the diagonal, the base-2 diagonal references (resident rows only) and the
// loss partials.  The backward's: the base-2 log-sum-exp vectors, the dscale
// partials, the scale of G', the padded gradients, and the partial sums of
// split row blocks (part_room).  A shard uses the same regions: its forward
// leaves at most as many pairs and it splits its row blocks as far as the room
// allows.
// base, without room for partial sums beyond the forward's pairs, grows with
// b, so that a workspace for one batch serves every smaller one.  total adds
// what the split of the batch uses, and for batches up to INFCL_SPLIT_BATCH
// INFCL_SPLIT_BYTES (or what the split of so small a batch can use), so that
// their shards split too: 8 shards of b = 32768, d = 512 15.3 -> 5.4 ms.  Beyond, it
// stays at 336 (780) bytes per sample, the memory that a loss linear in b
// promises, and a shard's caller adds the room where it wants it (8 shards,
// d = 512: b = 32800 13.6 ms without it and 5.9 with, b = 65536 28.5 and 19.0;
// d = 256, b = 65536 19.3 and 11.7).
Layout make_layout(int64_t b, int64_t d, int dtype) {
  Layout L;
  L.dk = kernel_width(d, dtype);
  const bool resident = infcl::fwd2_supported(L.dk, dtype);
  const size_t npair = (size_t)(resident ? infcl::fwd2_pairs(b, L.dk) : infcl::fwd1_pairs(b));
  const size_t fb = (size_t)b * sizeof(float);
  size_t off = 0;
  L.pad = off; off = align256(off + (L.dk != d ? 2 * (size_t)b * (size_t)L.dk * elem_size(dtype) : 0));  // img, txt
  L.pairs = off; off = align256(off + 2 * npair * fb + 1024);  // (each of the four arrays is aligned)
  L.udiag = off; off = align256(off + fb);
  L.ref2 = off; off = align256(off + (resident ? fb : 0));
  L.fwd_part = off; off = align256(off + (size_t)((b + 31) / 32) * sizeof(double));
  L.fwd_total = off;
  L.lse2 = off; off = align256(off + 2 * fb);
  L.bwd_part = off; off = align256(off + (size_t)2 * ((b + 63) / 64) * sizeof(double));  // 64 or 128 rows per WG
  L.g16 = off; off = align256(off + (dtype != INFCL_BF16 ? (size_t)(2 * infcl::kPrepBlocks) * sizeof(float) : 0));
  L.gpad = off; off = align256(off + (L.dk != d ? 2 * (size_t)b * (size_t)L.dk * sizeof(float) : 0));  // dimg, dtxt
  L.base = off;
  size_t want = 0;
  if (b <= INFCL_SPLIT_BATCH) {
    const size_t ntile = (size_t)(b + 31) / 32;
    want = 2 * (size_t)(b + 127) / 128 * 128 * (size_t)L.dk * sizeof(float) * ntile + 4096;  // every tile its part
    if (want > INFCL_SPLIT_BYTES) want = INFCL_SPLIT_BYTES;
  } else {
    want = align256(infcl::plan_bwd(b, b, L.dk, dtype, INFCL_SPLIT_BYTES).part_bytes);
  }
  L.total = want > L.fwd_total - L.pairs ? align256(off + want) : off;
  return L;
}

// Where the backward keeps partial sums in a workspace of ws_bytes >= L.base:
// at its end, or, where less than the forward's pairs is left there, in their
// place (the backward no longer needs them).  A whole batch takes at most what
// it would with L.total, so that any workspace from that on gives the same bits.
struct PartRoom {
  size_t off, bytes;
};
PartRoom part_room(const Layout& L, size_t ws_bytes) {
  PartRoom r{L.base, ws_bytes - L.base};
  if (r.bytes <= L.fwd_total - L.pairs) r = PartRoom{L.pairs, L.fwd_total - L.pairs};
  if (r.bytes > INFCL_SPLIT_BYTES) r.bytes = INFCL_SPLIT_BYTES;
  return r;
}

// What infcl_fwd_noalloc's fixed scratch is measured by: the workspace of a
// 32 x 8 (resident rows) or 64 x 8 (streamed) forward grid, both passes'
// vectors and padded copies.  Never less than the forward's share of the
// layout near the limit; where the limit lies is part of the interface.
size_t noalloc_need(int64_t b, int64_t d, int dtype) {
  const int64_t dk = kernel_width(d, dtype);
  const bool resident = infcl::fwd2_supported(dk, dtype);
  const int64_t bm = resident ? (dk > 512 ? 128 : 256) : 64, bn = resident ? 32 : 256, rmax = resident ? 32 : 64;
  const int64_t nrb = (b + bm - 1) / bm, nct = (b + bn - 1) / bn;
  const size_t ncol = (size_t)(nrb < rmax ? nrb : rmax), nrow = (size_t)(nct < 8 ? nct : 8) * (resident ? 1 : 4);
  const size_t fb = (size_t)b * sizeof(float);
  size_t n = 2 * align256(nrow * fb) + 2 * align256(ncol * fb) + align256(fb) + align256(resident ? fb : 0) +
             align256((size_t)((b + 255) / 256) * sizeof(double)) + align256(2 * fb) +
             align256((size_t)2 * ((b + 63) / 64) * sizeof(double));
  if (dtype == INFCL_F16) n += align256((size_t)(2 + 2 * ((b + 255) / 256)) * sizeof(float));
  if (dk != d)
    n += align256(2 * (size_t)b * (size_t)dk * elem_size(dtype)) + align256(2 * (size_t)b * (size_t)dk * sizeof(float));
  return n;
}

// Row copies between widths, both sides' in one launch: rows of cin 16-byte
// chunks into rows of cout chunks, cut or zero-filled at the end.
__global__ void __launch_bounds__(256) copy_rows(const uint4* __restrict__ src0, const uint4* __restrict__ src1,
                                                 uint4* __restrict__ dst0, uint4* __restrict__ dst1, int64_t rows,
                                                 int cin, int cout) {
  const uint4* __restrict__ src = blockIdx.y ? src1 : src0;
  uint4* __restrict__ dst = blockIdx.y ? dst1 : dst0;
  const int64_t n = rows * cout;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / cout;
    const int c = (int)(i - r * cout);
    dst[i] = c < cin ? src[r * cin + c] : make_uint4(0u, 0u, 0u, 0u);
  }
}

dim3 copy_grid(int64_t n) { return dim3((unsigned)(n / 256 + 1 < 65536 ? n / 256 + 1 : 65536), 2); }

// The inputs the sweeps read: img and txt as given, or, when d is not a width
// the sweeps are built for, their zero-padded copies in the workspace.
// Returns false on a launch failure.
bool stage_inputs(const void*& img, const void*& txt, int64_t b, int64_t d, int dtype, char* ws, const Layout& L,
                  hipStream_t stream) {
  if (L.dk == d) return true;
  const int cin = (int)(d * elem_size(dtype) / 16), cout = (int)(L.dk * elem_size(dtype) / 16);
  const int64_t n = b * cout;
  uint4* pi = (uint4*)(ws + L.pad);
  uint4* pt = pi + n;
  hipLaunchKernelGGL(copy_rows, copy_grid(n), dim3(256), 0, stream, (const uint4*)img, (const uint4*)txt, pi, pt, b, cin,
                     cout);
  if (hipGetLastError() != hipSuccess) return false;
  img = pi;
  txt = pt;
  return true;
}

// Gradient element type: 0 fp32, 1 the 16-bit input type; -1 for an unknown
// type, -2 for a known one that is neither (16-bit gradients of another type,
// or of fp32 inputs, are not built).
int grad_kind(int grad_dtype, int dtype) {
  if (grad_dtype != INFCL_BF16 && grad_dtype != INFCL_F32 && grad_dtype != INFCL_F16) return -1;
  if (grad_dtype == INFCL_F32) return 0;
  return grad_dtype == dtype ? 1 : -2;
}

// Where the sweeps write the gradients of `rows` own samples: the caller's
// dimg and dtxt, or padded buffers in the workspace that unstage_grads then
// copies, without the padding, into the caller's.  ges: gradient element size.
void grad_targets(void*& gi, void*& gt, int64_t b, int64_t d, size_t ges, char* ws, const Layout& L) {
  if (L.dk == d) return;
  gi = ws + L.gpad;
  gt = ws + L.gpad + (size_t)b * (size_t)L.dk * ges;
}
bool unstage_grads(void* dimg, void* dtxt, int64_t rows, int64_t b, int64_t d, size_t ges, char* ws,
                   const Layout& L, hipStream_t stream) {
  if (L.dk == d) return true;
  const int cin = (int)(L.dk * ges / 16), cout = (int)(d * ges / 16);
  const uint4* gi = (const uint4*)(ws + L.gpad);
  const uint4* gt = gi + b * cin;
  const int64_t n = rows * cout;
  hipLaunchKernelGGL(copy_rows, copy_grid(n), dim3(256), 0, stream, gi, gt, (uint4*)dimg, (uint4*)dtxt, rows, cin,
                     cout);
  return hipGetLastError() == hipSuccess;
}


bool aligned(const void* p, size_t a) { return p != nullptr && ((uintptr_t)p % a) == 0; }

bool shape_ok(int64_t b, int64_t d, int dtype) {
  return b >= 1 && d >= 1 && (dtype == INFCL_BF16 || dtype == INFCL_F32 || dtype == INFCL_F16);
}

bool shape_supported(int64_t b, int64_t d, int dtype) {
  return b <= kMaxB && width_ok(d, dtype) && infcl::bwd_supported(kernel_width(d, dtype), dtype);
}

// A shard: own samples [r0, r0 + bs) of the batch, r0 a multiple of 32 (so
// that own row blocks line up with the 32-row swept tiles).
bool shard_ok(int64_t b, int64_t r0, int64_t bs) { return r0 >= 0 && r0 % 32 == 0 && bs >= 1 && r0 + bs <= b; }

constexpr int64_t kMaxParts = 1 << 16;  // shards whose column pairs one finish merges

// ---- fixed scratch of infcl_fwd_noalloc: its workspace, for callers that
// cannot allocate.  Each device holds its own copy for the life of the
// process.  In host code the array's name is not a device address: the
// address comes from hipGetSymbolAddress, once per device, with that device
// current, and only that address is handed to kernels.
constexpr size_t kScratchBytes = (size_t)32 << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) char scratch[kScratchBytes];
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mu;

// The current device's scratch address (nullptr on a HIP error).
void* scratch_address() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return nullptr;
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}

}  // namespace

extern "C" {

infcl_status infcl_workspace_size(int64_t b, int64_t d, int dtype, size_t* bytes) {
  if (bytes == nullptr || !shape_ok(b, d, dtype)) return INFCL_ERR_INVALID;
  if (!shape_supported(b, d, dtype)) return INFCL_ERR_UNSUPPORTED;
  *bytes = make_layout(b, d, dtype).total;
  return INFCL_OK;
}

infcl_status infcl_fwd(const void* img, const void* txt, int64_t b, int64_t d, int dtype, const float* scale,
                       float* loss, double* loss64, float* lse_r, float* lse_c, float* aux, void* workspace,
                       size_t ws_bytes, void* stream) {
  if (!shape_ok(b, d, dtype)) return INFCL_ERR_INVALID;
  if (!aligned(img, 16) || !aligned(txt, 16) || !aligned(scale, 4) || !aligned(loss, 4) || !aligned(lse_r, 16) ||
      !aligned(lse_c, 16) || !aligned(aux, 16) || !aligned(workspace, 256))
    return INFCL_ERR_INVALID;
  if (loss64 != nullptr && ((uintptr_t)loss64 % 8) != 0) return INFCL_ERR_INVALID;
  if (!shape_supported(b, d, dtype)) return INFCL_ERR_UNSUPPORTED;
  const Layout L = make_layout(b, d, dtype);
  if (ws_bytes < L.base) return INFCL_ERR_WORKSPACE;
  char* ws = (char*)workspace;
  if (!stage_inputs(img, txt, b, d, dtype, ws, L, (hipStream_t)stream)) return INFCL_ERR_HIP;
  int rc = infcl::launch_fwd(img, txt, b, L.dk, dtype, scale, loss, loss64, lse_r, lse_c, aux, (hipStream_t)stream,
                             (float*)(ws + L.pairs), (float*)(ws + L.udiag), (float*)(ws + L.ref2),
                             (double*)(ws + L.fwd_part));
  return rc == 0 ? INFCL_OK : INFCL_ERR_HIP;
}

infcl_status infcl_fwd_noalloc(const void* img, const void* txt, int64_t b, int64_t d, int dtype, const float* scale,
                               float* loss, double* loss64, float* lse_r, float* lse_c, float* aux, void* stream) {
  if (!shape_ok(b, d, dtype)) return INFCL_ERR_INVALID;
  if (!aligned(img, 16) || !aligned(txt, 16) || !aligned(scale, 4) || !aligned(loss, 4) || !aligned(lse_r, 16) ||
      !aligned(lse_c, 16) || !aligned(aux, 16))
    return INFCL_ERR_INVALID;
  if (loss64 != nullptr && ((uintptr_t)loss64 % 8) != 0) return INFCL_ERR_INVALID;
  if (!shape_supported(b, d, dtype)) return INFCL_ERR_UNSUPPORTED;
  const Layout L = make_layout(b, d, dtype);
  if (noalloc_need(b, d, dtype) > kScratchBytes || L.fwd_total > kScratchBytes) return INFCL_ERR_WORKSPACE;
  char* ws = (char*)scratch_address();
  if (ws == nullptr) return INFCL_ERR_HIP;
  if (!stage_inputs(img, txt, b, d, dtype, ws, L, (hipStream_t)stream)) return INFCL_ERR_HIP;
  int rc = infcl::launch_fwd(img, txt, b, L.dk, dtype, scale, loss, loss64, lse_r, lse_c, aux, (hipStream_t)stream,
                             (float*)(ws + L.pairs), (float*)(ws + L.udiag), (float*)(ws + L.ref2),
                             (double*)(ws + L.fwd_part));
  return rc == 0 ? INFCL_OK : INFCL_ERR_HIP;
}

infcl_status infcl_bwd(const void* img, const void* txt, int64_t b, int64_t d, int dtype, const float* scale,
                       const float* lse_r, const float* lse_c, const float* aux, const float* dloss, void* dimg,
                       void* dtxt, int grad_dtype, float* dscale, void* workspace, size_t ws_bytes, void* stream) {
  const int gk = grad_kind(grad_dtype, dtype);
  if (!shape_ok(b, d, dtype) || gk == -1) return INFCL_ERR_INVALID;
  if (!aligned(img, 16) || !aligned(txt, 16) || !aligned(scale, 4) || !aligned(lse_r, 16) || !aligned(lse_c, 16) ||
      !aligned(aux, 16) || !aligned(dimg, 16) || !aligned(dtxt, 16) || !aligned(dscale, 4) ||
      !aligned(workspace, 256))
    return INFCL_ERR_INVALID;
  if (dloss != nullptr && ((uintptr_t)dloss % 4) != 0) return INFCL_ERR_INVALID;
  if (!shape_supported(b, d, dtype) || gk < 0) return INFCL_ERR_UNSUPPORTED;
  const Layout L = make_layout(b, d, dtype);
  if (ws_bytes < L.base) return INFCL_ERR_WORKSPACE;
  char* ws = (char*)workspace;
  if (!stage_inputs(img, txt, b, d, dtype, ws, L, (hipStream_t)stream)) return INFCL_ERR_HIP;
  const size_t ges = gk ? 2 : 4;
  void *gi = dimg, *gt = dtxt;
  grad_targets(gi, gt, b, d, ges, ws, L);
  const PartRoom room = part_room(L, ws_bytes);
  int rc = infcl::launch_bwd(img, txt, b, L.dk, dtype, 0, b, scale, lse_r, lse_c, aux, dloss, gi, gt, gk, dscale,
                             nullptr, (float*)(ws + L.lse2), (double*)(ws + L.bwd_part), (float*)(ws + L.g16),
                             (float*)(ws + room.off), room.bytes, (hipStream_t)stream);
  if (rc == 2) return INFCL_ERR_UNSUPPORTED;
  if (rc == 0 && !unstage_grads(dimg, dtxt, b, b, d, ges, ws, L, (hipStream_t)stream)) rc = 1;
  return rc == 0 ? INFCL_OK : INFCL_ERR_HIP;
}

// ------------------------------------------------------------------ shards

infcl_status infcl_fwd_shard(const void* img, const void* txt, int64_t b, int64_t d, int dtype, int64_t r0,
                             int64_t bs, const float* scale, float* colpair, void* workspace, size_t ws_bytes,
                             void* stream) {
  if (!shape_ok(b, d, dtype) || !shard_ok(b, r0, bs)) return INFCL_ERR_INVALID;
  if (!aligned(img, 16) || !aligned(txt, 16) || !aligned(scale, 4) || !aligned(colpair, 16) ||
      !aligned(workspace, 256))
    return INFCL_ERR_INVALID;
  if (!shape_supported(b, d, dtype)) return INFCL_ERR_UNSUPPORTED;
  const Layout L = make_layout(b, d, dtype);
  if (ws_bytes < L.base) return INFCL_ERR_WORKSPACE;
  char* ws = (char*)workspace;
  if (!stage_inputs(img, txt, b, d, dtype, ws, L, (hipStream_t)stream)) return INFCL_ERR_HIP;
  int rc = infcl::launch_fwd_shard(img, txt, b, L.dk, dtype, r0, bs, scale, colpair, (hipStream_t)stream,
                                   (float*)(ws + L.pairs), (float*)(ws + L.udiag), (float*)(ws + L.ref2));
  return rc == 0 ? INFCL_OK : INFCL_ERR_HIP;
}

infcl_status infcl_fwd_shard_finish(int64_t b, int64_t d, int dtype, int64_t r0, int64_t bs, int64_t nparts,
                                    const float* colpairs, const float* scale, float* lse_r, float* lse_c,
                                    float* aux, double* loss_part, void* workspace, size_t ws_bytes, void* stream) {
  if (!shape_ok(b, d, dtype) || !shard_ok(b, r0, bs) || nparts < 1 || nparts > kMaxParts) return INFCL_ERR_INVALID;
  if (!aligned(colpairs, 4) || !aligned(scale, 4) || !aligned(lse_r, 4) || !aligned(lse_c, 4) || !aligned(aux, 4) ||
      !aligned(loss_part, 8) || !aligned(workspace, 256))
    return INFCL_ERR_INVALID;
  if (!shape_supported(b, d, dtype)) return INFCL_ERR_UNSUPPORTED;
  const Layout L = make_layout(b, d, dtype);
  if (ws_bytes < L.base) return INFCL_ERR_WORKSPACE;
  char* ws = (char*)workspace;
  int rc = infcl::launch_fwd_shard_finish(b, L.dk, dtype, r0, bs, nparts, colpairs, scale, lse_r, lse_c, aux, loss_part,
                                          (hipStream_t)stream, (float*)(ws + L.pairs),
                                          (const float*)(ws + L.udiag), (double*)(ws + L.fwd_part));
  return rc == 0 ? INFCL_OK : INFCL_ERR_HIP;
}

infcl_status infcl_bwd_shard(const void* img, const void* txt, int64_t b, int64_t d, int dtype, int64_t r0,
                             int64_t bs, const float* scale, const float* lse_r, const float* lse_c, const float* aux,
                             const float* dloss, void* dimg, void* dtxt, int grad_dtype, double* dscale_part,
                             void* workspace, size_t ws_bytes, void* stream) {
  const int gk = grad_kind(grad_dtype, dtype);
  if (!shape_ok(b, d, dtype) || !shard_ok(b, r0, bs) || gk == -1) return INFCL_ERR_INVALID;
  if (!aligned(img, 16) || !aligned(txt, 16) || !aligned(scale, 4) || !aligned(lse_r, 16) || !aligned(lse_c, 16) ||
      !aligned(aux, 16) || !aligned(dimg, 16) || !aligned(dtxt, 16) || !aligned(dscale_part, 8) ||
      !aligned(workspace, 256))
    return INFCL_ERR_INVALID;
  if (dloss != nullptr && ((uintptr_t)dloss % 4) != 0) return INFCL_ERR_INVALID;
  if (!shape_supported(b, d, dtype) || gk < 0) return INFCL_ERR_UNSUPPORTED;
  const Layout L = make_layout(b, d, dtype);
  if (ws_bytes < L.base) return INFCL_ERR_WORKSPACE;
  char* ws = (char*)workspace;
  if (!stage_inputs(img, txt, b, d, dtype, ws, L, (hipStream_t)stream)) return INFCL_ERR_HIP;
  const size_t ges = gk ? 2 : 4;
  void *gi = dimg, *gt = dtxt;
  grad_targets(gi, gt, b, d, ges, ws, L);
  const PartRoom room = part_room(L, ws_bytes);
  int rc = infcl::launch_bwd(img, txt, b, L.dk, dtype, r0, bs, scale, lse_r, lse_c, aux, dloss, gi, gt, gk, nullptr,
                             dscale_part, (float*)(ws + L.lse2), (double*)(ws + L.bwd_part), (float*)(ws + L.g16),
                             (float*)(ws + room.off), room.bytes, (hipStream_t)stream);
  if (rc == 2) return INFCL_ERR_UNSUPPORTED;
  if (rc == 0 && !unstage_grads(dimg, dtxt, bs, b, d, ges, ws, L, (hipStream_t)stream)) rc = 1;
  return rc == 0 ? INFCL_OK : INFCL_ERR_HIP;
}

const char* infcl_status_str(int status) {
  switch (status) {
    case INFCL_OK: return "ok";
    case INFCL_ERR_INVALID: return "invalid argument (null or misaligned pointer, b < 1, d < 1 or unknown dtype)";
    case INFCL_ERR_UNSUPPORTED:
      return "unsupported shape (bf16, f16: d a multiple of 8 up to 1024; f32: d a multiple of 4 up to 512; "
             "b <= 2^30) or gradient type (f32, or the inputs' 16-bit type)";
    case INFCL_ERR_WORKSPACE: return "workspace too small (see infcl_workspace_size)";
    case INFCL_ERR_HIP: return "HIP kernel launch failed";
    default: return "unknown status";
  }
}

}  // extern "C"
