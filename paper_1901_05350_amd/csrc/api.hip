// C ABI of libtfx: argument validation, shape rules and kernel selection.
// Every entry point validates on the host before any HIP call and then only enqueues
// kernels on the caller's stream (enqueue-and-return, as the ops of Section 3.6 / 4.1).
#include "pack.h"
#include "tfx_internal.h"

namespace tfx {

int out_extent(int64_t in, int64_t k, int64_t s, int pad, int64_t* out, int64_t* before, int64_t* after) {
  if (in < 1 || k < 1) return TFX_ERR_SHAPE;
  if (s < 1) return TFX_ERR_ARG;
  if (pad == TFX_PAD_VALID) {
    if (in < k) return TFX_ERR_SHAPE;
    *out = (in - k) / s + 1;
    *before = *after = 0;
    return TFX_OK;
  }
  if (pad != TFX_PAD_SAME) return TFX_ERR_ARG;
  const int64_t o = (in + s - 1) / s;
  const int64_t need = (o - 1) * s + k - in;
  const int64_t total = need > 0 ? need : 0;
  *out = o;
  *before = total >> 1;
  *after = total - (total >> 1);
  return TFX_OK;
}

namespace {

constexpr int64_t kMaxElems = (int64_t(1) << 31) - 1;

bool valid_act(int act) { return act == TFX_ACT_NONE || act == TFX_ACT_RELU || act == TFX_ACT_RELU6; }

// numel, or -1 if it does not fit below 2^31
int64_t numel(const int64_t* d, int rank) {
  int64_t p = 1;
  for (int i = 0; i < rank; ++i) {
    if (d[i] > kMaxElems) return -1;
    p *= d[i];
    if (p > kMaxElems) return -1;
  }
  return p;
}

struct ConvGeom {
  int64_t out[4];
  int64_t pad[4];
};

int conv_geometry(const int64_t x[4], const int64_t f[4], int sh, int sw, int pad, bool depthwise, ConvGeom* g) {
  for (int i = 0; i < 4; ++i)
    if (x[i] < 1 || f[i] < 1) return TFX_ERR_SHAPE;
  if (x[3] != f[2]) return TFX_ERR_SHAPE;
  if (sh < 1 || sw < 1) return TFX_ERR_ARG;
  if (pad != TFX_PAD_VALID && pad != TFX_PAD_SAME) return TFX_ERR_ARG;
  int rc = out_extent(x[1], f[0], sh, pad, &g->out[1], &g->pad[0], &g->pad[1]);
  if (rc) return rc;
  rc = out_extent(x[2], f[1], sw, pad, &g->out[2], &g->pad[2], &g->pad[3]);
  if (rc) return rc;
  g->out[0] = x[0];
  g->out[3] = depthwise ? x[3] * f[3] : f[3];
  return TFX_OK;
}

int matmul_geometry(const int64_t a[2], const int64_t b[2], int ta, int tb, int64_t* m, int64_t* n, int64_t* k) {
  if (a[0] < 1 || a[1] < 1 || b[0] < 1 || b[1] < 1) return TFX_ERR_SHAPE;
  *m = ta ? a[1] : a[0];
  *k = ta ? a[0] : a[1];
  const int64_t kb = tb ? b[1] : b[0];
  *n = tb ? b[0] : b[1];
  return *k == kb ? TFX_OK : TFX_ERR_SHAPE;
}

int batch_matmul_impl(const float* a, const int64_t* a_shape, const float* b, const int64_t* b_shape, int64_t batch,
                      int ta, int tb, float* c, void* stream) {
  int64_t m, n, k;
  int rc = matmul_geometry(a_shape, b_shape, ta, tb, &m, &n, &k);
  if (rc) return rc;
  const int64_t da[3] = {batch, m, k}, db[3] = {batch, n, k}, dc[3] = {batch, m, n};
  if (numel(da, 3) < 0 || numel(db, 3) < 0 || numel(dc, 3) < 0) return TFX_ERR_UNSUPPORTED;
  // stored [M,K] (not transposed) means K is contiguous for A; stored [N,K] (transposed) for B
  return launch_gemm(a, b, c, nullptr, (int)batch, (int)m, (int)n, (int)k, !ta, tb != 0, TFX_ACT_NONE,
                     static_cast<hipStream_t>(stream));
}

// MobileNet v1 1.0 / 224 architecture (Section 3.9, Table 1 workload).
constexpr int kBlocks = 13;
constexpr int kChannels[kBlocks] = {64, 128, 128, 256, 256, 512, 512, 512, 512, 512, 512, 1024, 1024};
constexpr int kStrides[kBlocks] = {1, 2, 1, 2, 1, 2, 1, 1, 1, 1, 1, 2, 1};
constexpr int kImage = 224, kStemChannels = 32, kClasses = 1000, kFeatures = 1024;
constexpr size_t kAlign = 256;

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

bool valid_variant(const tfx_mobilenet_v1_variant* v) {
  return v && v->image_size >= 32 && v->image_size <= 256 && v->width_quarters >= 1 && v->width_quarters <= 4 &&
         v->classes >= 1 && v->classes <= 1024;
}

// On binary16 storage, each block's form: depthwise and pointwise layer in one launch, for few pixels with a workgroup per
// 4 x 4 patch (block_patch_f16.hip), with the filters stationary in LDS (block_stream_f16.hip: large batch, early block) or
// with the depthwise output there (block_tile_f16.hip), or as two.  The pointwise filters of the tile form are put in its
// order by one launch in front, for which one or two such blocks do not pay.  (All operands are taken to be aligned.)
enum BlockForm { kTwo, kPatch, kStream, kTile, kStem };
// Multiplications of the pointwise layer up to which the patch form is the fastest: each column slice of a patch computes its
// depthwise layer again, so its time grows with both.  Full width, batch 4 (14 x 14 x 512 -> 512 205e6) 102 us against 122
// without that block, batch 6 (308e6) 150 against 145; 3/4 width, whose other form is two launches for most blocks, batch 16
// 194 with blocks of 308e6, 212 without, batch 12 with blocks of 416e6 208 against 180.
constexpr int64_t kPatchProducts = 210000000, kPatchProductsTwo = 310000000;
struct BlockPlan {
  BlockForm form[kBlocks];
  int tiles, c[kBlocks], n[kBlocks];  // of all blocks
  size_t packed[kBlocks], packed_halfs;  // the tile blocks' filters
};
BlockPlan plan_blocks_f16(const tfx_mobilenet_v1_variant& v, int64_t batch) {
  BlockPlan p{};
  const int q = (int)v.width_quarters;
  int hw = (int)(v.image_size + 1) / 2;
  bool small[kBlocks];  // a block that the patch kernel computes faster than two launches do
  for (int b = 1; b < kBlocks; ++b) {  // (the first runs with the stem: block_rows_f16.hip)
    p.c[b] = kChannels[b - 1] * q / 4, p.n[b] = kChannels[b] * q / 4;
    const int out = (hw + kStrides[b] - 1) / kStrides[b];
    auto fits = [&](auto supported) {
      return supported((int)batch, hw, hw, p.c[b], p.n[b], kStrides[b], out, out, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
    };
    const bool patch = fits(separable_patch_f16_supported);
    const int64_t products = batch * out * out * p.c[b] * p.n[b];
    small[b] = patch && products <= kPatchProductsTwo;
    p.form[b] = patch && products <= kPatchProducts        ? kPatch
                : fits(separable_stream_f16_supported) ? kStream
                : fits(separable_tile_f16_supported)   ? kTile
                : small[b]                             ? kPatch
                                                       : kTwo;
    // The second block with the stem: us a pass, separate and together, full width 16 images 151 / 146, 64 images 257 / 253; 3/4 width 16
    // images 138 / 130, 64 of 192 x 192 218 / 203.  Half width, 32 images 132 / 131, quarter width, 64 of 160 x 160 107 / 115.  The two cross
    // between one image (full width 67.6 / 68.2) and 8 (126.5 / 122); the line lies behind 8 because a pass of up to 8 images and its
    // feature maps have a launch for each block, which costs 3.6 % there.
    if (b == 1 && q >= 3 && batch * out * out >= 30000) p.form[b] = kStem;
    if (p.form[b] == kTile) {
      ++p.tiles;
      p.packed[b] = p.packed_halfs;
      p.packed_halfs += align_up((size_t)p.c[b] * p.n[b] * sizeof(uint16_t)) / sizeof(uint16_t);
    }
    hw = out;
  }
  if (p.tiles < 3) {
    for (int b = 1; b < kBlocks; ++b)
      if (p.form[b] == kTile) p.form[b] = small[b] ? kPatch : kTwo;
    p.tiles = 0, p.packed_halfs = 0;
  }
  return p;
}

// The same for fp32.  kBlock: patches with the whole block in registers (block.hip), one to three images.  One image's pass is chained;
// where it stops at a feature map or may not be chained, its blocks take kBlock, kStream or kTwo.
enum BlockForm32 { kTwo32, kPatch32, kBlock32, kStream32, kTile32, kStem32 };
struct BlockPlan32 {
  BlockForm32 form[kBlocks], without[kBlocks];  // without: what a tile block is where there is no room for its filter
  int tiles, c[kBlocks], n[kBlocks];
  size_t packed[kBlocks], packed_bytes;  // the tile blocks' filters
  void drop_tiles() {
    for (int b = 0; b < kBlocks; ++b) form[b] = without[b];
    tiles = 0, packed_bytes = 0;
  }
};
BlockPlan32 plan_blocks(const tfx_mobilenet_v1_variant& v, int64_t batch) {
  BlockPlan32 p{};
  const int q = (int)v.width_quarters;
  int hw = (int)(v.image_size + 1) / 2;
  for (int b = 0; b < kBlocks; ++b) {
    const int c = p.c[b] = b == 0 ? kStemChannels * q / 4 : kChannels[b - 1] * q / 4, n = p.n[b] = kChannels[b] * q / 4, s = kStrides[b];
    const int out = (hw + s - 1) / s;
    auto fits = [&](auto supported) {
      return supported((int)batch, hw, hw, c, n, s, out, out, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
    };
    // The tile form takes the blocks of two launches with many outputs.  Of 1346 such blocks (336 passes: 2 - 64 images of 64 x 64 to
    // 224 x 224, every width) it is faster for 606 of the 608 from these lines on, .62 of their time (512 -> 512, 64 images 35 us
    // against 66, 8 images 12 and 18), and pays for the launch that prepares the filters in every one of the passes; it is slower for
    // 505 of the others, 1.18 times on average (512 -> 512, 32 pixels 9.8 and 6.2; as tiles they made the pass of 2 images of 64 x 64
    // 128 us instead of 82).  Below the lines for up to 384 channels its sums are also the less exact ones: the products of two
    // launches split the contraction there (256 -> 256, 2400 pixels 1.2e-7 against float64 and 1.0e-7; 192 -> 192, 10496 pixels 1.3
    // and 1.1; above them 1.3 and 2.0 for the kernels that it replaced; 96 -> 192, 12544 pixels 1.2e-7 and .9, 15680 pixels 1.2 and 1.3).
    // And the window kernel's 128 -> 128 where that has less than half a round of units (0.44 of 2048: 9.7 us against 14.1; from
    // there on 19.5 against 16.3 to 67.6 against 71.7 at six rounds).  The patch kernel and the window kernel's thinner filters keep
    // their blocks: their sums are the more accurate ones.
    const bool tile = batch > 1 && fits(separable_tile_supported);
    const bool many = batch * out * out * n >= (c >= 512 ? 400000 : n >= 256 ? 800000 : c >= 192 ? 2100000 : 3000000);
    const int64_t units = batch * ((out + 1) / 2) * ((out + 7) / 8);
    const bool wide = c == 128 && n == 128 && units <= 1024;
    p.without[b] = batch > 1 && separable_patch_pays((int)batch, c, n, s, out, out) && fits(separable_patch_supported) ? kPatch32
                   : separable_block_supported(batch, hw, hw, c, n, s, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr) ? kBlock32
                   : fits(separable_stream_supported) ? kStream32
                                                      : kTwo32;
    p.form[b] = tile && (p.without[b] == kTwo32 ? many : wide && p.without[b] == kStream32) ? kTile32 : p.without[b];
    // The second block with the stem, us a pass, separate and together: full width 3 images 147 / 143, 8 191 / 187, 64 570 / 523; 3/4 width
    // 16 of 192 x 192 221 / 201; half width 32 200 / 194; quarter width 32 155 / 138.  Below 9000 pixels few strips of few rows, which
    // compute most of theirs twice: 2 images 110 / 111, 4 of 128 x 128 96 / 100, 3 of 96 x 96 87 / 93.
    if (b == 1 && batch > 1 && batch * out * out >= 9000 && stem_two_blocks_supported(hw, q)) p.form[b] = p.without[b] = kStem32;
    if (p.form[b] == kTile32) ++p.tiles;
    // (room for the wide block's at any batch: a workspace is large enough for every smaller batch, one image apart)
    if (p.form[b] == kTile32 || (tile && c == 128 && n == 128 && p.form[b] == kStream32)) {
      p.packed[b] = p.packed_bytes;
      p.packed_bytes += align_up(separable_tile_packed_bytes(c, n));
    }
    hw = out;
  }
  return p;
}

// Workspace of tfx_mobilenet_v1_variant_forward_static: it lives in the library's code object, one copy per
// GPU, from the moment the library is loaded on that GPU until the process ends.
constexpr size_t kStaticScratchBytes = size_t(16) << 20;

struct NetPlan {
  size_t act_floats;  // per ping-pong buffer
  size_t off_buf[2], off_partial, off_chain, off_head, off_packed, bytes;  // off_packed: BlockPlan, BlockPlan32
  BlockPlan32 blocks;  // fp32
  bool chain;         // one image: room for the chained small-map kernel (chain.hip)
  bool head;          // and for blocks 2 - 4 as stages of one launch (block.hip): their three outputs at once
};

// most: a workspace whose size is given (the static one); an fp32 pass that fits it only without the tile blocks' filters goes without.
NetPlan plan_net(const tfx_mobilenet_v1_variant& v, int64_t batch, size_t elem_bytes = sizeof(float), size_t most = 0) {
  NetPlan p{};
  // largest feature map: the output of the first pointwise layer (half the image size, 64 alpha channels)
  const size_t half = (size_t)(v.image_size + 1) / 2;
  p.act_floats = (size_t)batch * half * half * (size_t)(kChannels[0] * v.width_quarters / 4);
  size_t off = 0;
  for (int i = 0; i < 2; ++i) {
    p.off_buf[i] = off;
    off = align_up(off + p.act_floats * elem_bytes);
  }
  p.off_partial = off;  // K-slice partial sums of the fully connected layer
  off = align_up(off + fc_partial_floats((int)batch, (int)(kFeatures * v.width_quarters / 4), (int)v.classes) * sizeof(float));
  p.off_chain = off;
  p.chain = elem_bytes == sizeof(float) && chain_supported((int)v.image_size, (int)v.width_quarters, (int)v.classes, batch);
  if (p.chain) off = align_up(off + chain_workspace_bytes((int)v.image_size, (int)v.classes, (int)v.width_quarters));
  // blocks 2 - 4 in one launch: the outputs of blocks 2 and 3 share the second ping-pong buffer, the output of block 4
  // (1/8-size map, 256 channels) gets a region of its own, because block 2 is still reading the first buffer; the
  // output of block 5 (a launch of its own) goes behind it
  const size_t quarter = (half + 1) / 2, eighth = (quarter + 1) / 2;
  p.off_head = off;
  p.head = p.chain && v.width_quarters == 4 && 2 * quarter * quarter * 128 <= p.act_floats;
  if (p.head) off = align_up(off + 2 * eighth * eighth * 256 * sizeof(float));  // outputs of blocks 4 and 5
  p.off_packed = off;
  if (elem_bytes == sizeof(uint16_t)) {
    off += plan_blocks_f16(v, batch).packed_halfs * sizeof(uint16_t);
    p.chain = chain_supported((int)v.image_size, (int)v.width_quarters, (int)v.classes, batch);
    if (p.chain) {
      p.off_chain = align_up(off);
      off = p.off_chain + chain_workspace_bytes_f16((int)v.image_size, (int)v.classes, (int)v.width_quarters);
    }
  } else {
    p.blocks = plan_blocks(v, batch);
    if (off <= most && off + p.blocks.packed_bytes > most) p.blocks.drop_tiles();
    off += p.blocks.packed_bytes;
  }
  p.bytes = off;
  return p;
}

constexpr tfx_mobilenet_v1_variant kBaseVariant = {kImage, 4, kClasses};

constexpr int kMaxDevices = 64;

}  // namespace
}  // namespace tfx

static __device__ __align__(256) unsigned char scratch[tfx::kStaticScratchBytes];

namespace tfx {
namespace {

// Device address of `scratch` on the calling thread's current device.  In host code the array's name is only a
// handle for the runtime; the address kernels can use is looked up once per device and kept.  Returns null if the
// lookup fails.  Safe to call from several threads (the lookup is idempotent).
void* static_scratch() {
  static std::atomic<void*> ptr[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  void* p = ptr[dev].load(std::memory_order_acquire);
  if (p) return p;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
  ptr[dev].store(p, std::memory_order_release);
  return p;
}

}  // namespace
}  // namespace tfx

using namespace tfx;

extern "C" {

const char* tfx_status_string(int status) {
  switch (status) {
    case TFX_OK: return "TFX_OK";
    case TFX_ERR_NULL: return "TFX_ERR_NULL: null pointer argument";
    case TFX_ERR_SHAPE: return "TFX_ERR_SHAPE: non-positive or mismatching dimensions";
    case TFX_ERR_ARG: return "TFX_ERR_ARG: bad stride or enum value";
    case TFX_ERR_UNSUPPORTED: return "TFX_ERR_UNSUPPORTED: tensor too large";
    case TFX_ERR_WORKSPACE: return "TFX_ERR_WORKSPACE: workspace too small or misaligned";
    case TFX_ERR_LAUNCH: return "TFX_ERR_LAUNCH: kernel enqueue failed";
    default: return "unknown tfx status";
  }
}

int tfx_matmul_out_shape(const int64_t a_shape[2], const int64_t b_shape[2], int transpose_a, int transpose_b,
                         int64_t out_shape[2]) {
  if (!a_shape || !b_shape || !out_shape) return TFX_ERR_NULL;
  int64_t m, n, k;
  int rc = matmul_geometry(a_shape, b_shape, transpose_a, transpose_b, &m, &n, &k);
  if (rc) return rc;
  out_shape[0] = m;
  out_shape[1] = n;
  return TFX_OK;
}

int tfx_conv2d_out_shape(const int64_t x_shape[4], const int64_t f_shape[4], int stride_h, int stride_w,
                         tfx_padding pad, int64_t out_shape[4], int64_t pad_tblr[4]) {
  if (!x_shape || !f_shape || !out_shape || !pad_tblr) return TFX_ERR_NULL;
  ConvGeom g;
  int rc = conv_geometry(x_shape, f_shape, stride_h, stride_w, (int)pad, false, &g);
  if (rc) return rc;
  for (int i = 0; i < 4; ++i) {
    out_shape[i] = g.out[i];
    pad_tblr[i] = g.pad[i];
  }
  return TFX_OK;
}

int tfx_depthwise_conv2d_out_shape(const int64_t x_shape[4], const int64_t f_shape[4], int stride_h, int stride_w,
                                   tfx_padding pad, int64_t out_shape[4], int64_t pad_tblr[4]) {
  if (!x_shape || !f_shape || !out_shape || !pad_tblr) return TFX_ERR_NULL;
  ConvGeom g;
  int rc = conv_geometry(x_shape, f_shape, stride_h, stride_w, (int)pad, true, &g);
  if (rc) return rc;
  for (int i = 0; i < 4; ++i) {
    out_shape[i] = g.out[i];
    pad_tblr[i] = g.pad[i];
  }
  return TFX_OK;
}

int tfx_matmul(const float* a, const int64_t a_shape[2], const float* b, const int64_t b_shape[2], int transpose_a,
               int transpose_b, float* c, void* stream) {
  if (!a || !b || !c || !a_shape || !b_shape) return TFX_ERR_NULL;
  return batch_matmul_impl(a, a_shape, b, b_shape, 1, transpose_a, transpose_b, c, stream);
}

int tfx_batch_matmul(const float* a, const int64_t a_shape[3], const float* b, const int64_t b_shape[3],
                     int transpose_a, int transpose_b, float* c, void* stream) {
  if (!a || !b || !c || !a_shape || !b_shape) return TFX_ERR_NULL;
  if (a_shape[0] < 1 || a_shape[0] != b_shape[0]) return TFX_ERR_SHAPE;
  return batch_matmul_impl(a, a_shape + 1, b, b_shape + 1, a_shape[0], transpose_a, transpose_b, c, stream);
}

int tfx_conv2d(const float* x, const int64_t x_shape[4], const float* filter, const int64_t f_shape[4],
               const float* bias, int stride_h, int stride_w, tfx_padding pad, tfx_activation act, float* y,
               void* stream) {
  if (!x || !filter || !y || !x_shape || !f_shape) return TFX_ERR_NULL;
  ConvGeom g;
  int rc = conv_geometry(x_shape, f_shape, stride_h, stride_w, (int)pad, false, &g);
  if (rc) return rc;
  if (!valid_act((int)act)) return TFX_ERR_ARG;
  if (numel(x_shape, 4) < 0 || numel(f_shape, 4) < 0 || numel(g.out, 4) < 0) return TFX_ERR_UNSUPPORTED;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int n = (int)x_shape[0], h = (int)x_shape[1], w = (int)x_shape[2], ci = (int)x_shape[3];
  const int fh = (int)f_shape[0], fw = (int)f_shape[1], co = (int)f_shape[3];
  const int oh = (int)g.out[1], ow = (int)g.out[2];
  if (fh == 1 && fw == 1 && stride_h == 1 && stride_w == 1) {
    // pointwise convolution = [N*H*W, Ci] x [Ci, Co] with the epilogue fused into the GEMM
    if (pointwise_stream_supported(n * h * w, ci, co, x, filter, bias, y))
      return launch_pointwise_stream(x, filter, bias, y, n * h * w, ci, co, (int)act, s);
    return launch_gemm(x, filter, y, bias, 1, n * h * w, co, ci, true, false, (int)act, s);
  }
  const bool aligned = reinterpret_cast<uintptr_t>(y) % 16 == 0;
  if (conv2d_stem_supported(ci, fh, fw, co, stride_h, stride_w) && aligned)
    return launch_conv2d_stem(x, filter, bias, y, n, h, w, co, oh, ow, stride_h, stride_w, (int)g.pad[0], (int)g.pad[2],
                              (int)act, s);
  if (conv2d_gemm_supported(numel(x_shape, 4), fh, fw, ci, co))
    return launch_conv2d_gemm(x, filter, bias, y, n, h, w, ci, fh, fw, co, oh, ow, stride_h, stride_w, (int)g.pad[0],
                              (int)g.pad[2], (int)act, s);
  return launch_conv2d_direct(x, filter, bias, y, n, h, w, ci, fh, fw, co, oh, ow, stride_h, stride_w, (int)g.pad[0],
                              (int)g.pad[2], (int)act, s);
}

int tfx_depthwise_conv2d(const float* x, const int64_t x_shape[4], const float* filter, const int64_t f_shape[4],
                         const float* bias, int stride_h, int stride_w, tfx_padding pad, tfx_activation act, float* y,
                         void* stream) {
  if (!x || !filter || !y || !x_shape || !f_shape) return TFX_ERR_NULL;
  ConvGeom g;
  int rc = conv_geometry(x_shape, f_shape, stride_h, stride_w, (int)pad, true, &g);
  if (rc) return rc;
  if (!valid_act((int)act)) return TFX_ERR_ARG;
  if (numel(x_shape, 4) < 0 || numel(f_shape, 4) < 0 || numel(g.out, 4) < 0) return TFX_ERR_UNSUPPORTED;
  return launch_depthwise(x, filter, bias, y, (int)x_shape[0], (int)x_shape[1], (int)x_shape[2], (int)x_shape[3],
                          (int)f_shape[0], (int)f_shape[1], (int)f_shape[3], (int)g.out[1], (int)g.out[2], stride_h,
                          stride_w, (int)g.pad[0], (int)g.pad[2], (int)act, static_cast<hipStream_t>(stream));
}

int tfx_add(const float* a, const float* b, int64_t n, float* c, void* stream) {
  if (n < 0) return TFX_ERR_SHAPE;
  if (n == 0) return TFX_OK;
  if (!a || !b || !c) return TFX_ERR_NULL;
  if (n > (int64_t(1) << 40)) return TFX_ERR_UNSUPPORTED;
  return launch_add_f32(a, b, c, n, static_cast<hipStream_t>(stream));
}

int tfx_add_f16(const uint16_t* a, const uint16_t* b, int64_t n, uint16_t* c, void* stream) {
  if (n < 0) return TFX_ERR_SHAPE;
  if (n == 0) return TFX_OK;
  if (!a || !b || !c) return TFX_ERR_NULL;
  if (n > (int64_t(1) << 40)) return TFX_ERR_UNSUPPORTED;
  return launch_add_f16(a, b, c, n, static_cast<hipStream_t>(stream));
}

int tfx_batch_matmul_f16(const uint16_t* a, const int64_t a_shape[3], const uint16_t* b, const int64_t b_shape[3],
                         int transpose_a, int transpose_b, const uint16_t* bias, tfx_activation act, uint16_t* c,
                         void* stream) {
  if (!a || !b || !c || !a_shape || !b_shape) return TFX_ERR_NULL;
  if (!valid_act((int)act)) return TFX_ERR_ARG;
  if (a_shape[0] < 1 || a_shape[0] != b_shape[0]) return TFX_ERR_SHAPE;
  int64_t m, n, k;
  int rc = matmul_geometry(a_shape + 1, b_shape + 1, transpose_a, transpose_b, &m, &n, &k);
  if (rc) return rc;
  const int64_t batch = a_shape[0];
  const int64_t da[3] = {batch, m, k}, db[3] = {batch, n, k}, dc[3] = {batch, m, n};
  if (numel(da, 3) < 0 || numel(db, 3) < 0 || numel(dc, 3) < 0) return TFX_ERR_UNSUPPORTED;
  return launch_gemm_f16(a, b, c, bias, (int)batch, (int)m, (int)n, (int)k, !transpose_a, transpose_b != 0, (int)act,
                         static_cast<hipStream_t>(stream));
}

int tfx_conv2d_f16(const uint16_t* x, const int64_t x_shape[4], const uint16_t* filter, const int64_t f_shape[4],
                   const uint16_t* bias, int stride_h, int stride_w, tfx_padding pad, tfx_activation act, uint16_t* y,
                   void* stream) {
  if (!x || !filter || !y || !x_shape || !f_shape) return TFX_ERR_NULL;
  if (!valid_act((int)act)) return TFX_ERR_ARG;
  ConvGeom g;
  int rc = conv_geometry(x_shape, f_shape, stride_h, stride_w, (int)pad, false, &g);
  if (rc) return rc;
  if (numel(x_shape, 4) < 0 || numel(f_shape, 4) < 0 || numel(g.out, 4) < 0) return TFX_ERR_UNSUPPORTED;
  const int n = (int)x_shape[0], h = (int)x_shape[1], w = (int)x_shape[2], ci = (int)x_shape[3];
  const int fh = (int)f_shape[0], fw = (int)f_shape[1], co = (int)f_shape[3];
  const int oh = (int)g.out[1], ow = (int)g.out[2];
  hipStream_t s = static_cast<hipStream_t>(stream);
  // a 1x1 stride-1 convolution is the matMul of the pixel rows [n*h*w, ci] with the filter [ci, co]
  if (fh == 1 && fw == 1 && stride_h == 1 && stride_w == 1)
    return launch_gemm_f16(x, filter, y, bias, 1, n * h * w, co, ci, true, false, (int)act, s);
  if (conv2d_stem_f16_supported(ci, fh, fw, co, y))
    return launch_conv2d_stem_f16(x, filter, bias, y, n, h, w, co, oh, ow, stride_h, stride_w, (int)g.pad[0],
                                  (int)g.pad[2], (int)act, s);
  if (conv3x3_stream_f16_supported((long long)n * oh * ow, numel(x_shape, 4), ci, fh, fw, co, stride_h, stride_w, x,
                                   filter, y))
    return launch_conv3x3_stream_f16(x, filter, bias, y, n, h, w, ci, co, oh, ow, (int)g.pad[0], (int)g.pad[2],
                                     (int)act, s);
  if (conv2d_gemm_f16_supported(numel(x_shape, 4), fh, fw, ci, co))
    return launch_conv2d_gemm_f16(x, filter, bias, y, n, h, w, ci, fh, fw, co, oh, ow, stride_h, stride_w,
                                  (int)g.pad[0], (int)g.pad[2], (int)act, s);
  return launch_conv2d_direct_f16(x, filter, bias, y, n, h, w, ci, fh, fw, co, oh, ow, stride_h, stride_w,
                                  (int)g.pad[0], (int)g.pad[2], (int)act, s);
}

int tfx_depthwise_conv2d_f16(const uint16_t* x, const int64_t x_shape[4], const uint16_t* filter,
                             const int64_t f_shape[4], const uint16_t* bias, int stride_h, int stride_w,
                             tfx_padding pad, tfx_activation act, uint16_t* y, void* stream) {
  if (!x || !filter || !y || !x_shape || !f_shape) return TFX_ERR_NULL;
  if (!valid_act((int)act)) return TFX_ERR_ARG;
  ConvGeom g;
  int rc = conv_geometry(x_shape, f_shape, stride_h, stride_w, (int)pad, true, &g);
  if (rc) return rc;
  if (numel(x_shape, 4) < 0 || numel(f_shape, 4) < 0 || numel(g.out, 4) < 0) return TFX_ERR_UNSUPPORTED;
  return launch_depthwise_f16(x, filter, bias, y, (int)x_shape[0], (int)x_shape[1], (int)x_shape[2], (int)x_shape[3],
                              (int)f_shape[0], (int)f_shape[1], (int)f_shape[3], (int)g.out[1], (int)g.out[2], stride_h,
                              stride_w, (int)g.pad[0], (int)g.pad[2], (int)act, static_cast<hipStream_t>(stream));
}

size_t tfx_mobilenet_v1_workspace_bytes(int64_t batch) {
  if (batch < 1 || batch > 1024) return 0;
  return plan_net(kBaseVariant, batch).bytes;
}

int tfx_mobilenet_v1_forward(const float* input, int64_t batch, const tfx_mobilenet_v1_weights* weights,
                             void* workspace, size_t workspace_bytes, float* probs, float* logits, void* stream) {
  return tfx_mobilenet_v1_variant_forward(&kBaseVariant, input, batch, weights, workspace, workspace_bytes, probs,
                                          logits, stream);
}

size_t tfx_mobilenet_v1_variant_workspace_bytes(const tfx_mobilenet_v1_variant* variant, int64_t batch) {
  if (!valid_variant(variant) || batch < 1 || batch > 1024) return 0;
  return plan_net(*variant, batch).bytes;
}

namespace {
// The checks of a forward pass's arguments that come before the workspace's, in their order.
int check_net_args(const tfx_mobilenet_v1_variant* variant, const float* input, int64_t batch,
                   const tfx_mobilenet_v1_weights* weights, const void* workspace, const void* out) {
  if (!variant || !input || !weights || !workspace || !out) return TFX_ERR_NULL;
  if (!weights->conv0_w || !weights->conv0_b || !weights->fc_w || !weights->fc_b) return TFX_ERR_NULL;
  for (int i = 0; i < kBlocks; ++i)
    if (!weights->dw_w[i] || !weights->dw_b[i] || !weights->pw_w[i] || !weights->pw_b[i]) return TFX_ERR_NULL;
  if (!valid_variant(variant)) return TFX_ERR_ARG;
  if (batch < 1) return TFX_ERR_SHAPE;
  if (batch > 1024) return TFX_ERR_UNSUPPORTED;
  return TFX_OK;
}

// The forward pass; end_block = 0: the whole network into probs / logits; end_block = 1 .. 13: stop after that
// depthwise-separable block, whose output goes to `features` instead of the workspace.  most: plan_net's.
int forward_impl(const tfx_mobilenet_v1_variant* variant, const float* input, int64_t batch,
                 const tfx_mobilenet_v1_weights* weights, void* workspace, size_t workspace_bytes, float* probs,
                 float* logits, int end_block, float* features, void* stream, size_t most = 0) {
  if (const int bad = check_net_args(variant, input, batch, weights, workspace,
                                     end_block == 0 ? (const void*)probs : (const void*)features))
    return bad;
  const NetPlan plan = plan_net(*variant, batch, sizeof(float), most);
  if (workspace_bytes < plan.bytes || reinterpret_cast<uintptr_t>(workspace) % kAlign != 0) return TFX_ERR_WORKSPACE;
  const int q = (int)variant->width_quarters;

  char* ws = static_cast<char*>(workspace);
  float* buf[2] = {reinterpret_cast<float*>(ws + plan.off_buf[0]), reinterpret_cast<float*>(ws + plan.off_buf[1])};
  float* partial = reinterpret_cast<float*>(ws + plan.off_partial);

  // Batch 1: the blocks from the last 1/8-size map on, the pool, the fully connected layer and the
  // softmax run as one persistent kernel (chain.hip) when every pointer allows its vector loads and 256 of its
  // workgroups are resident at once on this device; what its tasks wait for is prepared by the first kernel of the pass
  // (the stem of launch_conv2d_stem or of launch_stem_block; launch_stem_block_rows clears none).
  bool flags_ok = plan.chain;  // the workspace has the flag region, and the kernels that use it may run
  if (flags_ok) {
    auto al16 = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
    flags_ok = al16(input) && al16(weights->conv0_b) && al16(weights->fc_w) && al16(weights->fc_b);
    for (int i = 0; i < kBlocks && flags_ok; ++i)
      flags_ok = al16(weights->dw_w[i]) && al16(weights->dw_b[i]) && al16(weights->pw_w[i]) && al16(weights->pw_b[i]);
    flags_ok = flags_ok && chain_grids(q) > 0;
  }
  const bool chain = flags_ok && end_block == 0;
  // blocks 2 - 4 as stages of one launch and block 5 as a launch (block.hip): in the whole pass and when block 4's
  // or block 5's output is asked for
  const bool head_chain = flags_ok && plan.head && (end_block == 0 || end_block == 4 || end_block == 5);
  bool flags_cleared = false;  // by the first kernel, for the launches that wait for flags
  void* chain_ws = ws + plan.off_chain;
  ChainClear clear;
  if (chain || head_chain) {
    clear = ChainClear{static_cast<int*>(chain_ws), chain_flag_words((int)variant->image_size), block_chain_flag_stride(), nullptr, 0};
    if (chain) {
      const ChainFill fill = chain_fill((int)variant->image_size, (int)variant->classes, q, 4, chain_ws);
      clear.fill = static_cast<uint4*>(fill.at), clear.fill_pieces = (unsigned)(fill.bytes / 16);
    }
  }

  const int blocks = end_block ? end_block : kBlocks;
  const BlockPlan32& form = plan.blocks;  // of the whole network: a feature map is the one a pass computes
  auto aligned = [&](int b) {  // else the block runs as two launches, which take any element
    bool ok = true;
    for (const void* p : {weights->dw_w[b], weights->dw_b[b], weights->pw_w[b], weights->pw_b[b]})
      ok = ok && reinterpret_cast<uintptr_t>(p) % 16 == 0;
    return ok;
  };
  PackList filters;  // of the tile blocks, in their order from the stem's launch on (more than one image)
  for (int b = 1; b < blocks; ++b)
    if (form.tiles > 0 && form.form[b] == kTile32 && aligned(b)) filters.add(weights->pw_w[b], ws + plan.off_packed + form.packed[b], form.c[b], form.n[b]);

  // stem: 3x3 stride-2 convolution to 32 alpha channels, then the 13 depthwise-separable blocks
  int64_t shape[4] = {batch, variant->image_size, variant->image_size, 3};
  const int64_t f0[4] = {3, 3, 3, kStemChannels * q / 4};
  ConvGeom g;
  conv_geometry(shape, f0, 2, 2, TFX_PAD_SAME, false, &g);
  int rc;
  int first_block = 0;
  const int64_t c0 = kChannels[0] * q / 4;
  if (batch == 1 &&
      stem_block_supported((int)shape[1], (int)shape[2], (int)f0[3], (int)c0, input, weights->conv0_w,
                           weights->conv0_b, weights->dw_w[0], weights->dw_b[0], weights->pw_w[0], weights->pw_b[0],
                           end_block == 1 ? features : buf[0])) {
    // one image: stem and first block in one launch of patches (block.hip), which also prepares what later launches wait for
    rc = launch_stem_block(input, weights->conv0_w, weights->conv0_b, weights->dw_w[0], weights->dw_b[0],
                           weights->pw_w[0], weights->pw_b[0], end_block == 1 ? features : buf[0], (int)shape[1],
                           (int)shape[2], (int)g.out[1],
                           (int)g.out[2], (int)g.pad[0], (int)g.pad[2], (int)c0, TFX_ACT_RELU6,
                           static_cast<hipStream_t>(stream), chain || head_chain ? clear : ChainClear());
    first_block = 1;
    flags_cleared = chain || head_chain;
  } else if (chain) {
    rc = launch_conv2d_stem(input, weights->conv0_w, weights->conv0_b, buf[0], 1, (int)shape[1], (int)shape[2],
                            (int)f0[3], (int)g.out[1], (int)g.out[2], 2, 2, (int)g.pad[0], (int)g.pad[2], TFX_ACT_RELU6,
                            static_cast<hipStream_t>(stream), clear);
    flags_cleared = true;
  } else {
    // stem and first block in one launch that walks down rows (block_rows.hip)
    // (and the second, which the plan then says)
    const int64_t fd2[4] = {3, 3, c0, 1}, map[4] = {batch, g.out[1], g.out[2], c0};
    ConvGeom g2;
    conv_geometry(map, fd2, kStrides[1], kStrides[1], TFX_PAD_SAME, true, &g2);
    const SecondBlock<float> second{weights->dw_w[1], weights->dw_b[1], weights->pw_w[1], weights->pw_b[1],
                                    (int)g2.out[1], (int)g2.out[2], (int)g2.pad[0], (int)g2.pad[2]};
    first_block = plan.blocks.form[1] == kStem32 && end_block != 1 ? 2 : 1;
    rc = launch_stem_block_rows(input, weights->conv0_w, weights->conv0_b, weights->dw_w[0], weights->dw_b[0], weights->pw_w[0],
                                weights->pw_b[0], end_block == first_block ? features : buf[0], (int)batch, (int)shape[1], (int)shape[2],
                                (int)g.out[1], (int)g.out[2], (int)g.pad[0], (int)g.pad[2], q, static_cast<hipStream_t>(stream),
                                first_block == 2 ? &second : nullptr, filters);
    if (first_block == 2) g = g2;
  }
  if (rc) return rc;
  for (int i = 0; i < 4; ++i) shape[i] = g.out[i];
  if (first_block > 0) shape[3] = kChannels[first_block - 1] * q / 4;
  if (first_block > 0 && end_block == first_block) return TFX_OK;
  int cur = 0;
  if (head_chain && flags_cleared && first_block == 1) {
    // blocks 2 - 4 as three stages of one launch, block 5 as a launch of its own, then the chained kernel from block 6
    // on; flags (cleared by the first kernel) and failure word are shared with it
    const size_t quarter = (size_t)((shape[1] + 1) / 2), eighth = (quarter + 1) / 2;
    float* const region = reinterpret_cast<float*>(ws + plan.off_head);
    float* const b2_out = buf[1];
    float* const b3_out = buf[1] + quarter * quarter * 128;
    float* const b4_out = end_block == 4 ? features : region;
    float* const b5_out = end_block == 5 ? features : region + eighth * eighth * 256;
    const bool with_b5 = end_block != 4 && separable_block_supported(1, (int)eighth, (int)eighth, 256, 256, 1, b4_out,
                                                                  weights->dw_w[4], weights->dw_b[4], weights->pw_w[4],
                                                                  weights->pw_b[4], b5_out);
    if (block_chain_supported(buf[0], b2_out, b3_out, b4_out, weights) && (with_b5 || end_block == 4)) {
      struct Head {
        const float* x;
        float *b2, *b3, *b4, *b5;
        int h, w, eighth;
        bool with_b5;
        const tfx_mobilenet_v1_weights* wt;
        int* flags;
        int flag_base;
        hipStream_t stream;
      } head{buf[0], b2_out, b3_out, b4_out, b5_out, (int)shape[1], (int)shape[2], (int)eighth, with_b5, weights,
             static_cast<int*>(chain_ws), 1,
             static_cast<hipStream_t>(stream)};
      auto launch_head = [](void* p) -> int {
        const Head& a = *static_cast<const Head*>(p);
        const int rc = launch_block_chain(a.x, a.b2, a.b3, a.b4, a.h, a.w, a.wt, a.flags, a.flag_base, chain_spin_limit(), a.stream);
        if (rc != TFX_OK || !a.with_b5) return rc;
        // 28 x 28 x 256 -> 256, stride 1, SAME: one zero row / column before the map
        return launch_separable_block(a.b4, a.wt->dw_w[4], a.wt->dw_b[4], a.wt->pw_w[4], a.wt->pw_b[4], a.b5, 1, a.eighth, a.eighth,
                                      256, 256, a.eighth, a.eighth, 1, 1, 1, TFX_ACT_RELU6, TFX_ACT_RELU6, a.stream);
      };
      if (end_block != 0) return launch_ordered(static_cast<hipStream_t>(stream), launch_head, &head);
      return launch_chain(b5_out, (int)variant->image_size, weights, chain_ws, probs, logits, (int)variant->classes, q,
                          static_cast<hipStream_t>(stream), launch_head, &head, 5);
    }
  }
  for (int b = first_block; b < blocks; ++b) {
    float* const block_out = end_block == b + 1 ? features : buf[cur ^ 1];
    if (chain && b == 4)
      return launch_chain(buf[cur], (int)variant->image_size, weights, chain_ws, probs, logits, (int)variant->classes, q,
                          static_cast<hipStream_t>(stream));
    const int64_t fd[4] = {3, 3, shape[3], 1};
    const int64_t cout = kChannels[b] * q / 4;
    conv_geometry(shape, fd, kStrides[b], kStrides[b], TFX_PAD_SAME, true, &g);
    if (form.form[b] != kTwo32 && aligned(b)) {
      if (form.form[b] == kTile32) {
        rc = launch_separable_tile(buf[cur], weights->dw_w[b], weights->dw_b[b], weights->pw_w[b], weights->pw_b[b],
                                   ws + plan.off_packed + form.packed[b], block_out, (int)batch, (int)shape[1], (int)shape[2], (int)shape[3],
                                   (int)cout, (int)g.out[1], (int)g.out[2], kStrides[b], (int)g.pad[0], (int)g.pad[2], TFX_ACT_RELU6,
                                   static_cast<hipStream_t>(stream));
      } else {
        const auto launch = form.form[b] == kPatch32   ? launch_separable_patch
                            : form.form[b] == kBlock32 ? launch_separable_block
                                                       : launch_separable_stream;
        rc = launch(buf[cur], weights->dw_w[b], weights->dw_b[b], weights->pw_w[b], weights->pw_b[b], block_out, (int)batch,
                    (int)shape[1], (int)shape[2], (int)shape[3], (int)cout, (int)g.out[1], (int)g.out[2], kStrides[b], (int)g.pad[0],
                    (int)g.pad[2], TFX_ACT_RELU6, TFX_ACT_RELU6, static_cast<hipStream_t>(stream));
      }
      if (rc) return rc;
      if (end_block == b + 1) return TFX_OK;
      for (int i = 0; i < 3; ++i) shape[i] = g.out[i];
      shape[3] = cout;
      cur ^= 1;
      continue;
    }
    rc = tfx_depthwise_conv2d(buf[cur], shape, weights->dw_w[b], fd, weights->dw_b[b], kStrides[b], kStrides[b],
                              TFX_PAD_SAME, TFX_ACT_RELU6, buf[cur ^ 1], stream);
    if (rc) return rc;
    for (int i = 0; i < 4; ++i) shape[i] = g.out[i];
    cur ^= 1;
    const int64_t fp[4] = {1, 1, shape[3], cout};
    rc = tfx_conv2d(buf[cur], shape, weights->pw_w[b], fp, weights->pw_b[b], 1, 1, TFX_PAD_SAME, TFX_ACT_RELU6,
                    end_block == b + 1 ? features : buf[cur ^ 1], stream);
    if (rc) return rc;
    if (end_block == b + 1) return TFX_OK;
    shape[3] = cout;
    cur ^= 1;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  return launch_pool_fc_softmax(buf[cur], weights->fc_w, weights->fc_b, partial, logits, probs, (int)batch,
                                (int)(shape[1] * shape[2]), (int)shape[3], (int)variant->classes, s);
}
}  // namespace

int tfx_mobilenet_v1_variant_forward(const tfx_mobilenet_v1_variant* variant, const float* input, int64_t batch,
                                     const tfx_mobilenet_v1_weights* weights, void* workspace,
                                     size_t workspace_bytes, float* probs, float* logits, void* stream) {
  return forward_impl(variant, input, batch, weights, workspace, workspace_bytes, probs, logits, 0, nullptr, stream);
}

int tfx_mobilenet_v1_variant_features_shape(const tfx_mobilenet_v1_variant* variant, int64_t batch, int end_block,
                                            int64_t shape[4]) {
  if (!variant || !shape) return TFX_ERR_NULL;
  if (!valid_variant(variant) || end_block < 1 || end_block > kBlocks) return TFX_ERR_ARG;
  if (batch < 1) return TFX_ERR_SHAPE;
  int64_t hw = (variant->image_size + 1) / 2;  // the stem halves the image (stride 2, SAME padding)
  for (int b = 0; b < end_block; ++b) hw = (hw + kStrides[b] - 1) / kStrides[b];
  shape[0] = batch, shape[1] = hw, shape[2] = hw, shape[3] = kChannels[end_block - 1] * variant->width_quarters / 4;
  return TFX_OK;
}

int tfx_mobilenet_v1_variant_features(const tfx_mobilenet_v1_variant* variant, const float* input, int64_t batch,
                                      const tfx_mobilenet_v1_weights* weights, void* workspace, size_t workspace_bytes,
                                      int end_block, float* features, void* stream) {
  if (end_block < 1 || end_block > kBlocks) return variant && input && weights && workspace && features ? TFX_ERR_ARG : TFX_ERR_NULL;
  if (features && reinterpret_cast<uintptr_t>(features) % 16 != 0) return TFX_ERR_ARG;
  return forward_impl(variant, input, batch, weights, workspace, workspace_bytes, nullptr, nullptr, end_block, features,
                      stream);
}

size_t tfx_mobilenet_v1_static_scratch_bytes(void) { return kStaticScratchBytes; }

int tfx_mobilenet_v1_variant_forward_static(const tfx_mobilenet_v1_variant* variant, const float* input, int64_t batch,
                                            const tfx_mobilenet_v1_weights* weights, float* probs, float* logits,
                                            void* stream) {
  if (!variant || !input || !weights || !probs) return TFX_ERR_NULL;
  if (!valid_variant(variant)) return TFX_ERR_ARG;
  if (batch < 1) return TFX_ERR_SHAPE;
  if (batch > 1024) return TFX_ERR_UNSUPPORTED;
  if (plan_net(*variant, batch, sizeof(float), kStaticScratchBytes).bytes > kStaticScratchBytes) return TFX_ERR_WORKSPACE;
  void* ws = static_scratch();
  if (!ws) return TFX_ERR_LAUNCH;
  // Every kernel of the forward pass writes the part of the workspace it later reads (feature maps, the fully
  // connected layer's partial sums), so nothing has to be cleared between calls.
  return forward_impl(variant, input, batch, weights, ws, kStaticScratchBytes, probs, logits, 0, nullptr, stream, kStaticScratchBytes);
}

size_t tfx_mobilenet_v1_workspace_bytes_f16(const tfx_mobilenet_v1_variant* variant, int64_t batch) {
  if (!valid_variant(variant) || batch < 1 || batch > 1024) return 0;
  // (one image may need more than a few: the chained kernel's memory)
  const size_t one = plan_net(*variant, 1, sizeof(uint16_t)).bytes, all = plan_net(*variant, batch, sizeof(uint16_t)).bytes;
  return one > all ? one : all;
}

}  // extern "C"

namespace {

// end_block = 0: the whole network; else stop after that block and write its output to `features`
int forward_f16_impl(const tfx_mobilenet_v1_variant* variant, const uint16_t* input, int64_t batch,
                     const tfx_mobilenet_v1_weights_f16* weights, void* workspace, size_t workspace_bytes,
                     uint16_t* probs, uint16_t* logits, int end_block, uint16_t* features, void* stream) {
  if (!variant || !input || !weights || !workspace || !(end_block ? (void*)features : (void*)probs)) return TFX_ERR_NULL;
  if (!weights->conv0_w || !weights->conv0_b || !weights->fc_w || !weights->fc_b) return TFX_ERR_NULL;
  for (int i = 0; i < kBlocks; ++i)
    if (!weights->dw_w[i] || !weights->dw_b[i] || !weights->pw_w[i] || !weights->pw_b[i]) return TFX_ERR_NULL;
  if (!valid_variant(variant)) return TFX_ERR_ARG;
  if (batch < 1) return TFX_ERR_SHAPE;
  if (batch > 1024) return TFX_ERR_UNSUPPORTED;
  const NetPlan plan = plan_net(*variant, batch, sizeof(uint16_t));
  if (workspace_bytes < plan.bytes || reinterpret_cast<uintptr_t>(workspace) % kAlign != 0) return TFX_ERR_WORKSPACE;
  const int q = (int)variant->width_quarters;

  char* ws = static_cast<char*>(workspace);
  uint16_t* buf[2] = {reinterpret_cast<uint16_t*>(ws + plan.off_buf[0]), reinterpret_cast<uint16_t*>(ws + plan.off_buf[1])};
  float* partial = reinterpret_cast<float*>(ws + plan.off_partial);

  hipStream_t const s = static_cast<hipStream_t>(stream);

  const int blocks = end_block ? end_block : kBlocks;
  // of the whole network: a feature map is the one a pass computes (but for the chained blocks of one image, whose last bits differ)
  const BlockPlan form = plan_blocks_f16(*variant, batch);
  bool aligned = true;
  for (int b = 0; b < blocks; ++b)
    for (const void* p : {weights->dw_w[b], weights->dw_b[b], weights->pw_w[b], weights->pw_b[b]})
      aligned = aligned && reinterpret_cast<uintptr_t>(p) % 16 == 0;
  // One image: the blocks from the fifth or sixth on and the tail as one persistent kernel, as in fp32
  const int chain_first = q == 4 ? 5 : 4;
  const bool chain = aligned && end_block == 0 && plan.chain && reinterpret_cast<uintptr_t>(weights->fc_w) % 16 == 0 && chain_grids(q, true) > 0;
  const int separate = chain ? chain_first : blocks;  // blocks that are launches
  uint16_t* const packed_base = reinterpret_cast<uint16_t*>(ws + plan.off_packed);
  if (aligned && form.tiles > 0) {
    const uint16_t* filters[kBlocks];
    uint16_t* packed[kBlocks];
    int tiles = 0, c[kBlocks], n[kBlocks];
    for (int b = 0; b < separate; ++b)
      if (form.form[b] == kTile) {
        filters[tiles] = weights->pw_w[b], packed[tiles] = packed_base + form.packed[b];
        c[tiles] = form.c[b], n[tiles] = form.n[b];
        ++tiles;
      }
    if (tiles > 0)
      if (const int rc = launch_pack_filters_f16(tiles, filters, packed, c, n, s)) return rc;
  }

  int64_t shape[4] = {batch, variant->image_size, variant->image_size, 3};
  const int64_t f0[4] = {3, 3, 3, kStemChannels * q / 4};
  ConvGeom g;
  conv_geometry(shape, f0, 2, 2, TFX_PAD_SAME, false, &g);
  const int64_t fd2[4] = {3, 3, kChannels[0] * q / 4, 1};
  const int64_t map[4] = {batch, g.out[1], g.out[2], fd2[2]};
  ConvGeom g2;
  conv_geometry(map, fd2, kStrides[1], kStrides[1], TFX_PAD_SAME, true, &g2);
  const SecondBlock<uint16_t> second{weights->dw_w[1], weights->dw_b[1], weights->pw_w[1], weights->pw_b[1],
                                     (int)g2.out[1], (int)g2.out[2], (int)g2.pad[0], (int)g2.pad[2]};
  const int leading = form.form[1] == kStem && end_block != 1 ? 2 : 1;  // blocks that come with the stem
  ChainClear clear;
  if (chain) {
    const ChainFill fill = chain_fill_f16((int)variant->image_size, (int)variant->classes, q, chain_first, ws + plan.off_chain);
    clear = ChainClear{reinterpret_cast<int*>(ws + plan.off_chain), 1, 1, static_cast<uint4*>(fill.at), (unsigned)(fill.bytes / 16)};
  }
  int rc = launch_stem_block_rows_f16(input, weights->conv0_w, weights->conv0_b, weights->dw_w[0], weights->dw_b[0], weights->pw_w[0],
                                      weights->pw_b[0], end_block == leading ? features : buf[0], (int)batch, (int)shape[1], (int)shape[2],
                                      (int)g.out[1], (int)g.out[2], (int)g.pad[0], (int)g.pad[2], q, s, leading == 2 ? &second : nullptr, clear);
  if (rc || end_block == leading) return rc;
  for (int i = 0; i < 3; ++i) shape[i] = leading == 2 ? g2.out[i] : g.out[i];
  shape[3] = kChannels[leading - 1] * q / 4;
  int cur = 0;
  for (int b = leading; b < separate; ++b) {
    const int64_t fd[4] = {3, 3, shape[3], 1};
    const int64_t cout = kChannels[b] * q / 4;
    conv_geometry(shape, fd, kStrides[b], kStrides[b], TFX_PAD_SAME, true, &g);
    if (aligned && form.form[b] != kTwo) {
      const bool tile = form.form[b] == kTile;
      const auto launch = tile ? launch_separable_tile_f16 : form.form[b] == kPatch ? launch_separable_patch_f16 : launch_separable_stream_f16;
      rc = launch(buf[cur], weights->dw_w[b], weights->dw_b[b], tile ? packed_base + form.packed[b] : weights->pw_w[b],
                  weights->pw_b[b], end_block == b + 1 ? features : buf[cur ^ 1], (int)batch, (int)shape[1], (int)shape[2],
                  (int)shape[3], (int)cout, (int)g.out[1], (int)g.out[2], kStrides[b], (int)g.pad[0], (int)g.pad[2],
                  TFX_ACT_RELU6, TFX_ACT_RELU6, s);
      if (rc) return rc;
      if (end_block == b + 1) return TFX_OK;
      for (int i = 0; i < 3; ++i) shape[i] = g.out[i];
      shape[3] = cout;
      cur ^= 1;
      continue;
    }
    rc = tfx_depthwise_conv2d_f16(buf[cur], shape, weights->dw_w[b], fd, weights->dw_b[b], kStrides[b], kStrides[b],
                                  TFX_PAD_SAME, TFX_ACT_RELU6, buf[cur ^ 1], stream);
    if (rc) return rc;
    for (int i = 0; i < 4; ++i) shape[i] = g.out[i];
    cur ^= 1;
    const int64_t fp[4] = {1, 1, shape[3], cout};
    rc = tfx_conv2d_f16(buf[cur], shape, weights->pw_w[b], fp, weights->pw_b[b], 1, 1, TFX_PAD_SAME, TFX_ACT_RELU6,
                        end_block == b + 1 ? features : buf[cur ^ 1], stream);
    if (rc) return rc;
    if (end_block == b + 1) return TFX_OK;
    shape[3] = cout;
    cur ^= 1;
  }
  if (chain)
    return launch_chain_f16(buf[cur], (int)variant->image_size, weights, ws + plan.off_chain, probs, logits, (int)variant->classes, q, chain_first, s);
  return launch_pool_fc_softmax_f16(buf[cur], weights->fc_w, weights->fc_b, partial, logits, probs, (int)batch,
                                    (int)(shape[1] * shape[2]), (int)shape[3], (int)variant->classes, s);
}

}  // namespace

extern "C" {

int tfx_mobilenet_v1_forward_f16(const tfx_mobilenet_v1_variant* variant, const uint16_t* input, int64_t batch,
                                 const tfx_mobilenet_v1_weights_f16* weights, void* workspace,
                                 size_t workspace_bytes, uint16_t* probs, uint16_t* logits, void* stream) {
  return forward_f16_impl(variant, input, batch, weights, workspace, workspace_bytes, probs, logits, 0, nullptr, stream);
}

int tfx_mobilenet_v1_features_f16(const tfx_mobilenet_v1_variant* variant, const uint16_t* input, int64_t batch,
                                  const tfx_mobilenet_v1_weights_f16* weights, void* workspace, size_t workspace_bytes,
                                  int end_block, uint16_t* features, void* stream) {
  if (end_block < 1 || end_block > kBlocks) return TFX_ERR_ARG;
  if (features && reinterpret_cast<uintptr_t>(features) % 16 != 0) return TFX_ERR_ARG;
  return forward_f16_impl(variant, input, batch, weights, workspace, workspace_bytes, nullptr, nullptr, end_block, features,
                          stream);
}

}  // extern "C"
