// Host-side interface to the HIP kernels.
#pragma once
#include <hip/hip_runtime_api.h>

#include <string>

#include "conv_args.h"

namespace lic {

// Template configuration of one implicit-GEMM kernel instantiation:
// input channels per tap (K chunking), m-tiles (16 output channels each) and
// n-tiles (16 pixels each) per wave, waves per block, loader and epilogue.
struct KernelKey {
    int tag, cin, mt, nt, waves, ksplit, ld, ep, dt;   // tag = layer id (one kernel symbol per layer)
    bool operator==(const KernelKey& o) const
    {
        return tag == o.tag && cin == o.cin && mt == o.mt && nt == o.nt && waves == o.waves &&
               ksplit == o.ksplit && ld == o.ld && ep == o.ep && dt == o.dt;
    }
};

bool kernel_available(const KernelKey& k);
// GDN layers of whole frames with both operands staged in LDS (gdn_kernels.hip)
bool gdn_available(const KernelKey& k);
hipError_t launch_gdn(const KernelKey& k, const ConvArgs& args, int nblocks, hipStream_t stream);
// layers of small grids, split K over the waves of a block (split_kernels.hip):
// rg groups of mt 16-row blocks x nt 16-pixel tiles, ks K slots
struct SplitKey {
    int mt, nt, rg, ks, ld, ep, dt;
    bool operator==(const SplitKey& o) const
    {
        return mt == o.mt && nt == o.nt && rg == o.rg && ks == o.ks && ld == o.ld && ep == o.ep && dt == o.dt;
    }
};
bool split_available(const SplitKey& k);
hipError_t launch_split(const SplitKey& k, const ConvArgs& args, int nblocks, hipStream_t stream);
// GDN / IGDN of FP32 activations [pixel][cop] in place (128 or 192 channels)
hipError_t launch_gdn_apply(int cop, int ep, const ConvArgs& args, hipStream_t stream);
// g_s's output layer (rgb_kernels.hip): 3 x 3 neighbourhood, grid a multiple of 8 x 32
bool rgb_available(int cin, int dt);
hipError_t launch_rgb(int cin, int dt, const ConvArgs& args, hipStream_t stream);
// g_a's first layer (image_kernels.hip): 5 x 5, stride 2, 128 channels, grid rows
// of whole 32-pixel tiles
bool image_available(int cop, int dt);
hipError_t launch_image(int dt, const ConvArgs& args, hipStream_t stream);
// IGDN layers with the pixels of a tile and its halo in LDS (window_kernels.hip):
// every tap within one pixel; a.tw set
constexpr int kWindowPixels = 256;
bool window_available(int tag, int cin, int cop, int dt);
hipError_t launch_window(int tag, int cin, int cop, int dt, const ConvArgs& args, hipStream_t stream);
hipError_t launch_conv(const KernelKey& k, const ConvArgs& args, int nblocks, hipStream_t stream);

// Context model, element-wise steps of the two checkerboard passes (layout
// in conv_args.h): value into channels [off, off + C) of a [n][Hy][Wy][ld]
// float tensor at the positions of set `part`; y_hat = sym + mean of set
// `part` (checkerboard-major inputs) onto the full [n][Hy][Wy][C] grid as
// float32 (out32) and / or bf16 (out16), either may be null.
hipError_t launch_cb_fill(float* buf, int n, int Hy, int Wy, int ld, int off, int C, int part, float value,
                          hipStream_t s);
// bf16 (round to nearest even) copy of n floats.
hipError_t launch_f32_to_bf16(const float* in, void* out, long n, hipStream_t s);
hipError_t launch_cb_dequant(const int8_t* sym, const float* mean, float* out32, void* out16, int n, int Hy, int Wy,
                             int C, int part, hipStream_t s);

// Kernel tags beyond the codec's layer ids: the distilled synthesis network
// (forward layers, and the input gradients of its second and third layer).
enum { TAG_DT1 = 32, TAG_DT2 = 33, TAG_DT3 = 34, TAG_DB2 = 35, TAG_DB3 = 36 };

// What the tile policy needs to know of a packed layer.
struct ConvShape {
    int tag, ld, ep, dt, cin, cop, nphase;
    int halo1 = 0;     // stride-1 grid, every tap within one pixel (halo-tile loader allowed)
};

// The kernel of a layer over an a.n x a.Hg x a.Wg grid.
struct ConvRoute {
    enum Kernel { DIRECT, STAGED, WINDOW, SPLIT, TWO_PASS, IMAGE, RGB } kernel;
    KernelKey key;         // operand form and K slots; of the direct and staged kernels all of it
    SplitKey split;        // SPLIT, TWO_PASS: the tile (TWO_PASS: of the sums)
    int ncog, tw;          // blocks along the output channels; WINDOW: columns of a tile
    long nblocks;          // (IMAGE, RGB, WINDOW: their launches count their own)
};
// Host arithmetic only, on the grids and strides in a (its pointers are not
// looked at).  What fixes the order of the sums, the operand form and the K
// slots, comes from policy_pixels, the pixel grid of one image, so that results
// do not depend on the batch.  Returns a lic_status; *errp names the failure.
int choose_route(const ConvShape& L, const ConvArgs& a, long policy_pixels, ConvRoute* r, std::string* errp);
// The operand layouts that the kernels of a layer read at any size (ConvArgs).
struct Operands {
    bool w, wx, wt, ws, gsplit, gt;
};
Operands layer_operands(const ConvShape& L);
// Chooses and launches (sets a.ncog, a.tw).  With chosen non-null nothing is
// launched: the route's key is stored there.
int launch_conv_policy(const ConvShape& L, ConvArgs& a, long policy_pixels, hipStream_t s, std::string* errp,
                       KernelKey* chosen = nullptr);

}  // namespace lic
