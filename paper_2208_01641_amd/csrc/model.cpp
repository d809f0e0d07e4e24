// Model loading: weight blob parsing, entropy tables, weight packing for the
// implicit-GEMM kernels, per-layer geometry and launch planning.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <system_error>
#include <thread>

#include "codec.h"
#include "packing.h"

namespace lic {

#define HIP_TRY(expr)                                                              \
    do {                                                                           \
        hipError_t e_ = (expr);                                                    \
        if (e_ != hipSuccess) {                                                    \
            err = std::string(#expr) + ": " + hipGetErrorString(e_);               \
            return LIC_E_HIP;                                                      \
        }                                                                          \
    } while (0)

void* Codec::dev_alloc(size_t bytes)
{
    void* p = nullptr;
    if (hipMalloc(&p, bytes ? bytes : 16) != hipSuccess) return nullptr;
    dev_allocs.push_back(p);
    dev_bytes += bytes;
    alloc_events++;
    return p;
}

void* Codec::host_alloc(size_t bytes)
{
    void* p = nullptr;
    if (hipHostMalloc(&p, bytes ? bytes : 16, hipHostMallocMapped) != hipSuccess) return nullptr;
    host_allocs.push_back(p);
    alloc_events++;
    return p;
}

namespace {

using ParamMap = std::map<std::string, std::pair<std::vector<int>, std::vector<double>>>;

bool parse_blob(const uint8_t* b, size_t len, int* kind, int* N, int* M, ParamMap* P, std::string* err)
{
    auto rd32 = [&](size_t pos) {
        uint32_t v;
        memcpy(&v, b + pos, 4);
        return v;
    };
    if (len < 24 || memcmp(b, "LICW", 4) != 0) { *err = "weight blob: bad magic"; return false; }
    if (rd32(4) != 1) { *err = "weight blob: unsupported version"; return false; }
    *kind = (int)rd32(8);
    *N = (int)rd32(12);
    *M = (int)rd32(16);
    const uint32_t count = rd32(20);
    size_t pos = 24;
    for (uint32_t e = 0; e < count; ++e) {
        if (pos + 2 > len) { *err = "weight blob: truncated"; return false; }
        uint16_t nl;
        memcpy(&nl, b + pos, 2);
        pos += 2;
        if (pos + nl + 2 > len) { *err = "weight blob: truncated"; return false; }
        std::string name((const char*)b + pos, nl);
        pos += nl;
        const int code = b[pos], ndim = b[pos + 1];
        pos += 2;
        if ((code != 0 && code != 1) || ndim > 4 || pos + 4u * ndim > len) { *err = "weight blob: bad entry"; return false; }
        std::vector<int> dims(ndim);
        size_t count_el = 1;
        for (int d = 0; d < ndim; ++d) {
            dims[d] = (int)rd32(pos);
            pos += 4;
            count_el *= (size_t)dims[d];
        }
        const size_t esz = code == 0 ? 4 : 8;
        if (pos + count_el * esz > len) { *err = "weight blob: truncated data"; return false; }
        std::vector<double> vals(count_el);
        for (size_t i = 0; i < count_el; ++i) {
            if (code == 0) {
                float f;
                memcpy(&f, b + pos + 4 * i, 4);
                vals[i] = f;
            } else {
                memcpy(&vals[i], b + pos + 8 * i, 8);
            }
        }
        pos += count_el * esz;
        (*P)[name] = {dims, std::move(vals)};
    }
    return true;
}

}  // namespace

// float32 -> bfloat16, round to nearest even (NaN stays NaN)
uint16_t bf16_rne(float f)
{
    uint32_t u;
    memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Eight floats as three bf16 parts, each rounded to nearest from what the
// previous ones leave: part g at out + g pitch.
static void split_parts8(const float* v, uint16_t* out, size_t pitch)
{
    for (int e = 0; e < 8; ++e) {
        float rem = v[e];
        for (int g = 0; g < 3; ++g) {
            const uint16_t h = bf16_rne(rem);
            out[g * pitch + e] = h;
            const uint32_t u = (uint32_t)h << 16;
            float hv;
            memcpy(&hv, &u, 4);
            rem -= hv;
        }
    }
}

// GDN gamma [co][co] (row-major, FP64 from the weight blob, used as FP32)
// as three bf16 parts g0 + g1 + g2, each rounded to nearest from what the
// previous parts leave (remainders are exact in FP32), laid out for the
// GDN epilogue: part k of gamma[r][(2p + i/4) 16 + 4 kg + i%4] at
// (((k co + r) (co/32) + p) 4 + kg) 8 + i.
std::vector<uint16_t> gdn_gamma_split(const std::vector<double>& gamma, int co)
{
    const int npair = co / 32;
    std::vector<uint16_t> out((size_t)3 * co * co);
    for (int r = 0; r < co; ++r)
        for (int p = 0; p < npair; ++p)
            for (int kg = 0; kg < 4; ++kg)
                for (int i = 0; i < 8; ++i) {
                    const int c = (2 * p + i / 4) * 16 + 4 * kg + i % 4;
                    float rem = (float)gamma[(size_t)r * co + c];
                    for (int k = 0; k < 3; ++k) {
                        const uint16_t h = bf16_rne(rem);
                        out[((((size_t)k * co + r) * npair + p) * 4 + kg) * 8 + i] = h;
                        const uint32_t u = (uint32_t)h << 16;
                        float hv;
                        memcpy(&hv, &u, 4);
                        rem -= hv;
                    }
                }
    return out;
}

// The first `parts` parts of gdn_gamma_split in fragment order
// [p][16-row block][part][lane][8] (ConvArgs::gt).
std::vector<uint16_t> gdn_gamma_tiles(const std::vector<uint16_t>& gsplit, int co, int parts)
{
    const int npair = co / 32;
    std::vector<uint16_t> out;
    out.reserve((size_t)parts * co * co);
    for (int p = 0; p < npair; ++p)
        for (int mt = 0; mt < co / 16; ++mt)
            for (int g = 0; g < parts; ++g)
                for (int l = 0; l < 64; ++l) {
                    const size_t j = ((((size_t)g * co + mt * 16 + l % 16) * npair + p) * 4 + l / 16) * 8;
                    out.insert(out.end(), gsplit.begin() + j, gsplit.begin() + j + 8);
                }
    return out;
}

// OCP e4m3 (1 sign, 4 exponent bits with bias 7, 3 mantissa bits; largest
// finite 448, subnormal step 2^-9, no infinities) of f, rounding to nearest
// even and saturating at +-448.
uint8_t e4m3_rne(float f)
{
    const uint8_t sign = std::signbit(f) ? 0x80 : 0x00;
    double a = std::fabs((double)f);
    if (!(a == a)) return 0x7f;                     // NaN
    if (a >= 448.0) return sign | 0x7e;
    // quantum of the binade (2^-9 below the smallest normal 2^-6)
    int ex = 0;
    (void)std::frexp(a, &ex);                       // a = m 2^ex, m in [0.5, 1)
    int e = a > 0.0 ? ex - 1 : -6;
    if (e < -6) e = -6;
    const double q = std::ldexp(1.0, e - 3);
    double m = a / q;                               // exact: q is a power of two
    double r = std::nearbyint(m);                   // ties to even (default rounding mode)
    double v = r * q;
    if (v >= 448.0) return sign | 0x7e;
    if (v == 0.0) return sign;
    (void)std::frexp(v, &ex);
    const int ve = ex - 1;
    if (ve < -6) return sign | (uint8_t)std::lround(v / std::ldexp(1.0, -9));     // subnormal
    const int mant = (int)std::lround(v / std::ldexp(1.0, ve - 3)) - 8;
    return sign | (uint8_t)((ve + 7) << 3) | (uint8_t)mant;
}

bool build_tables(const ParamMap& P, int kind, int N, int M, std::vector<float>* medians,
                  std::vector<uint32_t>* fact_freq, std::vector<uint32_t>* gauss_freq, std::string* err)
{
    auto it = P.find("eb.density");
    const int C = kind == 0 ? M : N;
    if (it == P.end() || it->second.second.size() != (size_t)C * kDensityParams) {
        *err = "weight blob: eb.density missing or of the wrong size";
        return false;
    }
    const std::vector<double>& dens = it->second.second;
    medians->resize(C);
    fact_freq->assign((size_t)C * kNumSym, 0);
    std::vector<double> pmf(kNumSym);
    for (int c = 0; c < C; ++c) {
        const double* prm = dens.data() + (size_t)c * kDensityParams;
        (*medians)[c] = (float)density_median(prm);
        pmf_factorized(prm, (double)(*medians)[c], pmf.data());
        quantize_pmf(pmf.data(), fact_freq->data() + (size_t)c * kNumSym);
    }
    gauss_freq->clear();
    if (kind >= 1) {
        double t[kScales];
        scale_table(t);
        gauss_freq->assign((size_t)kScales * kNumSym, 0);
        for (int k = 0; k < kScales; ++k) {
            pmf_gaussian(t[k], pmf.data());
            quantize_pmf(pmf.data(), gauss_freq->data() + (size_t)k * kNumSym);
        }
    }
    return true;
}

namespace {

// Every layer takes what the layer before it gives, the ends of the chains are
// the image, y (M channels), z (N) and, in the context model, psi and the
// context (2M each), and no hidden layer is wider than N, for which the pools
// are sized.  (Layers that are missing are reported where they are packed.)
bool check_widths(const ParamMap& P, int kind, int N, int M, std::string* err)
{
    struct Link {
        const char* name;
        bool deconv;
        int from;          // input width; 0: the output of the layer before
        int to;            // output width; 0: a hidden layer
        bool pooled;       // a hidden layer's output goes to a buffer of width N
    };
    std::vector<Link> links = {
        {"ga0", false, 3, 0, true}, {"ga1", false, 0, 0, true}, {"ga2", false, 0, 0, true}, {"ga3", false, 0, M, true},
        {"gs0", true, M, 0, true},  {"gs1", true, 0, 0, true},  {"gs2", true, 0, 0, true},  {"gs3", true, 0, 3, true},
    };
    if (kind >= 1) {
        const std::vector<Link> hyper = {
            {"ha0", false, M, 0, true}, {"ha1", false, 0, 0, true}, {"ha2", false, 0, N, true},
            {"hs0", true, N, 0, true},  {"hs1", true, 0, 0, true},  {"hs2", false, 0, kind == 2 ? 2 * M : M, true},
        };
        links.insert(links.end(), hyper.begin(), hyper.end());
    }
    if (kind == 2) {
        const std::vector<Link> ctx = {
            {"cx", false, M, 2 * M, false}, {"ep0", false, 4 * M, 0, false}, {"ep1", false, 0, 0, false},
            {"ep2", false, 0, 2 * M, false},
        };
        links.insert(links.end(), ctx.begin(), ctx.end());
    }
    int last = 0;
    for (const Link& k : links) {
        auto it = P.find(std::string(k.name) + ".w");
        if (it == P.end() || it->second.first.size() != 4) return true;
        const std::vector<int>& dims = it->second.first;
        const int ci = dims[k.deconv ? 0 : 1], co = dims[k.deconv ? 1 : 0];
        const int want = k.from ? k.from : last;
        if (ci != want) {
            *err = std::string("weight blob: ") + k.name + " takes " + std::to_string(ci) + " channels, not " + std::to_string(want);
            return false;
        }
        if (k.to ? co != k.to : co < 1 || (k.pooled && co > N)) {
            *err = std::string("weight blob: ") + k.name + " gives " + std::to_string(co) + " channels, not " +
                   (k.to ? std::to_string(k.to) : "1 to " + std::to_string(N));
            return false;
        }
        last = co;
    }
    return true;
}

}  // namespace

int Codec::load(const void* blob, size_t len)
{
    ParamMap P;
    int bk, bn, bm;
    if (!parse_blob(static_cast<const uint8_t*>(blob), len, &bk, &bn, &bm, &P, &err)) return LIC_E_ARG;
    if (bk != cfg.kind || bn != cfg.N || bm != cfg.M) {
        err = "weight blob kind/N/M does not match the configuration";
        return LIC_E_MODEL;
    }
    kind = cfg.kind;
    N = cfg.N;
    M = cfg.M;
    if (!check_widths(P, kind, N, M, &err)) return LIC_E_MODEL;
    hs_exp = cfg.hs_out == LIC_HS_EXP ? 1 : 0;
    norm = cfg.norm;
    lanes = cfg.rans_lanes;
    S = cfg.y_slices;
    // The model id, a serial hash of every byte (two fifths of a create's time),
    // beside the rest; joined on every way out.
    struct Hash {
        std::thread t;
        ~Hash()
        {
            if (t.joinable()) t.join();
        }
    } hash;
    auto take_id = [this, blob, len] { model_id = fnv1a(blob, len); };
    try {
        hash.t = std::thread(take_id);
    } catch (const std::system_error&) {
        take_id();
    }

    // entropy model: per-channel medians, factorized and Gaussian tables
    std::vector<uint32_t> ff, gf;
    if (!build_tables(P, kind, N, M, &medians, &ff, &gf, &err)) return LIC_E_MODEL;
    fact.init(kind == 0 ? M : N, ff.data(), kind == 0);
    if (kind >= 1) {
        gauss.init(kScales, gf.data(), true);
        double t[kScales];
        scale_table(t);
        thr.resize(63);
        for (int k = 0; k < 63; ++k) thr[k] = hs_exp ? (float)log(t[k]) : (float)t[k];
    }
    return build_layers(P);
}

long blob_tables(const void* blob, size_t len, int which, uint32_t* freq, size_t cap, float* mu, size_t mu_cap)
{
    ParamMap P;
    int kind, N, M;
    std::string e;
    if (!parse_blob(static_cast<const uint8_t*>(blob), len, &kind, &N, &M, &P, &e)) return LIC_E_ARG;
    std::vector<float> med;
    std::vector<uint32_t> ff, gf;
    if (!build_tables(P, kind, N, M, &med, &ff, &gf, &e)) return LIC_E_MODEL;
    const std::vector<uint32_t>& src = which == 0 ? ff : gf;
    if (which != 0 && which != 1) return LIC_E_ARG;
    if (src.size() > cap || (mu && med.size() > mu_cap)) return LIC_E_SMALLBUF;
    std::copy(src.begin(), src.end(), freq);
    if (mu) std::copy(med.begin(), med.end(), mu);
    return (long)src.size();
}

std::vector<LayerSpec> layer_specs(int kind)
{
    std::vector<LayerSpec> specs = {
        {LIC_GA0, "ga0", LD_RGB, EP_GDN, false, 5}, {LIC_GA1, "ga1", LD_F32, EP_GDN, false, 5},
        {LIC_GA2, "ga2", LD_F32, EP_GDN, false, 5}, {LIC_GA3, "ga3", LD_F32, EP_QUANT, false, 5},
        {LIC_GS0, "gs0", LD_I8, EP_IGDN, true, 5},  {LIC_GS1, "gs1", LD_F32, EP_IGDN, true, 5},
        {LIC_GS2, "gs2", LD_F32, EP_IGDN, true, 5}, {LIC_GS3, "gs3", LD_F32, EP_RGB, true, 5},
    };
    if (kind >= 1) {
        // the context model's h_a sees y (the means need its signs), its h_s
        // ends in psi (2M channels, no activation) and g_s starts from the
        // float y_hat = sym + mean
        std::vector<LayerSpec> hyper = {
            {LIC_HA0, "ha0", kind == 1 ? LD_F32_ABS : LD_F32, EP_RELU, false, 3},
            {LIC_HA1, "ha1", LD_F32, EP_RELU, false, 5},
            {LIC_HA2, "ha2", LD_F32, EP_QUANT, false, 5},    {LIC_HS0, "hs0", LD_I8, EP_RELU, true, 5},
            {LIC_HS1, "hs1", LD_F32, EP_RELU, true, 5},
            {LIC_HS2, "hs2", LD_F32, kind == 1 ? EP_INDEX : EP_NONE, false, 3},
        };
        specs.insert(specs.end(), hyper.begin(), hyper.end());
    }
    if (kind == 2) {
        specs[4].ld = LD_F32;                            // gs0
        std::vector<LayerSpec> ctx = {
            {LIC_CX, "cx", LD_F32, EP_NONE, false, 5, 1},
            {LIC_EP0A, "ep0", LD_F32, EP_RELU, false, 1, 0},   {LIC_EP1A, "ep1", LD_F32, EP_RELU, false, 1, 0},
            {LIC_EP2A, "ep2", LD_F32, EP_MSCALE, false, 1, 0}, {LIC_EP0N, "ep0", LD_F32, EP_RELU, false, 1, 1},
            {LIC_EP1N, "ep1", LD_F32, EP_RELU, false, 1, 1},   {LIC_EP2N, "ep2", LD_F32, EP_MSCALE, false, 1, 1},
        };
        specs.insert(specs.end(), ctx.begin(), ctx.end());
    }
    return specs;
}

LayerForm layer_form(const LayerSpec& sp, int precision)
{
    LayerForm f{DT_F32, false, false};
    // bf16 operands for the analysis / synthesis transforms in the BF16
    // form; h_a and h_s always run in FP32 (fixed-order scale index)
    const bool is_gags = sp.id <= LIC_GA3 || (sp.id >= LIC_GS0 && sp.id <= LIC_GS3);
    if (is_gags) f.dt = precision == LIC_PREC_BF16 ? DT_BF16 : precision == LIC_PREC_FP8 ? DT_FP8 : DT_F32;
    // the e4m3 form's image layer: bf16 operands (a K of 75 is one
    // chunk; pixel values keep 8 bits), e4m3 activations out; so does
    // g_s's first layer (its symbol loader's conversion to e4m3 does not
    // fit two waves per SIMD, the bf16 kernel does; the context model's
    // y_hat = sym + mean arrives as bf16 anyway)
    f.out_e4m3 = f.dt == DT_FP8 && (sp.ld == LD_RGB || sp.id == LIC_GS0);
    if (f.out_e4m3) f.dt = DT_BF16;
    // and its output layer too (bf16 halo tiles: the 3 output channels
    // make a K chunk of 128 (tap, channel) pairs a poor fit), fed by a
    // last GDN layer that stores bf16
    if (f.dt == DT_FP8 && sp.id == LIC_GS3) f.dt = DT_BF16;
    f.out_bf16 = f.dt == DT_FP8 && sp.id == LIC_GS2;
    return f;
}

ConvShape layer_shape(const LayerSpec& sp, const LayerForm& f, int ci, int co)
{
    const bool rows = sp.ep == EP_RGB;                   // all phases as GEMM rows
    ConvShape L{};
    L.tag = sp.id;
    L.ld = sp.ld;
    L.ep = sp.ep;
    L.dt = f.dt;
    L.cin = sp.ld == LD_RGB ? 96 : ci;                   // the image: 75 (tap, channel) pairs in whole K chunks
    L.cop = rows ? 16 : co;
    L.nphase = sp.cb >= 0 ? 2 : sp.deconv && !rows ? 4 : 1;
    // taps within one pixel of a stride-1 grid: a stride-2 transposed 5 x 5, 3 x 3, 1 x 1
    L.halo1 = sp.ld != LD_RGB && (sp.deconv || sp.k <= 3) ? 1 : 0;
    return L;
}

int Codec::upload_rscale(LayerGPU& L)
{
    std::vector<float> rs(L.wsc.size());
    for (size_t r = 0; r < rs.size(); ++r) rs[r] = L.wsc[r] * L.in_scale;
    HIP_TRY(hipMemcpy(L.d_rscale, rs.data(), rs.size() * sizeof(float), hipMemcpyHostToDevice));
    return LIC_OK;
}

// Activation scales of the e4m3 form: each layer that stores e4m3
// activations gets q = 448 / (2 amax), amax the largest |value| it produces
// on the calibration frames (one binary order of headroom), with the scales
// of the layers before it already in place; the layer that reads its output
// undoes q in its epilogue.  The layers run once with bf16 outputs to
// measure amax and once more in e4m3 to feed the next layer.
int Codec::calibrate_fp8(const float* x, int n, int H, int W)
{
    if (cfg.precision != LIC_PREC_FP8) return LIC_OK;
    const FrameDims d(H, W);
    size_t cap = 0;
    for (int id : {LIC_GA0, LIC_GA1, LIC_GA2, LIC_GA3, LIC_GS0, LIC_GS1, LIC_GS2}) {
        size_t bi, bo, ba;
        layer_bytes(id, n, d, &bi, &bo, &ba);
        cap = std::max(cap, std::max(bi, std::max(bo, ba)) * 4);     // room for any storage type
    }
    // buf[0]: measured (bf16) outputs; buf[1], buf[2]: e4m3 activations; buf[3]: symbols of y
    void* buf[4] = {nullptr, nullptr, nullptr, nullptr};
    for (void*& b : buf)
        if (hipMalloc(&b, cap) != hipSuccess) {
            for (void* q : buf) (void)hipFree(q);
            err = "calibration buffers: device allocation failed";
            return LIC_E_NOMEM;
        }
    std::vector<uint16_t> host(cap / 2);
    std::string e;
    int rc = LIC_OK;
    // amax of layer id's output (bf16 storage) on input `in`
    auto measure = [&](int id, const void* in, float* amax) -> int {
        LayerGPU& L = layers[id];
        const bool e8 = L.out_e4m3, b16 = L.out_bf16;
        if (L.dt == DT_BF16) L.out_e4m3 = false; else L.out_bf16 = true;
        size_t bi, bo, ba;
        layer_bytes(id, n, d, &bi, &bo, &ba);
        int r = launch_layer(id, n, d, in, buf[0], nullptr, layer_stream, &e);
        L.out_e4m3 = e8;
        L.out_bf16 = b16;
        if (r != LIC_OK) { err = e; return r; }
        if (hipMemcpyAsync(host.data(), buf[0], bo, hipMemcpyDeviceToHost, layer_stream) != hipSuccess ||
            hipStreamSynchronize(layer_stream) != hipSuccess) { err = "calibration copy failed"; return LIC_E_HIP; }
        float m = 0.0f;
        for (size_t i = 0; i < bo / 2; ++i) {
            const uint32_t u = (uint32_t)host[i] << 16;
            float v;
            memcpy(&v, &u, 4);
            m = std::max(m, std::fabs(v));
        }
        *amax = m;
        return LIC_OK;
    };
    // sets layer id's scale from its output on `in`, runs it in e4m3 into out
    auto step = [&](int id, const void* in, void* out, void* aux) -> int {
        float amax = 0.0f;
        int r = measure(id, in, &amax);
        if (r != LIC_OK) return r;
        LayerGPU& L = layers[id];
        if (L.dt == DT_FP8 ? !L.out_bf16 : L.out_e4m3) {
            L.out_q = amax > 0.0f && std::isfinite(amax) ? 448.0f / (2.0f * amax) : kActQ;
            LayerGPU& next = layers[id + 1];
            next.in_scale = 1.0f / L.out_q;
            if ((r = upload_rscale(next)) != LIC_OK) return r;
        }
        if ((r = launch_layer(id, n, d, in, out, aux, layer_stream, &e)) != LIC_OK) { err = e; return r; }
        return LIC_OK;
    };
    if ((rc = step(LIC_GA0, x, buf[1], nullptr)) == LIC_OK && (rc = step(LIC_GA1, buf[1], buf[2], nullptr)) == LIC_OK &&
        (rc = step(LIC_GA2, buf[2], buf[1], nullptr)) == LIC_OK &&
        (rc = launch_layer(LIC_GA3, n, d, buf[1], buf[2], buf[3], layer_stream, &e)) == LIC_OK) {
        // the context model's g_s starts from y_hat = sym + mean in bf16; y
        // itself (within half a step of it) stands in for the calibration
        if (kind == 2) {
            const hipError_t he = launch_f32_to_bf16(static_cast<const float*>(buf[2]), buf[3],
                                                     (long)n * d.Hy * d.Wy * M, layer_stream);
            if (he != hipSuccess) { err = "calibration: conversion failed"; rc = LIC_E_HIP; }
        }
        if (rc == LIC_OK && (rc = step(LIC_GS0, buf[3], buf[1], nullptr)) == LIC_OK)
            rc = step(LIC_GS1, buf[1], buf[2], nullptr);
    }
    if (rc != LIC_OK && err.empty()) err = e;
    if (hipStreamSynchronize(layer_stream) != hipSuccess && rc == LIC_OK) { err = "calibration failed"; rc = LIC_E_HIP; }
    for (void* b : buf) (void)hipFree(b);
    // captured serving graphs hold the old scales in their kernel arguments
    server_drop_graphs(ST_GPU_ENC);
    server_drop_graphs(ST_GPU_GS);
    return rc;
}

int Codec::build_layers(const ParamMap& P)
{
    HIP_TRY(hipSetDevice(cfg.hip_device));
    if (cfg.precision == LIC_PREC_FP8) {
        d_sat = (unsigned long long*)dev_alloc(sizeof(unsigned long long));
        if (!d_sat) { err = "device allocation failed"; return LIC_E_NOMEM; }
        HIP_TRY(hipMemset(d_sat, 0, sizeof(unsigned long long)));
    }
    const int C = kind == 0 ? M : N;
    d_medians = (float*)dev_alloc(sizeof(float) * 512);
    d_zero = (float*)dev_alloc(sizeof(float) * 512);
    d_thr = (float*)dev_alloc(sizeof(float) * 64);
    if (!d_medians || !d_zero || !d_thr) { err = "device allocation failed"; return LIC_E_NOMEM; }
    std::vector<float> tmp(512, 0.0f);
    HIP_TRY(hipMemcpy(d_zero, tmp.data(), 512 * sizeof(float), hipMemcpyHostToDevice));
    std::copy(medians.begin(), medians.end(), tmp.begin());
    HIP_TRY(hipMemcpy(d_medians, tmp.data(), 512 * sizeof(float), hipMemcpyHostToDevice));
    if (!thr.empty()) HIP_TRY(hipMemcpy(d_thr, thr.data(), 63 * sizeof(float), hipMemcpyHostToDevice));
    (void)C;

    // (kept from layer to layer: fresh pages cost more than the packing)
    std::vector<float> wp;
    std::vector<uint16_t> hb, hx;                        // bf16 / split-FP32 / e4m3 operands
    std::vector<uint8_t> h8, wt;
    for (const LayerSpec& sp : layer_specs(kind)) {
        LayerGPU& L = layers[sp.id];
        auto wit = P.find(std::string(sp.name) + ".w");
        auto bit = P.find(std::string(sp.name) + ".b");
        if (wit == P.end() || bit == P.end() || wit->second.first.size() != 4) {
            err = std::string("weight blob: missing ") + sp.name;
            return LIC_E_MODEL;
        }
        const std::vector<int>& dims = wit->second.first;
        const std::vector<double>& w = wit->second.second;
        const std::vector<double>& b = bit->second.second;
        const int k = dims[2];
        if (k != sp.k || dims[3] != k) { err = std::string("weight blob: bad kernel size in ") + sp.name; return LIC_E_MODEL; }
        const int ci = sp.deconv ? dims[0] : dims[1];
        const int co = sp.deconv ? dims[1] : dims[0];
        if ((int)b.size() != co) { err = std::string("weight blob: bad bias in ") + sp.name; return LIC_E_MODEL; }
        L.present = true;
        L.ld = sp.ld;
        L.ep = sp.ep;
        L.k = k;
        L.deconv = sp.deconv;
        L.co = co;
        L.rows = sp.ep == EP_RGB;
        const LayerForm form = layer_form(sp, cfg.precision);
        const ConvShape shape = layer_shape(sp, form, ci, co);
        L.dt = form.dt;
        L.out_e4m3 = form.out_e4m3;
        L.out_bf16 = form.out_bf16;
        L.cin = shape.cin;
        L.cop = shape.cop;
        L.nphase = shape.nphase;
        L.halo1 = shape.halo1 != 0;
        if (sp.ld == LD_RGB && ci != 3) { err = "ga0 must take 3 channels"; return LIC_E_MODEL; }
        if (!L.rows && co % 16 != 0) { err = std::string("channels must be multiples of 16: ") + sp.name; return LIC_E_MODEL; }
        if (L.rows && co != 3) { err = "gs3 must produce 3 channels"; return LIC_E_MODEL; }
        // packed GEMM operands as index maps into the PyTorch-layout weights
        PackMap pm;
        if (sp.cb >= 0) pm = pack_map_checkerboard(ci, co, k, sp.cb, sp.ep == EP_MSCALE);
        else if (sp.ld == LD_RGB) pm = pack_map(PK_IMG, 3, co, k, 2, k / 2, false, L.cin);
        else if (!sp.deconv) pm = pack_map(PK_CONV, ci, co, k, 1, k / 2, false);
        else if (!L.rows) pm = pack_map(PK_DECONV, ci, co, k, 2, k / 2, true);
        else pm = pack_map(PK_ROWS, ci, co, k, 2, k / 2, true);
        std::vector<PhaseDesc> ph = pm.ph;
        bool halo1 = sp.ld != LD_RGB;
        for (const PhaseDesc& d : ph)
            for (int t = 0; t < d.ntaps; ++t)
                if (d.dy[t] < -1 || d.dy[t] > 1 || d.dx[t] < -1 || d.dx[t] > 1) halo1 = false;
        if (pm.cin != L.cin || pm.cop != L.cop || (int)ph.size() != L.nphase || halo1 != L.halo1) {
            err = std::string("packing mismatch in ") + sp.name;
            return LIC_E_MODEL;
        }

        const Operands use = layer_operands(shape);
        const size_t total = pm.idx.size();
        auto upload = [&](const void* src, size_t bytes) -> uint8_t* {
            void* dst = dev_alloc(bytes);
            if (dst && hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice) != hipSuccess) dst = nullptr;
            return static_cast<uint8_t*>(dst);
        };
        wp.resize(total);
        for (size_t j = 0; j < total; ++j) wp[j] = pm.idx[j] < 0 ? 0.0f : (float)w[pm.idx[j]];
        if (L.dt == DT_BF16) {
            hb.resize(total);
            for (size_t j = 0; j < total; ++j) hb[j] = bf16_rne(wp[j]);
        } else if (L.dt == DT_FP8) {
            // per packed row: scale = max |w| / 448 over every tap and phase
            // of the row, w8 = e4m3(w / scale); the epilogue multiplies by
            // scale and by the input's own scale (1 / kActQ for e4m3
            // activations, 1 for the image and for y_hat)
            const size_t cin = (size_t)L.cin;
            std::vector<double> amax(L.cop, 0.0);
            for (size_t i = 0; i < ph.size(); ++i) {
                const size_t end = i + 1 < ph.size() ? pm.off[i + 1] : total;
                for (size_t j = pm.off[i]; j < end; ++j) {
                    const size_t row = ((j - pm.off[i]) / cin) % (size_t)L.cop;
                    amax[row] = std::max(amax[row], (double)std::fabs(wp[j]));
                }
            }
            std::vector<float> wsc(L.cop);
            for (int r = 0; r < L.cop; ++r) wsc[r] = amax[r] > 0.0 ? (float)(amax[r] / 448.0) : 1.0f;
            h8.resize(total);
            for (size_t i = 0; i < ph.size(); ++i) {
                const size_t end = i + 1 < ph.size() ? pm.off[i + 1] : total;
                for (size_t j = pm.off[i]; j < end; ++j) h8[j] = e4m3_rne(wp[j] / wsc[((j - pm.off[i]) / cin) % (size_t)L.cop]);
            }
            L.in_scale = (sp.ld == LD_F32) ? 1.0f / kActQ : 1.0f;
            L.wsc = wsc;
            L.d_rscale = (float*)dev_alloc(L.cop * sizeof(float));
            if (!L.d_rscale) { err = "device allocation failed"; return LIC_E_NOMEM; }
            const int rc = upload_rscale(L);
            if (rc != LIC_OK) return rc;
        }
        for (size_t i = 0; i < ph.size(); ++i) ph[i].woff = (int64_t)pm.off[i];
        // Each layout only where a kernel of this layer reads it: row-major (the
        // image layer at 192 channels), and the same operands in fragment order, of
        // the staged, window and image kernels (FP32 as bf16 parts) and of the others.
        const void* const packed = L.dt == DT_BF16 ? (const void*)hb.data() : L.dt == DT_FP8 ? (const void*)h8.data() : wp.data();
        const size_t esz = L.dt == DT_BF16 ? 2 : L.dt == DT_FP8 ? 1 : 4;
        bool up = true;
        if (use.w) up = (L.d_w = (uint16_t*)upload(packed, total * esz)) != nullptr;
        if (total % 8 != 0) { err = std::string("packing mismatch in ") + sp.name; return LIC_E_MODEL; }
        if (up && use.wx) {                              // each group of 8 values as [part 0 x8][part 1 x8][part 2 x8]
            hx.resize(3 * total);
            for (size_t j = 0; j < total; j += 8) split_parts8(&wp[j], &hx[3 * j], 8);
            up = (L.d_wx = (uint16_t*)upload(hx.data(), hx.size() * sizeof(uint16_t))) != nullptr;
        }
        auto fragments = [&](int form) -> uint8_t* {
            const TileOrder to = tile_order(pm, form);
            static const uint8_t zeros[16] = {};
            wt.resize(to.run.size() * (form == DT_F32X ? 48 : 16));
            for (size_t j = 0; j < to.run.size(); ++j) {
                const size_t x = (size_t)to.run[j];
                if (form == DT_F32X)                     // the lane's 16 bytes of three fragments
                    split_parts8(&wp[x], reinterpret_cast<uint16_t*>(&wt[(j / 64) * 3072 + (j % 64) * 16]), 512);
                else
                    memcpy(&wt[16 * j], to.run[j] < 0 ? zeros : static_cast<const uint8_t*>(packed) + x * esz, 16);
            }
            for (size_t i = 0; i < ph.size(); ++i) ph[i].wtoff = (int64_t)to.off[i];
            return upload(wt.data(), wt.size());
        };
        const int staged_form = L.dt == DT_F32 ? DT_F32X : L.dt;
        if (up && use.wt) up = (L.d_wt = fragments(staged_form)) != nullptr;
        if (up && use.ws) {
            const int form = sp.ld == LD_RGB ? staged_form : L.dt;
            L.d_ws = use.wt && form == staged_form ? L.d_wt : fragments(form);
            up = L.d_ws != nullptr;
        }
        if (up) up = (L.d_ph = (PhaseDesc*)upload(ph.data(), ph.size() * sizeof(PhaseDesc))) != nullptr;
        std::vector<float> bias(L.cop, 0.0f);
        for (int r = 0; r < L.cop; ++r)
            if (pm.bias_idx[r] >= 0) bias[r] = (float)b[pm.bias_idx[r]];
        if (up) up = (L.d_bias = (float*)upload(bias.data(), L.cop * sizeof(float))) != nullptr;

        if (sp.ep == EP_GDN || sp.ep == EP_IGDN) {
            auto git = P.find(std::string(sp.name) + ".gamma");
            auto beit = P.find(std::string(sp.name) + ".beta");
            if (git == P.end() || beit == P.end() || git->second.second.size() != (size_t)co * co ||
                beit->second.second.size() != (size_t)co) {
                err = std::string("weight blob: GDN parameters missing in ") + sp.name;
                return LIC_E_MODEL;
            }
            if (co % 32 != 0) { err = std::string("GDN layers need a multiple of 32 channels: ") + sp.name; return LIC_E_MODEL; }
            const std::vector<uint16_t> g = gdn_gamma_split(git->second.second, co);
            std::vector<float> be(beit->second.second.begin(), beit->second.second.end());
            if (up) up = (L.d_beta = (float*)upload(be.data(), be.size() * sizeof(float))) != nullptr;
            if (up && use.gsplit) up = (L.d_gsplit = (uint16_t*)upload(g.data(), g.size() * sizeof(uint16_t))) != nullptr;
            if (up && use.gt) {
                const std::vector<uint16_t> gt = gdn_gamma_tiles(g, co, L.dt == DT_F32 ? 3 : 2);
                up = (L.d_gt = (uint16_t*)upload(gt.data(), gt.size() * sizeof(uint16_t))) != nullptr;
            }
        }
        if (!up) { err = std::string("device allocation or upload failed: ") + sp.name; return LIC_E_NOMEM; }
        // offsets: quantisation of y (factorized: channel medians; hyperprior: 0)
        // and of z (medians); dequantisation in the loaders likewise
        if (sp.id == LIC_GA3) L.d_qmu = kind == 0 ? d_medians : d_zero;
        if (sp.id == LIC_HA2) L.d_qmu = d_medians;
        if (sp.id == LIC_HS0) L.d_mu_in = d_medians;
        if (sp.id == LIC_GS0) L.d_mu_in = kind == 0 ? d_medians : d_zero;
    }
    if (kind == 2) {
        // kernels are instantiated for these widths (the entropy-parameter
        // layers' K is a template parameter)
        if (N != 128 || M != 192 || layers[LIC_EP1A].cin != 640 || layers[LIC_EP2A].cin != 512 ||
            layers[LIC_EP0A].cin != 4 * M || layers[LIC_EP2A].co != 2 * M || layers[LIC_HS2].co != 2 * M ||
            layers[LIC_CX].co != 2 * M || layers[LIC_CX].cin != M) {
            err = "context model: kernels exist for N = 128, M = 192 (entropy-parameter widths 768, 640, 512, 384)";
            return LIC_E_MODEL;
        }
    }
    return LIC_OK;
}

Geo layer_geo(int id, const FrameDims& d)
{
    const int Hp = d.Hp, Wp = d.Wp, Hy = d.Hy, Wy = d.Wy, Hz = d.Hz, Wz = d.Wz;
    switch (id) {
    case LIC_GA0: return {d.H, d.W, Hp / 2, Wp / 2, 2, Hp / 2, Wp / 2, 1};
    case LIC_GA1: return {Hp / 2, Wp / 2, Hp / 4, Wp / 4, 2, Hp / 4, Wp / 4, 1};
    case LIC_GA2: return {Hp / 4, Wp / 4, Hp / 8, Wp / 8, 2, Hp / 8, Wp / 8, 1};
    case LIC_GA3: return {Hp / 8, Wp / 8, Hy, Wy, 2, Hy, Wy, 1};
    case LIC_HA0: return {Hy, Wy, Hy, Wy, 1, Hy, Wy, 1};
    case LIC_HA1: return {Hy, Wy, Hy / 2, Wy / 2, 2, Hy / 2, Wy / 2, 1};
    case LIC_HA2: return {Hy / 2, Wy / 2, Hz, Wz, 2, Hz, Wz, 1};
    case LIC_HS0: return {Hz, Wz, Hz, Wz, 1, 2 * Hz, 2 * Wz, 2};
    case LIC_HS1: return {2 * Hz, 2 * Wz, 2 * Hz, 2 * Wz, 1, Hy, Wy, 2};
    case LIC_HS2: return {Hy, Wy, Hy, Wy, 1, Hy, Wy, 1};
    case LIC_GS0: return {Hy, Wy, Hy, Wy, 1, 2 * Hy, 2 * Wy, 2};
    case LIC_GS1: return {Hp / 8, Wp / 8, Hp / 8, Wp / 8, 1, Hp / 4, Wp / 4, 2};
    case LIC_GS2: return {Hp / 4, Wp / 4, Hp / 4, Wp / 4, 1, Hp / 2, Wp / 2, 2};
    case LIC_GS3: return {Hp / 2, Wp / 2, Hp / 2, Wp / 2, 1, Hp, Wp, 2};
    case LIC_CX: case LIC_EP0A: case LIC_EP1A: case LIC_EP2A: case LIC_EP0N: case LIC_EP1N: case LIC_EP2N:
        return {Hy, Wy, Hy / 2, Wy / 2, 2, Hy, Wy, 2};        // two stride-2 sub-grids per set
    }
    return {0, 0, 0, 0, 0, 0, 0, 0};
}

// Element size of the activations a layer stores (the GDN layers' forms).
static size_t act_bytes(const LayerGPU& L)
{
    if (L.dt == DT_F32 || L.dt == DT_F32X) return 4;
    if (L.dt == DT_BF16) return L.out_e4m3 ? 1 : 2;
    return L.out_bf16 ? 2 : 1;
}

void Codec::layer_bytes(int id, int n, const FrameDims& d, size_t* in, size_t* out, size_t* aux) const
{
    const Geo g = layer_geo(id, d);
    const size_t nn = (size_t)n;
    const size_t img = nn * 3 * d.H * d.W;
    const size_t px_in = nn * g.Hin * g.Win, px_out = nn * g.Hout * g.Wout;
    *aux = 0;
    if (id >= LIC_CX) {
        // context model (float32 tensors on the full latent grid): cx reads
        // y_hat, ep0 the concatenation [psi; ctx] (4M channels), ep1 / ep2 the
        // hidden layers; ep2 writes indices (and symbols) checkerboard-major
        const size_t pl = nn * d.Hy * d.Wy;
        const LayerGPU& L = layers[id];
        *in = pl * L.cin * 4;
        if (id == LIC_CX) *out = pl * 4 * M * 4;
        else if (L.ep == EP_MSCALE) { *out = pl * M; *aux = pl * M; }
        else *out = pl * L.co * 4;
        return;
    }
    // input: the image, int8 symbols, y / z / hyper activations (FP32), or
    // the previous layer's stored activations
    if (id == LIC_GA0) *in = img * 4;
    else if (id == LIC_GS0 && kind == 2) *in = px_in * layers[id].cin * (layers[id].dt == DT_F32 ? 4 : 2);
    else if (id == LIC_HS0 || id == LIC_GS0) *in = px_in * layers[id].cin;
    else if (id >= LIC_HA0 && id <= LIC_HS2) *in = px_in * layers[id].cin * 4;
    else *in = px_in * layers[id].cin * act_bytes(layers[id - 1]);
    switch (id) {
    case LIC_GA3: case LIC_HA2:                       // float values, int8 symbols
        *out = px_out * layers[id].co * 4;
        *aux = px_out * layers[id].co;
        break;
    case LIC_HS2:                                     // uint8 indices, float values
        if (kind == 2) {                              // psi into [psi; ctx]
            *out = px_out * 4 * M * 4;
            break;
        }
        *out = px_out * layers[id].co;
        *aux = px_out * layers[id].co * 4;
        break;
    case LIC_GS3:                                     // cropped image, padded pre-clamp image
        *out = img * 4;
        *aux = nn * 3 * d.Hp * d.Wp * 4;
        break;
    case LIC_HA0: case LIC_HA1: case LIC_HS0: case LIC_HS1:
        *out = px_out * layers[id].co * 4;
        break;
    default:                                          // GDN layers
        *out = px_out * layers[id].co * act_bytes(layers[id]);
    }
}

int Codec::launch_layer(int id, int n, const FrameDims& d, const void* in, void* out, void* aux, hipStream_t s,
                        std::string* errp, KernelKey* chosen, const void* in2, void* out2)
{
    if (id < 0 || id >= LIC_NUM_LAYERS || !layers[id].present) { *errp = "layer not present in this model"; return LIC_E_ARG; }
    const LayerGPU& L = layers[id];
    const Geo g = layer_geo(id, d);
    ConvArgs a{};
    a.in = in;
    a.out = out;
    a.aux = aux;
    a.ph = L.d_ph;
    a.w = L.d_w;
    a.wx = L.d_wx;
    a.wt = L.d_wt;
    a.ws = L.d_ws;
    a.cin = L.cin;
    a.gt = L.d_gt;
    a.zero = d_zero;
    a.bias = L.d_bias;
    a.mu_in = L.d_mu_in;
    a.gsplit = L.d_gsplit;
    a.beta = L.d_beta;
    a.qmu = L.d_qmu;
    a.thr = d_thr;
    a.n = n;
    a.Hin = g.Hin;
    a.Win = g.Win;
    a.Hg = g.Hg;
    a.Wg = g.Wg;
    a.s_in = g.s_in;
    a.Hout = g.Hout;
    a.Wout = g.Wout;
    a.s_out = g.s_out;
    a.Co = L.co;
    a.nphase = L.nphase;
    a.hs_exp = hs_exp;
    a.norm1 = norm;
    a.Hc = d.H;
    a.Wc = d.W;
    a.kk = L.k;
    a.pad = L.k / 2;
    a.rscale = L.d_rscale;
    a.out_q = L.out_q;
    a.sat = d_sat;
    a.out_e4m3 = L.out_e4m3 ? 1 : 0;
    a.out_bf16 = L.out_bf16 ? 1 : 0;

    // context model: psi and the context fill the two halves of [psi; ctx];
    // the last entropy-parameter layer takes y (encoder) and writes y_hat or
    // the means
    if (kind == 2 && (id == LIC_HS2 || id == LIC_CX)) {
        a.co_ld = 4 * M;
        a.co_off = id == LIC_CX ? 2 * M : 0;
    }
    if (L.ep == EP_MSCALE) {
        if (!out2 && !chosen) { *errp = "the last entropy-parameter layer needs its y_hat / mean output"; return LIC_E_ARG; }
        a.cb_part = id == LIC_EP2A ? 0 : 1;
        a.ysrc = static_cast<const float*>(in2);
        a.yq = static_cast<float*>(out2);
    }
    const ConvShape shape{id, L.ld, L.ep, L.dt, L.cin, L.cop, L.nphase, L.halo1 && g.s_in == 1 ? 1 : 0};
    return launch_conv_policy(shape, a, (long)g.Hg * g.Wg, s, errp, chosen);
}

int layer_route(int kind, int N, int M, int precision, int id, int n, int H, int W, ConvRoute* r, std::string* errp)
{
    for (const LayerSpec& sp : layer_specs(kind)) {
        if (sp.id != id) continue;
        int ci = N, co = N;
        switch (id) {
        case LIC_GA0: ci = 3; break;
        case LIC_GA3: co = M; break;
        case LIC_HA0: case LIC_GS0: ci = M; break;
        case LIC_GS3: co = 3; break;
        case LIC_HS2: co = kind == 2 ? 2 * M : M; break;
        case LIC_CX: ci = M; co = 2 * M; break;
        case LIC_EP0A: case LIC_EP0N: ci = 4 * M; co = 640; break;
        case LIC_EP1A: case LIC_EP1N: ci = 640; co = 512; break;
        case LIC_EP2A: case LIC_EP2N: ci = 512; co = 2 * M; break;
        }
        const Geo g = layer_geo(id, FrameDims(H, W));
        ConvShape L = layer_shape(sp, layer_form(sp, precision), ci, co);
        L.halo1 = L.halo1 && g.s_in == 1 ? 1 : 0;
        ConvArgs a{};
        a.n = n;
        a.Hin = g.Hin;
        a.Win = g.Win;
        a.Hg = g.Hg;
        a.Wg = g.Wg;
        a.s_in = g.s_in;
        a.s_out = g.s_out;
        a.kk = sp.k;
        a.Co = co;
        a.co_ld = kind == 2 && (id == LIC_HS2 || id == LIC_CX) ? 4 * M : 0;
        return choose_route(L, a, (long)g.Hg * g.Wg, r, errp);
    }
    *errp = "layer not present in this model";
    return LIC_E_ARG;
}

}  // namespace lic
