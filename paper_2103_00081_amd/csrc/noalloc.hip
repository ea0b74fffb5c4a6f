// hts_apply_operator without device allocation: every buffer the apply needs
// beyond the mesh's own data and the caller's x and y (the time slots and
// line-source coefficients of the heat operator) lives in one statically sized
// device array per GPU.  For callers that cannot allocate
// (code under graph capture, tight loops, harnesses that forbid it).
#include <cstring>
#include <functional>
#include <mutex>

#include "bc.h"
#include "internal.h"
#include "vec.h"

namespace hts {
hts_status guard_call(const std::function<void()> &f);

namespace {

constexpr size_t SCRATCH_BYTES = (size_t)40 << 20;   // 40 MiB per GPU
// Device scratch of the allocation-free entry point.  In host code this name
// is a host-side stand-in: only the address returned by hipGetSymbolAddress
// (kept per device in g_ptr) is passed to kernels and copies.
__device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];

constexpr int MAX_DEV = 64;
std::mutex g_mu;
unsigned char *g_ptr[MAX_DEV] = {};

unsigned char *scratch_ptr(int dev)
{
    if (dev < 0 || dev >= MAX_DEV) throw Error(HTS_ERR_ARG, "device index out of range");
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            throw Error(HTS_ERR_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_ptr[dev] = static_cast<unsigned char *>(p);
    }
    return g_ptr[dev];
}

// Small host structures reach the device as kernel arguments (no host
// buffer, no copy engine): one blob of up to 2 KiB per launch.
constexpr int BLOB = 2048;
struct Blob {
    unsigned char b[BLOB];
};

__global__ void k_put(unsigned char *__restrict__ dst, Blob blob, int nbytes)
{
    for (int i = threadIdx.x; i < nbytes; i += blockDim.x) dst[i] = blob.b[i];
}

void put(unsigned char *dst, const void *src, size_t nbytes, hipStream_t s)
{
    const unsigned char *p = static_cast<const unsigned char *>(src);
    for (size_t o = 0; o < nbytes; o += BLOB) {
        Blob b;
        const int n = (int)std::min<size_t>(BLOB, nbytes - o);
        std::memcpy(b.b, p + o, (size_t)n);
        k_put<<<dim3(1), dim3(256), 0, s>>>(dst + o, b, n);
        HTS_LAUNCH_CHECK();
    }
}

size_t up256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace
}  // namespace hts

using namespace hts;

extern "C" hts_status hts_apply_operator_noalloc(hts_mesh *m, hts_field field, hts_precision prec, double dt,
                                                 const void *x_dev, void *y_dev)
{
    return guard_call([&] {
        if (!m) throw Error(HTS_ERR_ARG, "null mesh");
        if (!m->has_mat) throw Error(HTS_ERR_STATE, "materials not set");
        if (m->dirty)
            throw Error(HTS_ERR_STATE, "mesh data not prepared: call hts_apply_operator, hts_autotune or a solve "
                                       "once after changing the mesh");
        if (field != 0 && field != 1) throw Error(HTS_ERR_ARG, "bad field");
        if (prec != HTS_FP64 && prec != HTS_FP32) throw Error(HTS_ERR_ARG, "bad precision");
        if (!x_dev || !y_dev || x_dev == y_dev) throw Error(HTS_ERR_ARG, "x and y must be distinct device buffers");
        if (field == 1 && !m->has_state[0]) throw Error(HTS_ERR_STATE, "pressure state not set");
        const hipStream_t s = m->stream;
        const bool fp32 = prec == HTS_FP32;
        const bool steady = field == 0 && (dt <= 0.0 || m->B <= 0.0);
        // What a call needs is the time slots and line sources.  The limit on sizes is an
        // older one and part of the interface (callers size their meshes by it): two
        // descriptors (768 bytes), the tile kernels' work list, the chunk list and an FP32
        // pressure have to fit the scratch as well
        const int family = kernel_family(m, false);
        int ntx, nty;
        tile_grid(m, family, field, !fp32, ntx, nty);
        const int zc = zc_for(m, family, field, fp32 ? 1 : 0, (int64_t)ntx * nty, 0);
        const int64_t nwork = (int64_t)ntx * nty * ((m->N[2] + zc - 1) / zc);
        const int nsrc = field == 1 ? (int)m->line_srcs.size() : 0;
        const int64_t nchunk = (field == 1 && fp32) ? (m->nnode + 1023) / 1024 : 0;
        // layout, 256-byte aligned pieces
        size_t o = 0;
        const size_t o_S = o;      o += up256(NSLOT * sizeof(double));
        const size_t o_src = o;    o += up256((size_t)std::max(1, nsrc) * sizeof(SrcDev));
        const size_t o_coef = o;   o += up256((size_t)std::max(1, nsrc) * sizeof(double));
        const size_t need = o + 768 + up256((size_t)nwork * sizeof(WorkItem)) +
                            up256((size_t)nchunk * sizeof(Chunk)) + up256((size_t)(nchunk ? m->nnode : 0) * sizeof(float));
        if (need > SCRATCH_BYTES || nwork > INT32_MAX)
            throw Error(HTS_ERR_ARG, "mesh too large for the allocation-free apply: needs " + std::to_string(need) +
                                         " bytes of the " + std::to_string(SCRATCH_BYTES) + "-byte scratch");
        HTS_HIP(hipSetDevice(m->desc.device));
        unsigned char *base = scratch_ptr(m->desc.device);
        double *S = reinterpret_cast<double *>(base + o_S);
        SrcDev *srcs = reinterpret_cast<SrcDev *>(base + o_src);
        double *coef = reinterpret_cast<double *>(base + o_coef);

        if (nsrc > 0) {
            // time slots of instance 0, then the line-source coefficients at t + dt
            double hS[NSLOT];
            for (int i = 0; i < NSLOT; i++) hS[i] = 0.0;
            hS[S_TNEW] = m->t + dt;
            hS[S_FSCALE] = dt;
            put(base + o_S, hS, sizeof(hS), s);
            std::vector<SrcDev> ls(m->line_srcs);
            for (SrcDev &sd : ls) sd.inst = 0;
            put(base + o_src, ls.data(), ls.size() * sizeof(SrcDev), s);
            launch_source_values(srcs, nsrc, S, coef, s);
        }
        // one launch, as hts_apply_operator
        const int szc = apply_depth(m, field, fp32);
        OpDev op = make_op(m, field, fp32, dt, steady, false);
        op.P = m->P.p;
        op.lcoef = coef;
        if (fp32) launch_strip_solo<float>(m, field, op, szc, static_cast<const float *>(x_dev),
                                           static_cast<float *>(y_dev), s);
        else launch_strip_solo<double>(m, field, op, szc, static_cast<const double *>(x_dev),
                                       static_cast<double *>(y_dev), s);
    });
}
