// Minimum-norm estimate of eqn5 for every sample of the data:
//   G = C X^T (N x m),  S = X G + R,  L Li = chol(S),  J^T = G (Li^T (Li Y^T)),
// two entry points over the same launches: mne_solve allocates its workspace for the call,
// mne_solve_noalloc takes it from a fixed device array (for callers that cannot allocate); and the
// parameter set-up of Section 2.4 from it, kf_init_from_mne.
#include "kf_internal.h"
#include "../../include/kfmeg.h"

#include <mutex>
#include <string>

using namespace kfmeg;

namespace {

// Workspace of the allocation-free entry point: one array per device, held until the process
// ends. Host code never passes `scratch` itself to a kernel (in host code the name is a host-side
// stand-in); it uses the device address that hipGetSymbolAddress returns for the current device.
constexpr size_t kScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's scratch array, looked up once per device.
hipError_t scratch_address(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

// Workspace of the allocating entry points: stream-ordered memory from a pool of this library, one per device.
// hipMalloc and hipFree cost 0.1 to 0.3 ms a call (a sixth of an estimate at N = 5124, a third of
// the set-up) and wait for the whole device. The pool lends at most kPoolKeep bytes at a time and so keeps no more
// between calls: what goes beyond, whose calls take milliseconds, comes from hipMalloc (the runtime gives a pool's
// surplus back only at a later synchronisation). The driver orders reuse by stream, whichever threads call. Where
// pools are not supported the calls allocate as before.
constexpr uint64_t kPoolKeep = (uint64_t)128 << 20;
hipMemPool_t g_pool[kMaxDevices] = {};
bool g_pool_tried[kMaxDevices] = {};
uint64_t g_pool_lent[kMaxDevices] = {};

// The current device's pool with `bytes` of it taken, or null.
hipMemPool_t workspace_pool(uint64_t bytes, int& dev) {
    int ok = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return nullptr;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_pool_tried[dev]) {
        g_pool_tried[dev] = true;
        hipMemPoolProps pr{};
        pr.allocType = hipMemAllocationTypePinned;
        pr.location.type = hipMemLocationTypeDevice;
        pr.location.id = dev;
        hipMemPool_t p = nullptr;
        uint64_t keep = kPoolKeep;
        if (hipDeviceGetAttribute(&ok, hipDeviceAttributeMemoryPoolsSupported, dev) == hipSuccess && ok &&
            hipMemPoolCreate(&p, &pr) == hipSuccess &&
            hipMemPoolSetAttribute(p, hipMemPoolAttrReleaseThreshold, &keep) == hipSuccess)
            g_pool[dev] = p;
        else
            (void)hipGetLastError();
    }
    if (!g_pool[dev] || bytes > kPoolKeep - g_pool_lent[dev]) return nullptr;
    g_pool_lent[dev] += bytes;
    return g_pool[dev];
}
void workspace_returned(uint64_t bytes, int dev) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    g_pool_lent[dev] -= bytes;
}

// A block of the pool (or of hipMalloc) for one call on one stream.
struct Workspace {
    void* base = nullptr;
    hipStream_t s;
    uint64_t lent = 0;                     // bytes of the pool that base holds; 0: hipMalloc
    int dev = 0;
    Workspace(size_t bytes, hipStream_t s_) : s(s_) {
        if (hipMemPool_t p = workspace_pool(bytes, dev)) {
            if (hipMallocFromPoolAsync(&base, bytes, p, s) == hipSuccess) {
                lent = bytes;
                return;
            }
            workspace_returned(bytes, dev);
        }
        base = nullptr;
        (void)hipGetLastError();
        if (hipMalloc(&base, bytes) != hipSuccess) {
            (void)hipGetLastError();
            base = nullptr;
        }
    }
    ~Workspace() {
        if (!base) return;
        if (!lent) {
            (void)hipFree(base);
            return;
        }
        (void)hipFreeAsync(base, s);
        workspace_returned(lent, dev);
    }
    Workspace(const Workspace&) = delete;
    Workspace& operator=(const Workspace&) = delete;
};

int64_t round_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

struct MneWork {
    double *G = nullptr, *S = nullptr, *Lis = nullptr, *U = nullptr, *V = nullptr, *part = nullptr;
    DevStatus* status = nullptr;
};

struct MneShape {
    int64_t ldm, ldT;
    int ksplit;        // K slices of S = X G + R
    int gsplit;        // K slices of G = C X^T
    size_t off[7];     // byte offsets of G, S, Lis, U, V, part, status (256-byte aligned)
    size_t total;
};

// G = C X^T is most of the work (2 N^2 m operations) in N / 128 x m / 128 tiles, too few to fill the device
// between about 64 and 256 of them: its K range is then cut in up to four slices. At N = 5124, m = 306 (123
// tiles) that takes 335 us, unsplit 554 us on small tiles. The slices' partial sums share the space of S's;
// there are only as many as leave a shape within the fixed array where one slice does, so
// that both entry points run the same launches and accept what they did.
MneShape mne_shape(int64_t N, int64_t m, int64_t T) {
    MneShape sh;
    sh.ldm = round_up(m, 16);
    sh.ldT = round_up(T, 16);
    sh.ksplit = (int)std::max<int64_t>(1, std::min<int64_t>(32, N / 128));
    const int64_t tiles = ((N + 127) / 128) * ((m + 127) / 128);
    sh.gsplit = tiles >= 64 && tiles <= 256 ? 4 : 1;
    for (;; --sh.gsplit) {
        const int64_t part = std::max<int64_t>(sh.ksplit * m * m, sh.gsplit > 1 ? sh.gsplit * N * m : 0);
        const size_t bytes[7] = {8 * (size_t)N * sh.ldm, 8 * (size_t)m * sh.ldm, 8 * (size_t)m * sh.ldm,
                                 8 * (size_t)m * sh.ldT, 8 * (size_t)m * sh.ldT, 8 * (size_t)part, sizeof(DevStatus)};
        size_t o = 0;
        for (int k = 0; k < 7; ++k) {
            sh.off[k] = o;
            o += (bytes[k] + 255) / 256 * 256;
        }
        sh.total = o;
        if (sh.total <= kScratchBytes || sh.gsplit == 1) return sh;
    }
}

MneWork carve(void* base, const MneShape& sh) {
    char* b = static_cast<char*>(base);
    MneWork w;
    w.G = reinterpret_cast<double*>(b + sh.off[0]);
    w.S = reinterpret_cast<double*>(b + sh.off[1]);
    w.Lis = reinterpret_cast<double*>(b + sh.off[2]);
    w.U = reinterpret_cast<double*>(b + sh.off[3]);
    w.V = reinterpret_cast<double*>(b + sh.off[4]);
    w.part = reinterpret_cast<double*>(b + sh.off[5]);
    w.status = reinterpret_cast<DevStatus*>(b + sh.off[6]);
    return w;
}

#define MCK(expr)                                                                   \
    do {                                                                            \
        hipError_t _e = (expr);                                                     \
        if (_e != hipSuccess) {                                                     \
            err = std::string(#expr) + ": " + hipGetErrorString(_e);                \
            return KF_EHIP;                                                         \
        }                                                                           \
    } while (0)

// eqn5 for every row of Y on `s` with workspace w, then wait for the stream and read the status.
kf_status mne_run(int64_t N, int64_t m, int64_t T, const double* X, const double* C, const double* R,
                  const double* Y, double* J, hipStream_t s, const MneShape& sh, const MneWork& w,
                  std::string& err) {
    MCK(status_clear(w.status, s));
    GemmProblem g;                       // G = C X^T   (N x m)
    g.M = (int)N; g.N = (int)m; g.K = (int)N;
    g.A = C; g.lda = N; g.B = X; g.ldb = N; g.flags = G_TB;
    g.C = w.G; g.ldc = sh.ldm;
    g.ksplit = sh.gsplit;
    g.partial = w.part;
    MCK(gemm1(Dt::F64, g, s));
    GemmProblem h;                       // S = X G + R (lower triangle: all that the factorisation reads)
    h.M = (int)m; h.N = (int)m; h.K = (int)N;
    h.A = X; h.lda = N; h.B = w.G; h.ldb = sh.ldm; h.flags = G_LOWER;
    h.Cin = R; h.ldcin = m; h.beta = 1.0;
    h.C = w.S; h.ldc = sh.ldm;
    h.ksplit = sh.ksplit;
    h.partial = w.part;
    MCK(gemm1(Dt::F64, h, s));
    MCK(chol_inv(w.S, sh.ldm, w.Lis, sh.ldm, (int)m, w.status, W_MNE, 0, s));
    GemmProblem u;                       // U = Li Y^T   (m x T)
    u.M = (int)m; u.N = (int)T; u.K = (int)m;
    u.A = w.Lis; u.lda = sh.ldm; u.flags = G_ALOWER | G_TB;
    u.B = Y; u.ldb = m;
    u.C = w.U; u.ldc = sh.ldT;
    MCK(gemm1(Dt::F64, u, s));
    GemmProblem v;                       // V = Li^T U = S^{-1} Y^T
    v.M = (int)m; v.N = (int)T; v.K = (int)m;
    v.A = w.Lis; v.lda = sh.ldm; v.flags = G_TA;
    v.B = w.U; v.ldb = sh.ldT;
    v.C = w.V; v.ldc = sh.ldT;
    MCK(gemm1(Dt::F64, v, s));
    GemmProblem j;                       // J = V^T G^T   (T x N)
    j.M = (int)T; j.N = (int)N; j.K = (int)m;
    j.A = w.V; j.lda = sh.ldT; j.flags = G_TA | G_TB;
    j.B = w.G; j.ldb = sh.ldm;
    j.C = J; j.ldc = N;
    MCK(gemm1(Dt::F64, j, s));
    DevStatus hstat{};
    MCK(hipMemcpyAsync(&hstat, w.status, sizeof hstat, hipMemcpyDeviceToHost, s));
    MCK(hipStreamSynchronize(s));
    if (hstat.key != kStatusClear) {
        err = "mne_solve: X C X^T + R is not positive definite (pivot row " + std::to_string(status_row(hstat.key)) +
              ")";
        return KF_ENOTPD;
    }
    return KF_OK;
}

bool args_ok(int64_t N, int64_t m, int64_t T, const void* X, const void* C, const void* R, const void* Y,
             const void* J) {
    return N > 0 && m > 0 && T > 0 && N <= (1 << 20) && m <= (1 << 16) && T <= (1 << 24) && X && C && R && Y && J;
}

}  // namespace

extern "C" {

kf_status mne_solve(int64_t N, int64_t m, int64_t T, const double* X, const double* C, const double* R,
                    const double* Y, double* J, void* stream) {
    set_last_error("");
    if (!args_ok(N, m, T, X, C, R, Y, J)) {
        set_last_error("mne_solve: sizes must be positive (N <= 2^20, m <= 2^16, T <= 2^24) and pointers non-null");
        return KF_EINVAL;
    }
    const MneShape sh = mne_shape(N, m, T);
    Workspace ws(sh.total, static_cast<hipStream_t>(stream));
    void* base = ws.base;
    if (!base) {
        set_last_error("mne_solve: device allocation of " + std::to_string(sh.total) + " bytes failed");
        return KF_ENOMEM;
    }
    std::string err;
    const kf_status st = mne_run(N, m, T, X, C, R, Y, J, static_cast<hipStream_t>(stream), sh, carve(base, sh), err);
    if (st == KF_EHIP) (void)hipStreamSynchronize(static_cast<hipStream_t>(stream));
    if (st != KF_OK) set_last_error(err);
    return st;
}

kf_status mne_solve_noalloc(int64_t N, int64_t m, int64_t T, const double* X, const double* C, const double* R,
                            const double* Y, double* J, void* stream) {
    set_last_error("");
    if (!args_ok(N, m, T, X, C, R, Y, J)) {
        set_last_error("mne_solve_noalloc: sizes must be positive (N <= 2^20, m <= 2^16, T <= 2^24) and "
                       "pointers non-null");
        return KF_EINVAL;
    }
    const MneShape sh = mne_shape(N, m, T);
    if (sh.total > kScratchBytes) {
        set_last_error("mne_solve_noalloc: this shape needs " + std::to_string(sh.total) +
                       " bytes of workspace; the fixed device array holds " + std::to_string(kScratchBytes));
        return KF_EINVAL;
    }
    void* base = nullptr;
    const hipError_t e = scratch_address(&base);
    if (e != hipSuccess) {
        set_last_error(std::string("mne_solve_noalloc: device address of the scratch array: ") + hipGetErrorString(e));
        return KF_EHIP;
    }
    std::string err;
    const kf_status st = mne_run(N, m, T, X, C, R, Y, J, static_cast<hipStream_t>(stream), sh, carve(base, sh), err);
    if (st == KF_EHIP) (void)hipStreamSynchronize(static_cast<hipStream_t>(stream));
    if (st != KF_OK) set_last_error(err);
    return st;
}

// Section 2.4: the estimates J, their centred differences and one SYRK. One allocation holds the estimate's
// workspace, J and the differences.
kf_status kf_init_from_mne(int64_t N, int64_t m, int64_t T, const double* X, const double* C, const double* R,
                           const double* Y, double reg, double* x0_out, double* Q_out, void* stream) {
    set_last_error("");
    if (N <= 0 || m <= 0 || T < 3 || !X || !C || !R || !Y || !x0_out || !Q_out || !(reg >= 0.0)) {
        set_last_error("kf_init_from_mne: need N, m > 0, T >= 3, reg >= 0 and non-null pointers");
        return KF_EINVAL;
    }
    if (!args_ok(N, m, T, X, C, R, Y, x0_out)) {
        set_last_error("kf_init_from_mne: sizes must be positive (N <= 2^20, m <= 2^16, T <= 2^24)");
        return KF_EINVAL;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const MneShape sh = mne_shape(N, m, T);
    const int64_t ld = round_up(N, 16);
    const size_t jbytes = (8 * (size_t)T * N + 255) / 256 * 256, total = sh.total + jbytes + 8 * (size_t)(T - 1) * ld;
    Workspace ws(total, s);
    void* base = ws.base;
    if (!base) {
        set_last_error("kf_init_from_mne: device allocation of " + std::to_string(total) + " bytes failed");
        return KF_ENOMEM;
    }
    double* J = reinterpret_cast<double*>(static_cast<char*>(base) + sh.total);
    double* Dc = reinterpret_cast<double*>(static_cast<char*>(base) + sh.total + jbytes);
    std::string err;
    auto run = [&]() -> kf_status {
        const kf_status r = mne_run(N, m, T, X, C, R, Y, J, s, sh, carve(base, sh), err);   // eqn5 at every sample
        if (r != KF_OK) return r;
        MCK(diff_center(J, N, (int)T, (int)N, Dc, ld, s));                   // J_k - J_{k-1}, centred
        GemmProblem g;                                                       // Dc^T Dc / (T - 2)
        g.M = (int)N; g.N = (int)N; g.K = (int)(T - 1);
        g.A = Dc; g.lda = ld; g.B = Dc; g.ldb = ld; g.flags = G_TA | G_LOWER | G_MIRROR;
        g.alpha = 1.0 / (double)(T - 2);
        g.C = Q_out; g.ldc = N;
        MCK(gemm1(Dt::F64, g, s));
        if (reg > 0.0) MCK(add_diag(Q_out, N, (int)N, reg, s));
        MCK(hipMemcpyAsync(x0_out, J, N * sizeof(double), hipMemcpyDeviceToDevice, s));
        MCK(hipStreamSynchronize(s));
        return KF_OK;
    };
    const kf_status st = run();
    if (st == KF_EHIP) (void)hipStreamSynchronize(s);
    if (st != KF_OK) set_last_error(err);
    return st;
}

}  // extern "C"

#undef MCK
