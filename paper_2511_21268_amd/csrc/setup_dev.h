// Device execution of the hierarchy set-up (setup_dev.hip): the same
// hierarchy as build_hierarchy on the host, bit for bit.
#pragma once
#include <utility>

#include "host.h"

namespace amgiga {

// While one exists on a thread, the device memory that these functions release
// there is kept for their next requests; the outermost gives it back.  All of
// them then take the same stream.
class SetupMemory {
  public:
    SetupMemory();
    ~SetupMemory();
    SetupMemory(const SetupMemory &) = delete;
    SetupMemory &operator=(const SetupMemory &) = delete;
    static void trim();   // give back what is idle

  private:
    void *pool_ = nullptr;
};

// A CSR matrix in device memory, owned.
struct DevCsr {
    int64_t n = 0, nnz = 0;
    int64_t *rp = nullptr;
    int32_t *ci = nullptr;
    double *v = nullptr;
    DevCsr() = default;
    DevCsr(const DevCsr &) = delete;
    DevCsr &operator=(const DevCsr &) = delete;
    DevCsr(DevCsr &&o) noexcept { *this = std::move(o); }
    DevCsr &operator=(DevCsr &&o) noexcept
    {
        std::swap(n, o.n); std::swap(nnz, o.nnz);
        std::swap(rp, o.rp); std::swap(ci, o.ci); std::swap(v, o.v);
        return *this;
    }
    ~DevCsr();
};

struct DevSetupInfo {
    int sweeps = 0;         // matching sweeps run
    int rounds_total = 0;   // rounds of locally dominant edges, summed
    int rounds_max = 0;     // and the most in one sweep
    std::vector<DevCsr> levels;   // the levels' matrices, for the images built next (level 0: may be there before)
};

// Returns 0 or an amg_status code (err set): -1 unsupported input (smoothed
// prolongator, 2^31 or more stored entries, structurally nonsymmetric matrix),
// -3 HIP failure, -4 host allocation failure; otherwise as build_hierarchy.
int build_hierarchy_on_device(const CsrView &K0, const double *w, const SetupParams &prm, HostHierarchy &H,
                              std::string &err, void *stream, DevSetupInfo *info);

// The pieces of the image set-up that run on the device (stream: hipStream_t);
// 0, or with err set -3, or -4 where device or host memory ran out.
//
// Device copy of a host CSR.
int csr_to_device(const CsrView &K, void *stream, DevCsr &D, std::string &err);
// Whether validate_csr would accept the entries (its row pointers are valid).
int check_csr(const DevCsr &K, void *stream, bool &valid, std::string &err);
// K P (kp_product's bits) from the device copies of K, the aggregates and the
// prolongator's coefficients; rp: its row pointers on the host, max_gap: the
// widest column gap within a row.  K has fewer than 2^31 entries.
int kp_on_device(const DevCsr &K, int64_t nc, const int32_t *agg, const double *pc, void *stream, DevCsr &KP,
                 std::vector<int64_t> &rp, int64_t &max_gap, std::string &err);
// The entries of a SELL-C image laid out by sell_layout, from the device copy
// of its matrix; the arrays that are not wanted are NULL (v32 rounds v).
struct SellFill {
    const int64_t *soff, *ibase;
    const int32_t *perm, *shoff, *ulen;   // perm: NULL in row order; shoff, ulen: NULL without shared lists
    double *v64;
    float *v32;
    uint16_t *d16;
    int32_t *col0, *c32, *gcol;
};
int fill_sell(const DevCsr &K, int C, int64_t nslices, const SellFill &F, void *stream, std::string &err);
// The same from the host's CSR, uploaded piece by piece; returns with the
// stream idle.
int fill_sell(const CsrView &K, int C, const SellFill &F, void *stream, std::string &err);

}  // namespace amgiga
