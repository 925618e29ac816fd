// libsv host: the batched p = 1 landscape scan (sv_batch_p1_scan).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "sv_host.h"

// ============================================================================ batch scan
// Direct scan: every grid point of every instance mixes its 2^n amplitudes.  Outputs of
// instance i start at n_gamma * n_beta * i.
static int direct_scan(int n_inst, const sv_ising* insts, int n_gamma, const double* gammas, int n_beta,
                       const double* betas, sv_dtype dtype, void* stream, double* energy_out, double* pgs_out) {
    const int wide = dtype == SV_C64 ? knob_for("batchwide", (int)dtype, 0) : knob_for("batch128", (int)dtype, 0);
    const int lut_cap = batch_lut_cap((int)dtype, wide);
    const int S = batch_lds_bits((int)dtype, wide);
    std::vector<BatchInst> bi(n_inst);
    std::vector<double> hh, JJ;
    std::vector<int32_t> ii, jj;
    uint64_t etot = 0;
    int max_n = 1;
    for (int i = 0; i < n_inst; i++) {
        const sv_ising_s* H = insts[i];
        BatchInst& b = bi[i];
        b.n = H->n;
        b.m = H->m;
        b.hoff = (int32_t)hh.size();
        b.coff = (int32_t)JJ.size();
        b.eoff = etot;
        etot += 1ull << H->n;
        max_n = std::max(max_n, H->n);
        hh.insert(hh.end(), H->h.begin(), H->h.end());
        JJ.insert(JJ.end(), H->J.begin(), H->J.end());
        ii.insert(ii.end(), H->ei.begin(), H->ei.end());
        jj.insert(jj.end(), H->ej.begin(), H->ej.end());
        b.emin = 0.0;  // filled on the device
        b.etol = ground_tol(H);
        const int L = (int)std::ceil(H->scale);
        if (H->integer && 2 * L + 1 <= lut_cap) {
            b.lut_lo = -L;
            b.lut_n = 2 * L + 1;
        } else {
            b.lut_lo = 0;
            b.lut_n = 0;
        }
    }
    // work units (instance, gamma), largest state first
    std::vector<int32_t> uinst, ugam;
    std::vector<int> order(n_inst);
    for (int i = 0; i < n_inst; i++) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return bi[x].n > bi[y].n; });
    for (int i : order)
        for (int a = 0; a < n_gamma; a++) {
            uinst.push_back(i);
            ugam.push_back(a);
        }
    const size_t elem = elem_size(dtype);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    const int grid = device_cu_count(dev) * (wide == 2 ? 2 : 1);
    // states above the LDS tile: the sliced path (slab launches) where the variant has
    // 13-bit LDS states, else per-workgroup slots of the persistent kernel
    const int slab_mb = knob_for("batchslab", (int)dtype, 0);
    const bool sliced = slab_mb > 0 && S == 13 && max_n > S;
    const uint64_t slot = (max_n > S && !sliced) ? (1ull << max_n) : 0;
    const size_t slab_bytes = sliced ? std::max((size_t)slab_mb << 20, (size_t(1) << max_n) * elem_size(dtype)) : 0;
    auto states_per_launch = [&](int n) -> int64_t {
        return std::max<int64_t>(1, (int64_t)(slab_bytes / ((size_t(1) << n) * elem_size(dtype))));
    };
    size_t part_doubles = 0;
    if (sliced)
        for (int n = S + 1; n <= max_n; n++)
            part_doubles = std::max(part_doubles, (size_t)states_per_launch(n) * 2 << (n - batch_slice_bits((int)dtype, n)));
    const size_t nout = (size_t)n_inst * n_gamma * n_beta;
    hipStream_t st = (hipStream_t)stream;
    // device buffers
    std::vector<void*> bufs;
    bool oom = false;
    auto dalloc = [&](size_t bytes) -> void* {
        void* p = nullptr;
        if (hipMalloc(&p, std::max<size_t>(bytes, 16)) != hipSuccess) {
            (void)hipGetLastError();
            oom = true;
            return nullptr;
        }
        bufs.push_back(p);
        return p;
    };
    auto cleanup = [&]() {
        for (void* p : bufs) (void)hipFree(p);
        bufs.clear();
    };
    BatchArgs ba;
    memset(&ba, 0, sizeof(ba));
    BatchInst* d_inst = (BatchInst*)dalloc(bi.size() * sizeof(BatchInst));
    double* d_h = (double*)dalloc(hh.size() * sizeof(double));
    double* d_J = (double*)dalloc(JJ.size() * sizeof(double));
    int32_t* d_ei = (int32_t*)dalloc(ii.size() * sizeof(int32_t));
    int32_t* d_ej = (int32_t*)dalloc(jj.size() * sizeof(int32_t));
    double* d_e = (double*)dalloc(etot * sizeof(double));
    uint16_t* d_x = (uint16_t*)dalloc(etot * sizeof(uint16_t));
    int32_t* d_ui = (int32_t*)dalloc(uinst.size() * sizeof(int32_t));
    int32_t* d_ug = (int32_t*)dalloc(ugam.size() * sizeof(int32_t));
    double* d_g = (double*)dalloc(n_gamma * sizeof(double));
    double* d_b = (double*)dalloc(n_beta * sizeof(double));
    double* d_oe = (double*)dalloc(nout * sizeof(double));
    double* d_op = (double*)dalloc(nout * sizeof(double));
    unsigned* d_cnt = (unsigned*)dalloc(sizeof(unsigned));
    void* d_scr = dalloc(slot * grid * elem);
    void* d_slab = sliced ? dalloc(slab_bytes) : nullptr;
    // partial sums, two buffers: a launch's columns fill one while its slice kernel
    // finishes the previous launch's states from the other
    double* d_part = sliced ? (double*)dalloc(2 * part_doubles * sizeof(double)) : nullptr;
    if (oom) {
        cleanup();
        return fail(SV_ERR_OOM, "sv_batch_p1_scan: device allocation failed");
    }
    hipError_t e = hipSuccess;
    auto up = [&](void* d, const void* h, size_t bytes) {
        if (e == hipSuccess && bytes) e = hipMemcpyAsync(d, h, bytes, hipMemcpyHostToDevice, st);
    };
    up(d_inst, bi.data(), bi.size() * sizeof(BatchInst));
    up(d_h, hh.data(), hh.size() * sizeof(double));
    up(d_J, JJ.data(), JJ.size() * sizeof(double));
    up(d_ei, ii.data(), ii.size() * sizeof(int32_t));
    up(d_ej, jj.data(), jj.size() * sizeof(int32_t));
    up(d_ui, uinst.data(), uinst.size() * sizeof(int32_t));
    up(d_ug, ugam.data(), ugam.size() * sizeof(int32_t));
    up(d_g, gammas, n_gamma * sizeof(double));
    up(d_b, betas, n_beta * sizeof(double));
    if (e == hipSuccess) e = hipMemsetAsync(d_cnt, 0, sizeof(unsigned), st);
    ba.inst = d_inst;
    ba.ninst = n_inst;
    ba.h = d_h;
    ba.ei = d_ei;
    ba.ej = d_ej;
    ba.J = d_J;
    ba.etab = d_e;
    ba.eidx = d_x;
    ba.unit_inst = d_ui;
    ba.unit_gam = d_ug;
    ba.nunits = (int32_t)uinst.size();
    ba.gammas = d_g;
    ba.ng = n_gamma;
    ba.betas = d_b;
    ba.nb = n_beta;
    ba.out_e = d_oe;
    ba.out_p = d_op;
    ba.counter = d_cnt;
    ba.scratch = d_scr;
    ba.scratch_elems = slot;
    int ke = 0;
    if (e == hipSuccess) ke = launch_batch_energy(ba, max_n, st);
    if (e == hipSuccess && !ke) {
        hipEvent_t ev0;
        const bool prof = prof_begin(st, &ev0);
        if (!sliced) {
            ke = launch_batch_scan((int)dtype, ba, grid, wide, st);
        } else {
            // units are sorted by n, largest first: those with n <= S take the persistent
            // kernel, the others go through slab launches of one n each
            size_t first_small = 0;
            while (first_small < uinst.size() && bi[uinst[first_small]].n > S) first_small++;
            if (first_small < uinst.size()) {
                BatchArgs bs = ba;
                bs.unit_inst = d_ui + first_small;
                bs.unit_gam = d_ug + first_small;
                bs.nunits = (int32_t)(uinst.size() - first_small);
                ke = launch_batch_scan((int)dtype, bs, grid, wide, st);
            }
            BatchArgs prev = ba;  // the launch whose states are still to be finished
            prev.s_count = 0;
            int nlaunch = 0;
            auto finish_of = [&](BatchArgs& bs) {
                bs.f_n = prev.s_n;
                bs.f_nh = prev.s_count > 0 ? prev.s_n - batch_slice_bits((int)dtype, prev.s_n) : 0;
                bs.f_u0 = prev.s_u0;
                bs.f_base = prev.s_base;
                bs.f_count = prev.s_count;
                bs.f_part = prev.part;
            };
            for (size_t u0 = 0; u0 < first_small && !ke;) {
                const int n = bi[uinst[u0]].n;
                size_t u1 = u0;
                while (u1 < first_small && bi[uinst[u1]].n == n) u1++;
                const int64_t states = (int64_t)(u1 - u0) * n_beta;
                const int64_t per = states_per_launch(n);
                for (int64_t s0 = 0; s0 < states && !ke; s0 += per) {
                    BatchArgs bs = ba;
                    bs.s_n = n;
                    bs.s_u0 = (int32_t)u0;
                    bs.s_base = s0;
                    bs.s_count = (int32_t)std::min(per, states - s0);
                    bs.slab = d_slab;
                    bs.part = d_part + (nlaunch & 1) * part_doubles;
                    finish_of(bs);
                    ke = launch_batch_sliced((int)dtype, bs, wide, st);
                    prev = bs;
                    nlaunch++;
                }
                u0 = u1;
            }
            if (!ke && prev.s_count > 0) {
                BatchArgs bs = ba;
                finish_of(bs);
                ke = launch_batch_finish(bs, st);
            }
        }
        if (prof) prof_end(st, ev0, std::string("batch_") + (dtype == SV_C128 ? "c128" : "c64"), 0.0);
    }
    if (e == hipSuccess && !ke) e = hipMemcpyAsync(energy_out, d_oe, nout * sizeof(double), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && !ke) e = hipMemcpyAsync(pgs_out, d_op, nout * sizeof(double), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && !ke) e = hipStreamSynchronize(st);
    cleanup();
    if (ke) return fail(SV_ERR_HIP, "batch launch failed: %s", hipGetErrorString((hipError_t)ke));
    if (e != hipSuccess) return fail(SV_ERR_HIP, "sv_batch_p1_scan: %s", hipGetErrorString(e));
    return SV_OK;
}

// Device memory of one scan: one allocation, carved up, freed with the object.
namespace {
struct Arena {
    char* base = nullptr;
    size_t used = 0;
    size_t take(size_t bytes) {
        const size_t at = used;
        used += (bytes + 255) & ~size_t(255);
        return at;
    }
    bool alloc() {
        if (hipMalloc(&base, std::max<size_t>(used, 256)) == hipSuccess) return true;
        (void)hipGetLastError();
        base = nullptr;
        return false;
    }
    template <typename X>
    X* at(size_t off) const {
        return reinterpret_cast<X*>(base + off);
    }
    ~Arena() {
        if (base) (void)hipFree(base);
    }
};
}  // namespace

// The instances an energy grid and their table sizes allow the sphere sums for.
static bool scan_by_spheres(const sv_ising_s* H) {
    if (H->qden <= 0 || H->n > kScanMaxN) return false;
    const double L = H->qden * H->scale;
    return (H->n + 1) * (2.0 * L + 1.0) * 4.0 <= (double)kScanMaxLds;
}

constexpr int kScanGammas = 1024;  // gammas of one launch at most
static int64_t scan_coef_blocks(int n_gamma) { return ((int64_t)n_gamma + 3) / 4; }

// Instances of one sphere_scan: the launches over instances (of 256 threads, with scan_coef_blocks,
// kScanGammas or 32 workgroups for each) hold less than 2^32 threads.
static size_t scan_instances(int n_gamma) {
    const int64_t per = std::max<int64_t>({scan_coef_blocks(n_gamma), std::min(n_gamma, kScanGammas), 32});
    return (size_t)(((int64_t(1) << 24) - 1) / per);
}

// Scan by sphere sums (sv_scan.hip) of instances idx[].  done[k] = 0 for those with too many
// ground states, which are left to the direct scan.
static int sphere_scan(const std::vector<int>& idx, const sv_ising* insts, int n_gamma, const double* gammas,
                       int n_beta, const double* betas, hipStream_t st, double* energy_out, double* pgs_out,
                       std::vector<char>& done) {
    const int ni = (int)idx.size();
    const size_t pts = (size_t)n_gamma * n_beta;
    // A ground state costs one pass over 2^n indices, a grid point of the direct scan n mixer
    // passes over 2^n amplitudes: as many ground states as grid points are taken (at most 4096,
    // which bounds the list).
    const size_t zmax = std::min<size_t>(pts, 4096);
    std::vector<ScanInst> si(ni);
    std::vector<int32_t> hq, cq, stat(3 * (size_t)ni);
    uint64_t xtot = 0;
    int64_t ztot = 0;
    int max_n = 1;
    for (int k = 0; k < ni; k++) {
        const sv_ising_s* H = insts[idx[k]];
        ScanInst& s = si[k];
        s.n = H->n;
        s.m = H->m;
        s.hoff = (int32_t)hq.size();
        s.coff = (int32_t)(cq.size() / 3);
        s.xoff = xtot;
        s.q = H->qden;
        s.lo = -(int32_t)std::lround(H->qden * H->scale);
        s.zcap = (int32_t)std::min<size_t>(zmax, size_t(1) << H->n);
        s.zoff = ztot;
        s.out = k;
        xtot += std::max<uint64_t>(8, 1ull << H->n);
        ztot += s.zcap;
        max_n = std::max(max_n, H->n);
        for (double v : H->h) hq.push_back((int32_t)std::lround(v * H->qden));
        for (int e = 0; e < H->m; e++) {
            cq.push_back(H->ei[e]);
            cq.push_back(H->ej[e]);
            cq.push_back((int32_t)std::lround(H->J[e] * H->qden));
        }
        stat[3 * (size_t)k] = INT32_MAX;
        stat[3 * (size_t)k + 1] = -1;
        stat[3 * (size_t)k + 2] = 0;
    }
    // one allocation: inputs (copied in one go), tables, outputs
    Arena ar;
    const size_t o_inst = ar.take(ni * sizeof(ScanInst)), o_h = ar.take(hq.size() * 4), o_c = ar.take(cq.size() * 4),
                 o_stat = ar.take(stat.size() * 4), o_g = ar.take(n_gamma * sizeof(double)),
                 o_b = ar.take(n_beta * sizeof(double));
    const size_t in_bytes = ar.used;
    const size_t o_x = ar.take(xtot * 2), o_z = ar.take((size_t)ztot * 4),
                 o_coef = ar.take((size_t)ni * n_gamma * 3 * sizeof(double));
    const size_t nout = (size_t)ni * pts;
    const size_t o_e = ar.take(nout * sizeof(double)), o_p = ar.take(nout * sizeof(double));
    if (!ar.alloc()) return fail(SV_ERR_OOM, "sv_batch_p1_scan: device allocation failed");
    std::vector<char> blob(in_bytes);
    memcpy(blob.data() + o_inst, si.data(), ni * sizeof(ScanInst));
    memcpy(blob.data() + o_h, hq.data(), hq.size() * 4);
    if (!cq.empty()) memcpy(blob.data() + o_c, cq.data(), cq.size() * 4);
    memcpy(blob.data() + o_stat, stat.data(), stat.size() * 4);
    memcpy(blob.data() + o_g, gammas, n_gamma * sizeof(double));
    memcpy(blob.data() + o_b, betas, n_beta * sizeof(double));
    hipError_t e = hipMemcpyAsync(ar.base, blob.data(), in_bytes, hipMemcpyHostToDevice, st);
    ScanArgs a;
    memset(&a, 0, sizeof(a));
    a.inst = ar.at<ScanInst>(o_inst);
    a.hq = ar.at<int32_t>(o_h);
    a.cq = ar.at<int32_t>(o_c);
    a.x = ar.at<uint16_t>(o_x);
    a.stat = ar.at<int32_t>(o_stat);
    a.z = ar.at<uint32_t>(o_z);
    a.coef = ar.at<double>(o_coef);
    a.gammas = ar.at<double>(o_g);
    a.betas = ar.at<double>(o_b);
    a.out_e = ar.at<double>(o_e);
    a.out_p = ar.at<double>(o_p);
    a.ng = n_gamma;
    a.nb = n_beta;
    a.bpi = (uint32_t)std::min(32, std::max(1, (1 << max_n) / (256 * 8)));
    a.gpb = (uint32_t)scan_coef_blocks(n_gamma);
    int ke = 0;
    if (e == hipSuccess) ke = launch_scan_tables(a, ni, st);
    if (e == hipSuccess && !ke)
        e = hipMemcpyAsync(stat.data(), a.stat, stat.size() * 4, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && !ke) e = hipStreamSynchronize(st);
    if (ke || e != hipSuccess)
        return fail(SV_ERR_HIP, "sv_batch_p1_scan: %s", hipGetErrorString(ke ? (hipError_t)ke : e));
    // units: the ground states of the instances taken, largest states first
    std::vector<int> order(ni);
    for (int k = 0; k < ni; k++) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return si[x].n > si[y].n; });
    std::vector<int32_t> uinst, oinst;
    std::vector<int64_t> uoff(ni, 0);
    size_t lds = 0;
    for (int k : order) {
        done[k] = stat[3 * (size_t)k + 2] <= si[k].zcap;
        if (!done[k]) continue;
        uoff[k] = (int64_t)uinst.size();
        uinst.insert(uinst.end(), (size_t)stat[3 * (size_t)k + 2], k);
        oinst.push_back(k);
        lds = std::max(lds, (size_t)(si[k].n + 1) * (stat[3 * (size_t)k + 1] - stat[3 * (size_t)k] + 1) * 4);
    }
    if (uinst.empty()) return SV_OK;
    // sphere sums of a launch: up to 1024 gammas, and as many ground states as fit 64 MiB
    const int gc = std::min(n_gamma, kScanGammas);
    const size_t per_unit = (size_t)gc * (kScanMaxN + 1) * sizeof(double2);
    const int64_t units_max =
        std::max<int64_t>(1, std::min<int64_t>((int64_t)uinst.size(), (int64_t)((size_t(64) << 20) / per_unit)));
    Arena au;
    const size_t o_uoff = au.take(ni * sizeof(int64_t)), o_oinst = au.take(oinst.size() * 4),
                 o_uinst = au.take(uinst.size() * 4);
    const size_t u_bytes = au.used, o_amps = au.take((size_t)units_max * per_unit);
    if (!au.alloc()) return fail(SV_ERR_OOM, "sv_batch_p1_scan: device allocation failed");
    blob.assign(u_bytes, 0);
    memcpy(blob.data() + o_uoff, uoff.data(), ni * sizeof(int64_t));
    memcpy(blob.data() + o_oinst, oinst.data(), oinst.size() * 4);
    memcpy(blob.data() + o_uinst, uinst.data(), uinst.size() * 4);
    a.amps = au.at<double2>(o_amps);
    a.uinst = au.at<int32_t>(o_uinst);
    a.uoff = au.at<int64_t>(o_uoff);
    a.oinst = au.at<int32_t>(o_oinst);
    e = hipMemcpyAsync(au.base, blob.data(), u_bytes, hipMemcpyHostToDevice, st);
    for (int64_t g0 = 0; g0 < n_gamma && e == hipSuccess && !ke; g0 += gc) {
        a.g0 = g0;
        a.gc = (int32_t)std::min<int64_t>(gc, n_gamma - g0);
        size_t first = 0;  // first entry of oinst that still has units
        for (int64_t u0 = 0; u0 < (int64_t)uinst.size() && !ke; u0 += units_max) {
            a.u0 = u0;
            a.ucount = std::min<int64_t>(units_max, (int64_t)uinst.size() - u0);
            while (uoff[oinst[first]] + stat[3 * (size_t)oinst[first] + 2] <= u0) first++;
            size_t last = first;
            while (last < oinst.size() && uoff[oinst[last]] < u0 + a.ucount) last++;
            a.o0 = (uint32_t)first;
            ke = launch_scan_points(a, (int)(last - first), lds, st);
        }
    }
    std::vector<double> tmp;
    const bool whole = ni == (int)done.size() && oinst.size() == (size_t)ni && idx.back() == ni - 1;
    double *oe = energy_out, *op = pgs_out;
    if (!whole) {
        tmp.resize(2 * nout);
        oe = tmp.data();
        op = tmp.data() + nout;
    }
    if (e == hipSuccess && !ke) e = hipMemcpyAsync(oe, a.out_e, nout * sizeof(double), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && !ke) e = hipMemcpyAsync(op, a.out_p, nout * sizeof(double), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && !ke) e = hipStreamSynchronize(st);
    if (ke || e != hipSuccess)
        return fail(SV_ERR_HIP, "sv_batch_p1_scan: %s", hipGetErrorString(ke ? (hipError_t)ke : e));
    if (!whole)
        for (int k = 0; k < ni; k++) {
            if (!done[k]) continue;
            memcpy(energy_out + (size_t)idx[k] * pts, oe + (size_t)k * pts, pts * sizeof(double));
            memcpy(pgs_out + (size_t)idx[k] * pts, op + (size_t)k * pts, pts * sizeof(double));
        }
    return SV_OK;
}

extern "C" int sv_batch_p1_scan(int n_inst, const sv_ising* insts, int n_gamma, const double* gammas, int n_beta,
                                const double* betas, sv_dtype dtype, void* stream, double* energy_out,
                                double* pgs_out) {
    if (n_inst < 1 || !insts) return fail(SV_ERR_ARG, "sv_batch_p1_scan: no instances");
    if (n_gamma < 1 || n_beta < 1 || !gammas || !betas) return fail(SV_ERR_ARG, "sv_batch_p1_scan: empty grid");
    if (!energy_out || !pgs_out) return fail(SV_ERR_ARG, "sv_batch_p1_scan: NULL output");
    if (!dtype_ok(dtype)) return fail(SV_ERR_ARG, "sv_batch_p1_scan: bad dtype");
    if ((int64_t)n_gamma * n_beta > (1 << 24)) return fail(SV_ERR_ARG, "sv_batch_p1_scan: grid too large");
    for (int a = 0; a < n_gamma; a++)
        if (!std::isfinite(gammas[a])) return fail(SV_ERR_NUMERIC, "sv_batch_p1_scan: gamma %d not finite", a);
    for (int b = 0; b < n_beta; b++)
        if (!std::isfinite(betas[b])) return fail(SV_ERR_NUMERIC, "sv_batch_p1_scan: beta %d not finite", b);
    const int S = batch_lds_bits(
        (int)dtype, dtype == SV_C64 ? knob_for("batchwide", (int)dtype, 0) : knob_for("batch128", (int)dtype, 0));
    const int nmax_batch = S + 5;  // direct scan: the high bits of a state fit one thread's 32 registers
    for (int i = 0; i < n_inst; i++) {
        if (!insts[i]) return fail(SV_ERR_ARG, "sv_batch_p1_scan: instance %d is NULL", i);
        if (insts[i]->n > nmax_batch)
            return fail(SV_ERR_UNSUPPORTED, "sv_batch_p1_scan: instance %d has n=%d > %d", i, insts[i]->n, nmax_batch);
    }
    const size_t pts = (size_t)n_gamma * n_beta;
    std::vector<int> grid, rest;
    const bool spheres = knob_for("batchsphere", (int)dtype, 0) != 0;
    for (int i = 0; i < n_inst; i++) (spheres && scan_by_spheres(insts[i]) ? grid : rest).push_back(i);
    const size_t step = scan_instances(n_gamma);
    for (size_t k0 = 0; k0 < grid.size(); k0 += step) {
        const std::vector<int> part(grid.begin() + k0, grid.begin() + std::min(k0 + step, grid.size()));
        std::vector<char> done(part.size(), 0);
        hipEvent_t ev0;
        const bool prof = prof_begin((hipStream_t)stream, &ev0);
        const int rc = sphere_scan(part, insts, n_gamma, gammas, n_beta, betas, (hipStream_t)stream, energy_out, pgs_out,
                                   done);
        if (prof) prof_end((hipStream_t)stream, ev0, std::string("batch_") + (dtype == SV_C128 ? "c128" : "c64"), 0.0);
        if (rc) return rc;
        for (size_t k = 0; k < part.size(); k++)
            if (!done[k]) rest.push_back(part[k]);
    }
    if (rest.empty()) return SV_OK;
    if ((int)rest.size() == n_inst)
        return direct_scan(n_inst, insts, n_gamma, gammas, n_beta, betas, dtype, stream, energy_out, pgs_out);
    std::vector<sv_ising> sub;
    for (int i : rest) sub.push_back(insts[i]);
    std::vector<double> en(sub.size() * pts), pg(sub.size() * pts);
    const int rc = direct_scan((int)sub.size(), sub.data(), n_gamma, gammas, n_beta, betas, dtype, stream, en.data(),
                               pg.data());
    if (rc) return rc;
    for (size_t k = 0; k < rest.size(); k++) {
        memcpy(energy_out + (size_t)rest[k] * pts, en.data() + k * pts, pts * sizeof(double));
        memcpy(pgs_out + (size_t)rest[k] * pts, pg.data() + k * pts, pts * sizeof(double));
    }
    return SV_OK;
}
