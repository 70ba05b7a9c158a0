// C ABI of the barotropic subcycle library: argument validation, mesh and
// plan management, and the launch sequences of the forward paths.
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstring>
#include <initializer_list>
#include <string>

#include "consumers.h"
#include "ensemble.h"
#include "kernels.h"
#include "se_internal.h"

namespace sesub {

namespace {
thread_local std::string g_err;
}

void set_error(const std::string &msg) { g_err = msg; }

DevBuf::~DevBuf() {
    if (p) (void)hipFree(p);
}

se_status DevBuf::alloc(size_t bytes) {
    if (p) {
        (void)hipFree(p);
        p = nullptr;
        n = 0;
    }
    if (bytes == 0) return SE_OK;
    if (hipMalloc(&p, bytes) != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
        set_error("device allocation of " + std::to_string(bytes) + " bytes failed");
        return SE_ERR_OOM;
    }
    n = bytes;
    return SE_OK;
}

se_status DevBuf::upload(const void *src, size_t bytes) {
    se_status s = alloc(bytes);
    if (s != SE_OK || bytes == 0) return s;
    if (hipMemcpy(p, src, bytes, hipMemcpyHostToDevice) != hipSuccess) {
        set_error("host to device copy failed");
        return SE_ERR_HIP;
    }
    return SE_OK;
}

namespace {

struct DeviceGuard {
    int prev = -1;
    bool ok = true;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) ok = hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceGuard() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

se_status hip_fail(hipError_t e, const char *where) {
    set_error(std::string(where) + ": " + hipGetErrorString(e));
    return SE_ERR_HIP;
}

#define SE_TRY(x)                         \
    do {                                  \
        se_status _s = (x);               \
        if (_s != SE_OK) return _s;       \
    } while (0)

#define HIP_TRY(x, where)                         \
    do {                                          \
        hipError_t _e = (x);                      \
        if (_e != hipSuccess) return hip_fail(_e, where); \
    } while (0)

constexpr size_t kAlign = 256;
inline size_t al(size_t b) { return (b + kAlign - 1) & ~(kAlign - 1); }

constexpr int kEpts[] = {1, 2, 3, 4, 6, 8};

int pick_ept(int need) {
    for (int e : kEpts)
        if (e >= need) return e;
    return -1;
}

// Geometry of a triangle set as 5 SoA arrays (gbx gby gcx gcy Ae).
template <typename T>
std::vector<T> pack_geom(const HostMesh &m, const std::vector<int32_t> *sel, int64_t off) {
    const int64_t n = sel ? static_cast<int64_t>(sel->size()) : m.ne;
    std::vector<T> g(5 * n);
    for (int64_t i = 0; i < n; ++i) {
        const int64_t e = sel ? (*sel)[i] - off : i;
        const double *gn = &m.gN[6 * e];
        g[i] = static_cast<T>(gn[2]);
        g[n + i] = static_cast<T>(gn[3]);
        g[2 * n + i] = static_cast<T>(gn[4]);
        g[3 * n + i] = static_cast<T>(gn[5]);
        g[4 * n + i] = static_cast<T>(m.Ae[e]);
    }
    return g;
}

// Register tiers that compile without scratch spills (triangles per thread).
bool ept_ok(bool f32, int ept, int block, bool sm = false) {
    if (ept < 0) return false;
    if (block == 256) return f32 ? ept <= 8 : ept <= 6;
    if (block == 512) return f32 ? ept <= 8 : ept <= 4;
    // 1024 threads: at most 128 VGPRs (the AB3-AM4 form holds two more transports)
    return f32 ? ept <= (sm ? 3 : 4) : ept <= (sm ? 1 : 3);
}

// Host-side construction and statistics of a plan (no device memory).
se_status plan_host(const std::vector<const HostMesh *> &members, const std::vector<int64_t> &voff,
                    const std::vector<int64_t> &eoff, int32_t T, int32_t K, int32_t block,
                    HostTiles &ht, se_plan_stats_t &st) {
    if (T < 64 || T > 8192 || K < 1 || K > 8 || (block != 256 && block != 512 && block != 1024)) {
        set_error("se_set_plan: tile in [64, 8192], k_fused in [1, 8], block 256, 512 or 1024");
        return SE_ERR_ARG;
    }
    SE_TRY(build_tiles(members, voff, eoff, T, K, ht));
    // a few tiles with more local triangles than the rest (a long coast, a fold of the
    // curve) set the register tier of all: when at most one tile in 50 exceeds the tier
    // below, those tiles are halved instead
    {
        const int e0 = pick_ept((ht.max_ne + block - 1) / block);
        int lower = 0;
        for (int e : kEpts)
            if (e < e0) lower = e;
        if (e0 > 0 && lower > 0) {
            const int32_t cap = lower * block;
            const size_t nt = ht.hdr.size();
            size_t over = 0;
            for (size_t t = 0; t < nt; ++t) over += ht.nE[t * (K + 1) + K] > cap;
            if (over > 0 && over * 50 <= nt) {
                HostTiles hs;
                SE_TRY(build_tiles(members, voff, eoff, T, K, hs, cap));
                // the workspace holds volume partials of one tile per 64 vertices of a member
                // (whatever the plan): halves beyond that, which tiles near 64 vertices
                // can give, would write past it
                std::vector<int64_t> cnt(members.size(), 0);
                for (const TileHdr &h : hs.hdr) ++cnt[h.member];
                bool fits = hs.max_ne <= cap;
                for (size_t i = 0; i < members.size(); ++i)
                    fits = fits && cnt[i] <= (members[i]->nv + 63) / 64;
                if (fits) ht = std::move(hs);
            }
        }
    }
    st = se_plan_stats_t{};
    const int ept = pick_ept((ht.max_ne + block - 1) / block);
    st.ntiles = static_cast<int32_t>(ht.hdr.size());
    st.max_tri = ht.max_ne;
    st.max_vtx = ht.max_nv;
    st.tri_per_thread = ept;
    st.lds_f32 = tile_lds_bytes(true, false, block, K, ht.max_nv, ht.max_ne, ht.max_nvu, ht.max_cs);
    st.lds_f64 = tile_lds_bytes(false, false, block, K, ht.max_nv, ht.max_ne, ht.max_nvu, ht.max_cs);
    // owned triangles must fit the slots that carry running sums
    const bool own_ok = ept > 0 && ht.max_nown <= own_slots(ept) * block;
    st.ok_f32 = own_ok && ept_ok(true, ept, block) && st.lds_f32 <= 160 * 1024;
    st.ok_f64 = own_ok && ept_ok(false, ept, block) && st.lds_f64 <= 160 * 1024;
    st.lds_sesm_f32 = tile_lds_bytes(true, true, block, K, ht.max_nv, ht.max_ne, ht.max_nvu,
                                     ht.max_cs);
    st.lds_sesm_f64 = tile_lds_bytes(false, true, block, K, ht.max_nv, ht.max_ne, ht.max_nvu,
                                     ht.max_cs);
    st.ok_sesm_f32 = own_ok && ept_ok(true, ept, block, true) && st.lds_sesm_f32 <= 160 * 1024;
    st.ok_sesm_f64 = own_ok && ept_ok(false, ept, block, true) && st.lds_sesm_f64 <= 160 * 1024;
    int64_t nv = 0, ne = 0;
    for (const HostMesh *m : members) {
        nv += m->nv;
        ne += m->ne;
    }
    // compulsory bytes of one launch (all tiles), per precision s
    int64_t sumV = 0, sumVu = 0, sumE = 0, sumC = 0;
    for (size_t t = 0; t < ht.hdr.size(); ++t) {
        sumV += ht.nV[t * (K + 1) + K];
        sumVu += ht.nV[t * (K + 1) + K - 1];
        sumE += ht.nE[t * (K + 1) + K];
    }
    sumC = ht.n_ent;
    st.tri_overhead = static_cast<double>(sumE) / ne;
    st.vtx_overhead = static_cast<double>(sumV) / nv;
    for (int f = 0; f < 2; ++f) {
        const double s = f == 0 ? 4.0 : 8.0;
        const double bytes = sumV * (4 + 2 * s) + sumVu * (s + 2) + sumC * 0.0 +
                             sumE * (ht.ell ? 8 : 12) + (sumE - ne) * 4 +
                             sumE * (5 * s + 2 * s + 2 * s + s) +
                             ne * (32.0 + 2 * s) + nv * (s + 8.0);
        (f == 0 ? st.bytes_per_vs_f32 : st.bytes_per_vs_f64) = bytes / (static_cast<double>(nv) * K);
    }
    return SE_OK;
}

// The reverse tile kernel has a variant for a plan of these sizes: up to four triangles per
// thread, with 1024-thread workgroups three in FP32 and two in FP64; a tile's owned vertices
// within two per thread; its LDS within 160 KiB.
bool adj_fits(bool f32, int32_t max_nv, int32_t max_nvu, int32_t max_cs, int32_t T, int32_t K,
              int32_t block, int32_t ept) {
    return ept >= 1 && ept <= (block < 1024 ? 4 : f32 ? 3 : 2) && T <= 2 * block &&
           adj_tile_lds_bytes(f32, block, K, max_nv, max_nvu, max_cs) <= 160 * 1024;
}

// Upload a tile plan built by plan_host (ht is used up).  Values go up for the precisions in
// precs alone (bit 0: FP64, bit 1: FP32); the plan does not run in the other.
se_status upload_plan(const std::vector<const HostMesh *> &members, const std::vector<int64_t> &voff,
                      const std::vector<int64_t> &eoff, int32_t T, int32_t K, int32_t block,
                      HostTiles &ht, const se_plan_stats_t &st, int precs,
                      std::unique_ptr<DevTiles> &out) {
    const bool with64 = precs & 1, with32 = precs & 2;
    const int ept = st.tri_per_thread;
    if (!st.ok_f32 && !st.ok_f64) {
        set_error("se_set_plan: tile too large for the register or LDS budget (reduce tile or "
                  "k_fused)");
        return SE_ERR_ARG;
    }
    // tables at a fixed stride per tile, the rest of each tile's entries copies of its last
    // one (valid ids and indices, never used); odd multiples of 16 entries, so that tiles
    // loading in step start on different memory channels
    const int32_t se = ((ht.max_ne + 15) & ~15) | 16, sv = ((ht.max_nv + 15) & ~15) | 16;
    const size_t nt = ht.hdr.size();
    {
        std::vector<int32_t> le(nt * se), lv(nt * sv);
        std::vector<uint32_t> lt(3 * nt * se), lr(ht.ell ? 2 * nt * se : 0);
        for (size_t t = 0; t < nt; ++t) {
            const TileHdr &h = ht.hdr[t];
            const int32_t n = h.nE[K], nl = h.nV[K];
            for (int32_t i = 0; i < se; ++i) {
                const size_t s = h.le_off + std::min(i, n - 1), d = t * se + i;
                le[d] = ht.le_gid[s];
                for (int q = 0; q < 3; ++q) lt[3 * d + q] = ht.le_tri[3 * s + q];
                if (ht.ell)
                    for (int q = 0; q < 2; ++q) lr[2 * d + q] = ht.le_rank[2 * s + q];
            }
            for (int32_t i = 0; i < sv; ++i) lv[t * sv + i] = ht.lv_gid[h.lv_off + std::min(i, nl - 1)];
        }
        ht.le_gid.swap(le);
        ht.lv_gid.swap(lv);
        ht.le_tri.swap(lt);
        ht.le_rank.swap(lr);
    }
    auto p = std::make_unique<DevTiles>();
    p->se = se;
    p->sv = sv;
    p->T = T;
    p->K = K;
    p->block = block;
    p->ept = ept;
    p->ntiles = static_cast<int32_t>(ht.hdr.size());
    p->max_nv = ht.max_nv;
    p->max_ne = ht.max_ne;
    p->max_nvu = ht.max_nvu;
    p->max_cs = ht.max_cs;
    p->ell = ht.ell;
    p->lds_bytes64 = st.lds_f64;
    p->lds_bytes32 = st.lds_f32;
    p->ok32 = st.ok_f32 && with32;
    p->ok64 = st.ok_f64 && with64;
    p->lds_sm32 = st.lds_sesm_f32;
    p->lds_sm64 = st.lds_sesm_f64;
    p->ok_sm32 = st.ok_sesm_f32 && with32;
    p->ok_sm64 = st.ok_sesm_f64 && with64;
    p->hdr_host = ht.hdr;
    p->le_gid_host = ht.le_gid;
    p->nE_host = ht.nE;
    static_assert(sizeof(TileHdr) == sizeof(TileHdrK), "tile header layouts differ");
    SE_TRY(p->hdr.upload(ht.hdr.data(), ht.hdr.size() * sizeof(TileHdr)));
    SE_TRY(p->lv_gid.upload(ht.lv_gid.data(), ht.lv_gid.size() * 4));
    const int64_t nle = static_cast<int64_t>(ht.le_gid.size());
    SE_TRY(p->le_gid.upload(ht.le_gid.data(), ht.le_gid.size() * 4));
    if (ht.ell) {
        SE_TRY(p->le_rec.upload(ht.le_rank.data(), ht.le_rank.size() * 4));
    } else {
        std::vector<uint32_t> rec(2 * nle), pos(nle);
        for (int64_t i = 0; i < nle; ++i) {
            for (int k = 0; k < 2; ++k) rec[2 * i + k] = ht.le_tri[3 * i + k];
            pos[i] = ht.le_tri[3 * i + 2];
        }
        SE_TRY(p->le_rec.upload(rec.data(), rec.size() * 4));
        SE_TRY(p->le_pos.upload(pos.data(), pos.size() * 4));
    }
    SE_TRY(p->cs_row.upload(ht.cs_row.data(), ht.cs_row.size() * 2));
    // local geometry per tile, gathered member by member
    std::vector<double> g64(with64 ? 4 * nle : 0), a64e(with64 ? nle : 0);
    std::vector<float> g32(with32 ? 4 * nle : 0), a32e(with32 ? nle : 0);
    for (int64_t i = 0; i < nle; ++i) {
        const int64_t ge = ht.le_gid[i];
        size_t mi = std::upper_bound(eoff.begin(), eoff.end(), ge) - eoff.begin() - 1;
        const HostMesh &m = *members[mi];
        const int64_t e = ge - eoff[mi];
        const double *gn = &m.gN[6 * e];
        if (with64) {
            for (int q = 0; q < 4; ++q) g64[4 * i + q] = gn[2 + q];
            a64e[i] = m.Ae[e];
        }
        if (with32) {
            for (int q = 0; q < 4; ++q) g32[4 * i + q] = static_cast<float>(gn[2 + q]);
            a32e[i] = static_cast<float>(m.Ae[e]);
        }
    }
    SE_TRY(p->geo64.upload(g64.data(), g64.size() * 8));
    SE_TRY(p->geo32.upload(g32.data(), g32.size() * 4));
    SE_TRY(p->ae64.upload(a64e.data(), a64e.size() * 8));
    SE_TRY(p->ae32.upload(a32e.data(), a32e.size() * 4));
    // reciprocal dual-cell areas per local vertex (contiguous per tile: no index round
    // trip); FP32: of the FP32-rounded area, rounded once
    const int64_t nlv = static_cast<int64_t>(ht.lv_gid.size());
    std::vector<double> a64(with64 ? nlv : 0);
    std::vector<float> a32(with32 ? nlv : 0);
    for (int64_t i = 0; i < nlv; ++i) {
        const int64_t gv = ht.lv_gid[i];
        size_t mi = std::upper_bound(voff.begin(), voff.end(), gv) - voff.begin() - 1;
        const double av = members[mi]->Av[gv - voff[mi]];
        if (with64) a64[i] = 1.0 / av;
        if (with32) a32[i] = 1.0f / static_cast<float>(av);
    }
    SE_TRY(p->lav64.upload(a64.data(), a64.size() * 8));
    SE_TRY(p->lav32.upload(a32.data(), a32.size() * 4));
    // raise the LDS limit of the forward-backward tile kernels this plan runs now, so
    // that a later launch needs no attribute call (the adjoint may be graph-captured)
    for (int f = 0; f < 2; ++f)
        p->prepared[f] = p->ok(f == 1, false) && prepare_tile(f == 1, 0, p->ept, p->block) == hipSuccess;
    // the adjoint on the plan: recompute with trajectory output (mode 3) and the reverse
    // tile kernel
    for (int f = 0; f < 2; ++f) {
        const bool f32 = f == 1;
        p->lds_adj[f] = static_cast<size_t>(adj_tile_lds_bytes(f32, block, K, p->max_nv,
                                                               p->max_nvu, p->max_cs));
        p->adj_ready[f] = p->prepared[f] &&
                          adj_fits(f32, p->max_nv, p->max_nvu, p->max_cs, T, K, block, ept) &&
                          prepare_tile(f32, 3, ept, block) == hipSuccess &&
                          prepare_adj_tile(f32, ept, block) == hipSuccess;
    }
    out = std::move(p);
    return SE_OK;
}

// Build and upload a tile plan for a set of meshes forming a disjoint union.
se_status make_plan(const std::vector<const HostMesh *> &members, const std::vector<int64_t> &voff,
                    const std::vector<int64_t> &eoff, int32_t T, int32_t K, int32_t block,
                    std::unique_ptr<DevTiles> &out) {
    HostTiles ht;
    se_plan_stats_t st;
    SE_TRY(plan_host(members, voff, eoff, T, K, block, ht, st));
    return upload_plan(members, voff, eoff, T, K, block, ht, st, 3, out);
}

// LDS of the viscous form of a plan whose forward-backward form takes lds bytes: the
// velocities u = U / H_e of the tile's triangles and their edge-neighbour ids besides.
size_t visc_lds(size_t lds, bool f32, int32_t max_ne) {
    const size_t n = static_cast<size_t>(max_ne);
    return ((lds + 2 * (f32 ? 4 : 8) * n + 15) & ~static_cast<size_t>(15)) + 8 * n;
}
// Register budget of the viscous form (no spills): 1024-thread workgroups up to three
// triangles per thread (FP32; FP64 one), 512-thread ones up to six (FP32) or four (FP64).
bool visc_regs_ok(bool f32, int block, int ept) {
    return block == 1024 ? ept <= (f32 ? 3 : 1) : block == 512 ? ept <= (f32 ? 6 : 4) : true;
}

struct Layout {
    size_t eta_alt, U_alt, sum, U0c, phi, vol, total;
    size_t vub, vRb, vRe;  // viscous term: U / H_e, R - V^0, R - V^0 + V^m
    size_t sv[8], se[7];   // AB3-AM4 only: 8 vertex arrays, 7 triangle (transport) arrays
};

Layout fwd_layout(int64_t nv, int64_t ne, bool f32, int32_t nsub, int64_t width,
                  bool sesm = false, bool visc = false) {
    const size_t s = f32 ? 4 : 8;
    Layout L{};
    size_t o = 0;
    if (sesm) {
        for (int k = 0; k < 8; ++k) {
            L.sv[k] = o;
            o += al(nv * s);
        }
        for (int k = 0; k < 7; ++k) {
            L.se[k] = o;
            o += al(2 * ne * s);
        }
    }
    L.eta_alt = o;
    o += al(nv * s);
    L.U_alt = o;
    o += al(2 * ne * s);
    L.sum = o;
    o += al(16 * ne);
    L.U0c = o;
    o += al(2 * ne * s);
    L.phi = o;
    o += al(3 * ne * s);
    L.vol = o;
    o += al(static_cast<size_t>(nsub + 1) * width * 8);
    if (visc) {
        L.vub = o;
        o += al(2 * ne * s);
        L.vRb = o;
        o += al(2 * ne * s);
        L.vRe = o;
        o += al(2 * ne * s);
    }
    L.total = o;
    return L;
}

struct AdjLayout {
    size_t ckpt, traj[2], lam_eta, lam_U, psi, gR, gH0, total;
    size_t etraj, lam_eta2, lam_U2;   // tile reverse sweep: forward elevations (two
                                      // segments), second adjoint state
    int32_t nseg, k;
};

AdjLayout adj_layout(int64_t nv, int64_t ne, bool f32, int32_t nsub, int32_t k, size_t base) {
    const size_t s = f32 ? 4 : 8;
    const size_t st = al((nv + 2 * ne) * s);   // one state (eta then U)
    AdjLayout L{};
    L.k = k;
    L.nseg = (nsub + k - 1) / k;
    size_t o = base;
    L.ckpt = o;
    o += st * L.nseg;
    // two segment buffers: the reverse sweep of one segment reads one while the
    // recompute of the previous segment writes the other
    L.traj[0] = o;
    o += st * k;
    L.traj[1] = o;
    o += st * k;
    L.lam_eta = o;
    o += al(nv * s);
    L.lam_U = o;
    o += al(2 * ne * s);
    L.psi = o;
    o += al(4 * ne * s);
    L.gR = o;
    o += al(2 * ne * s);
    L.gH0 = o;
    o += al(nv * s);
    // the tile reverse sweep: elevations of one segment's substeps (slot m at m nv), the
    // second buffer of the adjoint state (launches alternate between the two)
    L.etraj = o;
    o += 2 * al(static_cast<size_t>(k) * nv * s);
    L.lam_eta2 = o;
    o += al(nv * s);
    L.lam_U2 = o;
    o += al(2 * ne * s);
    L.total = o;
    return L;
}

int64_t vol_width(int64_t nv) { return std::max<int64_t>((nv + 63) / 64, (nv + 255) / 256); }

// Largest |lambda| among the roots of the SESM characteristic polynomial of
// eq. (eqdp_1) at CFL number c (Durand-Kerner iteration on the monic degree-6
// polynomial; the printed '+-' of its lambda^2 term read as '-').
double sesm_max_root(double c, double b, double d, double g, double z) {
    const double c2 = c * c;
    const double co[7] = {
        b * z * c2,
        c2 * (b * (g - 2 * z) - z / 2),
        -c2 * ((d + 3 * g - 1) * b + g / 2 - 1.5 * z),
        c2 / 2 * (b * (6 * d + 6 * g + 4 * z - 4) + d + 4 * g + z - 1),
        1 + c2 / 2 * (b * (-6 * d - 2 * g - 2 * z + 2) - 4 * d - 3 * g - 3 * z + 3),
        -2 + c2 * d / 2 * (2 * b + 3),
        1.0};
    using cd = std::complex<double>;
    auto P = [&](cd x) {
        cd r = co[6];
        for (int k = 5; k >= 0; --k) r = r * x + co[k];
        return r;
    };
    cd rt[6];
    for (int k = 0; k < 6; ++k) rt[k] = std::pow(cd(0.4, 0.9), k);
    for (int it = 0; it < 500; ++it) {
        double delta = 0.0;
        for (int k = 0; k < 6; ++k) {
            cd den = 1.0;
            for (int j = 0; j < 6; ++j)
                if (j != k) den *= rt[k] - rt[j];
            const cd step = P(rt[k]) / den;
            rt[k] -= step;
            delta = std::max(delta, std::abs(step));
        }
        if (delta < 1e-14) break;
    }
    double mx = 0.0;
    for (int k = 0; k < 6; ++k) mx = std::max(mx, std::abs(rt[k]));
    return mx;
}

// Whether every CFL number in (0, c] is stable for the SESM coefficients.
bool sesm_stable_upto(double c, double b, double d, double g, double z) {
    const int n = 400;
    for (int i = 1; i <= n; ++i)
        if (sesm_max_root(c * i / n, b, d, g, z) > 1.0 + 1e-9) return false;
    return true;
}

inline bool visc_on(const se_params *p) { return p->visc_A0 > 0.0 || p->visc_Cv > 0.0; }

se_status check_params(const se_mesh *m, const se_params *p, int32_t nsub, double dt) {
    if (!m || !p) {
        set_error("null mesh or params");
        return SE_ERR_ARG;
    }
    if (p->precision != SE_F64 && p->precision != SE_F32_MIXED) {
        set_error("unknown precision");
        return SE_ERR_ARG;
    }
    if (nsub < 1 || !(dt > 0.0) || !std::isfinite(dt)) {
        set_error("need nsub >= 1 and a finite dt > 0");
        return SE_ERR_ARG;
    }
    if (!(p->g > 0.0) || !std::isfinite(p->g) || !(p->theta >= 0.0) || !std::isfinite(p->theta) ||
        !std::isfinite(p->eta_ref)) {
        set_error("need g > 0, theta >= 0 and a finite eta_ref");
        return SE_ERR_ARG;
    }
    if (p->scheme != SE_SCHEME_SE && p->scheme != SE_SCHEME_SESM) {
        set_error("unknown scheme");
        return SE_ERR_ARG;
    }
    if (p->reserved != 0) {
        set_error("se_params.reserved must be 0");
        return SE_ERR_ARG;
    }
    if (!(p->visc_A0 >= 0.0) || !std::isfinite(p->visc_A0) || !(p->visc_Cv >= 0.0) ||
        !std::isfinite(p->visc_Cv)) {
        set_error("visc_A0 and visc_Cv must be finite and >= 0");
        return SE_ERR_ARG;
    }
    const bool sesm = p->scheme == SE_SCHEME_SESM;
    if (sesm && !(std::isfinite(p->beta) && std::isfinite(p->delta) && std::isfinite(p->gamma) &&
                  std::isfinite(p->zeta))) {
        set_error("SESM coefficients must be finite");
        return SE_ERR_ARG;
    }
    if (p->flags & SE_CHECK_CFL) {
        if (!(p->h_max > 0.0)) {
            set_error("SE_CHECK_CFL needs h_max > 0");
            return SE_ERR_ARG;
        }
        const double dts = dt / nsub;
        const double c = dts * std::sqrt(p->g * p->h_max * m->h.mu_max);
        if (sesm) {
            if (!sesm_stable_upto(c, p->beta, p->delta, p->gamma, p->zeta)) {
                set_error("CFL: dt_s sqrt(g h_max mu_max) = " + std::to_string(c) +
                          " is beyond the stability range of the SESM coefficients");
                return SE_ERR_CFL;
            }
        } else {
            const double lim = 2.0 / std::sqrt(1.0 + 2.0 * p->theta);
            if (c > lim) {
                set_error("CFL: dt_s sqrt(g h_max mu_max) = " + std::to_string(c) +
                          " exceeds the stability bound " + std::to_string(lim));
                return SE_ERR_CFL;
            }
        }
    }
    return SE_OK;
}

StepC make_step(const se_params *p, int32_t nsub, double dt) {
    StepC c{};
    c.dts = dt / nsub;
    c.g = p->g;
    c.theta = p->theta;
    c.opt = 1.0 + p->theta;
    c.thM = p->theta / static_cast<double>(nsub);
    c.Mdbl = static_cast<double>(nsub);
    c.eta_ref = p->eta_ref;
    c.dts_f = static_cast<float>(c.dts);
    c.g_f = static_cast<float>(c.g);
    c.theta_f = static_cast<float>(c.theta);
    c.opt_f = static_cast<float>(c.opt);
    c.eta_ref_f = static_cast<float>(c.eta_ref);
    c.nsub = nsub;
    c.flags = ((p->flags & SE_LINEAR_H) ? KF_LINEAR_H : 0) |
              ((p->flags & SE_TRACK_VOLUME) ? KF_TRACK_VOLUME : 0);
    if (p->scheme == SE_SCHEME_SESM) {   // eq. (eq4_7)
        c.ab0 = 1.5 + p->beta;
        c.ab1 = 0.5 + 2.0 * p->beta;
        c.ab2 = p->beta;
        c.am0 = p->delta;
        c.am1 = 1.0 - p->delta - p->gamma - p->zeta;
        c.am2 = p->gamma;
        c.am3 = p->zeta;
        c.ab0_f = static_cast<float>(c.ab0);
        c.ab1_f = static_cast<float>(c.ab1);
        c.ab2_f = static_cast<float>(c.ab2);
        c.am0_f = static_cast<float>(c.am0);
        c.am1_f = static_cast<float>(c.am1);
        c.am2_f = static_cast<float>(c.am2);
        c.am3_f = static_cast<float>(c.am3);
    }
    return c;
}

se_status check_device(const se_mesh *m) {
    if (m->device < 0) {
        set_error("host-only mesh (created with device < 0) cannot run kernels");
        return SE_ERR_ARG;
    }
    return SE_OK;
}

// Forms of the subcycle that a default plan is chosen for.
// + 1: FP32; ANY: every form, ANY + 1: every form but the viscous one
enum : int { CL_FB = 0, CL_SESM = 2, CL_VISC = 4, CL_ADJ = 6, CL_ANY = 8 };

bool plan_fits(int cl, const HostTiles &ht, const se_plan_stats_t &st, int32_t K, int32_t block) {
    const bool f32 = cl & 1;
    switch (cl & ~1) {
        case CL_FB: return f32 ? st.ok_f32 : st.ok_f64;
        case CL_SESM: return f32 ? st.ok_sesm_f32 : st.ok_sesm_f64;
        case CL_VISC:
            return (f32 ? st.ok_f32 : st.ok_f64) && K >= 2 &&
                   visc_lds(f32 ? st.lds_f32 : st.lds_f64, f32, ht.max_ne) <= 160 * 1024 &&
                   visc_regs_ok(f32, block, st.tri_per_thread);
        case CL_ADJ:
            return (f32 ? st.ok_f32 : st.ok_f64) &&
                   adj_fits(f32, ht.max_nv, ht.max_nvu, ht.max_cs, ht.T, K, block, st.tri_per_thread);
        default:
            return st.ok_f32 && st.ok_f64 && st.ok_sesm_f32 && st.ok_sesm_f64 &&
                   (cl != CL_ANY || (plan_fits(CL_VISC, ht, st, K, block) &&
                                     plan_fits(CL_VISC + 1, ht, st, K, block)));
    }
}

// The viscous form of this precision runs on a plan.
bool visc_fits(const DevTiles &P, bool f32) {
    return P.ok(f32, false) && P.K >= 2 &&
           visc_lds(P.lds(f32, false), f32, P.max_ne) <= 160 * 1024 &&
           visc_regs_ok(f32, P.block, P.ept);
}

// A candidate of a form's default plan: at most ept triangles per thread, and ntiles
// tiles (0: any number).
struct PlanCand {
    int32_t T, K, block, ept, ntiles;
};

// Candidates of a form's default plan, best first, from the mesh size alone.
//
// A launch costs its dependent round trips and its substeps' barriers whatever the tile
// holds, so a mesh of up to about 200,000 vertices runs fastest as one tile per CU (256 of
// them, or tiles of 64 vertices where that leaves CUs idle), with as many rings as the
// register tier takes: fewer launches beat the larger halo.  Two 512-thread workgroups on
// a CU hold what one of 1024 threads does; the larger one has less halo and, alone, loads
// faster.  Beyond, FP64 keeps 1024-thread tiles of at most 776 vertices in whole rounds of
// 256, and FP32 from about 400,000 vertices (both precisions from 700,000) the two-per-CU
// tiles whose loads overlap the other's substeps.  Each line is the fastest, or within 3%
// of it, of 20 to 130 plans timed per size (60 substeps, us; vertices: FP32, FP64):
//   forward-backward  2,048: 90, 91   31,439: 110, 119   69,721: 123, 141
//                     131,230: 158, 229   195,440: 214, 307   358,386: 381, 539
//                     550,482: 525, 852   979,989: 869, 1448
//   AB3-AM4           11,397: 116, 129   195,440: 275, 511   550,482: 674, 1512
//   viscous           11,397: 210, 241   195,440: 595, 1108   550,482: 1577, 3074
// The adjoint's (a gradient of 30 substeps, forward sweep included, us) has two triangles per
// thread in FP64, which is what its registers allow at 1024 threads:
//   2,048: 87, 94   65,536: 124, 154   104,000: 164, 238   202,500: 257, 460
//   490,000: 574, 1118
// and, without a plan of its own, ran the per-substep kernels wherever the forward plan was
// not one for its kernel: 104,000 vertices FP64 809, 490,000 650 and 3,377.
// One list for every mesh and form (512,4,512 on most) took e.g. 145 FP64 at 11,397
// vertices and 37 substeps (81 now), 1,140 viscous FP32 at 196,608 (611).
std::vector<PlanCand> default_plans(int cl, int64_t nv) {
    std::vector<PlanCand> c;
    // tiles of at most tmax vertices in whole rounds of 256, a little larger where the
    // halving of oversized tiles adds some beyond; rings ks, largest first
    auto rounds = [&](int32_t tmax, std::initializer_list<int32_t> ks, int32_t block, int32_t ept) {
        const int64_t m = std::max<int64_t>(1, (nv + 256 * static_cast<int64_t>(tmax) - 1) /
                                                   (256 * static_cast<int64_t>(tmax)));
        const int32_t T = static_cast<int32_t>(((nv + 256 * m - 1) / (256 * m) + 7) / 8 * 8);
        for (int32_t K : ks)
            for (int32_t d = 0; d <= 16; d += 8)
                c.push_back({std::max<int32_t>(64, T) + d, K, block, ept,
                             static_cast<int32_t>(256 * m)});
    };
    const bool tiny = nv <= 64 * 256;
    switch (cl) {
        case CL_FB + 1:
            if (tiny) c.push_back({64, 8, 512, 4, 0});
            else if (nv <= 288 * 256) rounds(288, {8, 6, 5}, 512, 4);
            if (nv <= 1024 * 256) rounds(1024, {8, 6, 5}, 1024, 4);
            else if (nv <= 400000) rounds(784, {8, 6, 5}, 1024, 4);
            if (nv <= 700000) c.push_back({384, 5, 512, 4, 0});
            c.push_back({512, 4, 512, 4, 0});
            c.push_back({448, 4, 512, 4, 0});
            break;
        case CL_FB:
            if (tiny) c.push_back({64, 6, 1024, 1, 0});
            if (nv <= 320 * 256) rounds(320, {8}, 1024, 2);
            if (nv <= 700000) rounds(776, {6, 5, 4}, 1024, 3);
            c.push_back({320, 4, 512, 3, 0});
            c.push_back({256, 4, 512, 3, 0});
            break;
        case CL_SESM + 1:
            if (tiny) c.push_back({64, 8, 512, 4, 0});
            else if (nv <= 800 * 256) rounds(800, {8, 6, 5}, 1024, 3);
            c.push_back({384, 5, 512, 4, 0});
            c.push_back({384, 4, 512, 4, 0});
            break;
        case CL_SESM:
            if (tiny) c.push_back({64, 8, 512, 4, 0});
            else if (nv <= 400000) rounds(392, {6, 5, 4}, 512, 4);
            c.push_back({384, 5, 512, 4, 0});
            c.push_back({384, 4, 512, 4, 0});
            break;
        case CL_VISC + 1:
            if (tiny) c.push_back({64, 8, 1024, 3, 0});
            else if (nv <= 700000) rounds(800, {8, 6, 4}, 1024, 3);
            c.push_back({352, 4, 512, 3, 0});
            c.push_back({320, 4, 512, 3, 0});
            break;
        case CL_VISC:
            if (tiny) c.push_back({64, 6, 1024, 1, 0});
            else if (nv <= 200 * 256) rounds(200, {4}, 1024, 1);
            if (nv <= 400000) rounds(392, {6, 4}, 512, 4);
            c.push_back({448, 4, 512, 4, 0});
            c.push_back({384, 4, 512, 4, 0});
            break;
        case CL_ADJ + 1:
            if (tiny) c.push_back({64, 6, 512, 2, 0});
            if (nv <= 288 * 256) rounds(288, {6}, 1024, 2);
            if (nv <= 480 * 256) rounds(480, {8, 6, 5}, 1024, 3);
            else if (nv <= 300000) rounds(800, {4, 3}, 1024, 3);
            c.push_back({416, 4, 512, 4, 0});
            c.push_back({256, 4, 512, 4, 0});
            c.push_back({128, 4, 512, 4, 0});
            break;
        case CL_ADJ:
            if (tiny) c.push_back({64, 6, 512, 2, 0});
            if (nv <= 288 * 256) rounds(288, {6, 5}, 1024, 2);
            if (nv <= 464 * 256) rounds(464, {4}, 1024, 2);
            else if (nv <= 528 * 256) rounds(528, {3}, 1024, 2);
            rounds(464, {4}, 1024, 2);
            c.push_back({416, 4, 1024, 2, 0});
            c.push_back({256, 4, 512, 4, 0});
            c.push_back({128, 4, 512, 4, 0});
            break;
        default: break;
    }
    return c;
}

// Plans that run every form without spills, largest tiles first: the one that a call that
// may not allocate falls back on (a mesh none of them runs the viscous form on, such as one
// of long rows, takes the first that runs the others).
const std::vector<PlanCand> kAnyPlans = {
    {1024, 4, 512, 8, 0}, {512, 4, 512, 8, 0}, {512, 4, 256, 8, 0}, {512, 2, 256, 8, 0},
    {256, 4, 256, 8, 0},  {256, 2, 256, 8, 0}, {128, 2, 256, 8, 0}, {64, 1, 256, 8, 0}};

// Build the first candidate that fits the form on this mesh, with the tables of the form's own
// precision (half of the memory and of the upload of both); of both where the plan is one for
// every form, or runs every form and any_ok is asked for.
se_status make_default(se_mesh *m, int cl, const std::vector<PlanCand> &cand,
                       std::unique_ptr<DevTiles> &out, bool *any_ok) {
    const std::vector<const HostMesh *> mem{&m->h};
    const std::vector<int64_t> vo{0, m->h.nv}, eo{0, m->h.ne};
    for (const auto &c : cand) {
        HostTiles ht;
        se_plan_stats_t st;
        // not worth building: the local triangles of a square tile and its rings, less the
        // tenth that a coast or the edge of the mesh takes off
        const double side = std::sqrt(static_cast<double>(c.T)) + 2.0 * c.K;
        if (c.T < m->h.nv && 0.9 * 2.0 * side * side > static_cast<double>(c.ept) * c.block) continue;
        if (plan_host(mem, vo, eo, c.T, c.K, c.block, ht, st) != SE_OK) continue;
        if (st.tri_per_thread < 1 || st.tri_per_thread > c.ept || (c.ntiles && st.ntiles > c.ntiles) ||
            !plan_fits(cl, ht, st, c.K, c.block))
            continue;
        if (any_ok) *any_ok = plan_fits(CL_ANY, ht, st, c.K, c.block);
        const int precs = cl >= CL_ANY || (any_ok && *any_ok) ? 3 : 1 << (cl & 1);
        return upload_plan(mem, vo, eo, c.T, c.K, c.block, ht, st, precs, out);
    }
    set_error("no default plan fits this mesh");
    return SE_ERR_ARG;
}

// The plan a call of form cl runs on: the caller's (se_set_plan), else the form's default,
// made at its first call, else (nothing may be allocated: se_subcycle_noalloc, or a stream
// under capture once some default exists) one that runs every form.  The first default of
// a mesh brings such a plan along, so a call that found a plan before still finds one.
// The fields do not depend on the plan, the volume to rounding.
se_status mesh_plan(se_mesh *m, int cl, bool may_alloc, hipStream_t s, DevTiles **out) {
    *out = nullptr;
    if (m->plan) {
        *out = m->plan.get();
        return SE_OK;
    }
    std::lock_guard<std::mutex> lk(m->plan_mu);
    if (m->dflt[cl]) {
        *out = m->dflt[cl].get();
        return SE_OK;
    }
    DevTiles *any = m->dflt[CL_ANY].get();
    if (any && may_alloc && s) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone)
            may_alloc = false;
    }
    if (!may_alloc) {
        *out = any;   // null: no plan yet
        return SE_OK;
    }
    if (m->no_own[cl]) {
        *out = (cl & ~1) == CL_ADJ ? nullptr : any;
        return SE_OK;
    }
    std::unique_ptr<DevTiles> p;
    bool any_ok = false;
    auto cand = default_plans(cl, m->h.nv);
    if ((cl & ~1) == CL_ADJ) {   // none fits: the forward plans are asked, now and later
        if (make_default(m, cl, cand, p, nullptr) == SE_OK) {
            m->dflt[cl] = std::move(p);
            *out = m->dflt[cl].get();
        } else {
            m->no_own[cl] = true;
        }
        return SE_OK;
    }
    cand.insert(cand.end(), kAnyPlans.begin(), kAnyPlans.end());
    const se_status own = make_default(m, cl, cand, p, any ? nullptr : &any_ok);
    if (!any && (own != SE_OK || !any_ok)) {
        // (a form whose own plan runs every form needs no second one)
        std::unique_ptr<DevTiles> a;
        auto make_any = [&] {
            return make_default(m, CL_ANY, kAnyPlans, a, nullptr) == SE_OK
                       ? SE_OK : make_default(m, CL_ANY + 1, kAnyPlans, a, nullptr);
        };
        if (make_any() != SE_OK) {   // no memory for both
            if (!p) return own;
            p.reset();
            SE_TRY(make_any());
        }
        m->dflt[CL_ANY] = std::move(a);
    }
    const DevTiles *first = p ? p.get() : m->dflt[CL_ANY].get();
    if (!any) {
        m->plan_T = first->T;
        m->plan_K = first->K;
        m->plan_block = first->block;
    }
    if (p) {
        m->dflt[cl] = std::move(p);
        if (!m->dflt[CL_ANY]) m->dflt[CL_ANY] = m->dflt[cl];
        *out = m->dflt[cl].get();
    } else {   // no memory for a plan of its own: the one for every form, now and later
        m->no_own[cl] = true;
        *out = m->dflt[CL_ANY].get();
    }
    return SE_OK;
}

}  // namespace
}  // namespace sesub

using namespace sesub;

static se_status ensure_visc(se_mesh *m);
static se_status ensure_tile_visc(const se_mesh *m, DevTiles &P);
static ViscArgs visc_args(const se_mesh *m, bool f32, const se_params *p, const void *H0,
                          const void *eta, const void *U, void *ubar);

extern "C" {

const char *se_last_error(void) { return g_err.c_str(); }

se_status se_sesm_coefficients(double theta, double beta, double *out) {
    if (!out || !std::isfinite(theta) || !std::isfinite(beta)) {
        set_error("se_sesm_coefficients: bad argument");
        return SE_ERR_ARG;
    }
    const double chi = 0.5 * theta;            // SE dissipation 2 chi = theta
    const double zeta = 0.010 - 0.135 * chi;    // eq. (eqdp_6), second line
    const double gamma = 0.083 - 0.514 * chi;
    out[0] = beta > 0.0 ? beta : 0.281105;      // largest stability range (Sec. 3.2)
    out[1] = 2.0 * chi + gamma + 2.0 * zeta + 0.5;   // eq. (eqdp_4)
    out[2] = gamma;
    out[3] = zeta;
    return SE_OK;
}

se_status se_mesh_create(const se_mesh_desc *desc, int device, se_mesh **out) {
    if (!desc || !out) {
        set_error("se_mesh_create: null argument");
        return SE_ERR_ARG;
    }
    *out = nullptr;
    auto m = std::make_unique<se_mesh>();
    m->device = device;
    SE_TRY(build_host_mesh(*desc, m->h));
    for (double v : m->h.Av) m->h.Av_total += v;
    if (device < 0) {   // host-only mesh: reordering and geometry, no device arrays
        *out = m.release();
        return SE_OK;
    }
    DeviceGuard dg(device);
    if (!dg.ok) {
        set_error("se_mesh_create: cannot select device " + std::to_string(device));
        return SE_ERR_HIP;
    }
    const HostMesh &h = m->h;
    DevMesh &d = m->d;
    d.nv = h.nv;
    d.ne = h.ne;
    SE_TRY(d.tri.upload(h.tri.data(), h.tri.size() * 4));
    SE_TRY(d.row_ptr.upload(h.row_ptr.data(), h.row_ptr.size() * 4));
    std::vector<int32_t> pcol(h.col.size());
    for (size_t j = 0; j < h.col.size(); ++j) pcol[j] = 3 * (h.col[j] >> 2) + (h.col[j] & 3);
    SE_TRY(d.pcol.upload(pcol.data(), pcol.size() * 4));
    auto g64 = pack_geom<double>(h, nullptr, 0);
    auto g32 = pack_geom<float>(h, nullptr, 0);
    SE_TRY(d.geom64.upload(g64.data(), g64.size() * 8));
    SE_TRY(d.geom32.upload(g32.data(), g32.size() * 4));
    SE_TRY(d.Av64.upload(h.Av.data(), h.Av.size() * 8));
    std::vector<float> av32(h.Av.begin(), h.Av.end());
    SE_TRY(d.Av32.upload(av32.data(), av32.size() * 4));
    const uint32_t zero = 0;
    SE_TRY(d.faults.upload(&zero, 4));
    *out = m.release();
    return SE_OK;
}

void se_mesh_destroy(se_mesh *mesh) {
    if (!mesh) return;
    if (mesh->device < 0) {
        delete mesh;
        return;
    }
    DeviceGuard dg(mesh->device);
    delete mesh;
}

se_status se_mesh_info(const se_mesh *m, int64_t *nv, int64_t *ne, int64_t *nnz, double *mu_max) {
    if (!m) {
        set_error("se_mesh_info: null mesh");
        return SE_ERR_ARG;
    }
    if (nv) *nv = m->h.nv;
    if (ne) *ne = m->h.ne;
    if (nnz) *nnz = 3 * m->h.ne;
    if (mu_max) *mu_max = m->h.mu_max;
    return SE_OK;
}

se_status se_mesh_perm(const se_mesh *m, int32_t *vperm, int32_t *eperm) {
    if (!m) {
        set_error("se_mesh_perm: null mesh");
        return SE_ERR_ARG;
    }
    if (vperm) std::memcpy(vperm, m->h.vperm.data(), m->h.nv * 4);
    if (eperm) std::memcpy(eperm, m->h.eperm.data(), m->h.ne * 4);
    return SE_OK;
}

se_status se_mesh_csr(const se_mesh *m, int32_t *tri, int32_t *row_ptr, int32_t *col) {
    if (!m) {
        set_error("se_mesh_csr: null mesh");
        return SE_ERR_ARG;
    }
    if (tri) std::memcpy(tri, m->h.tri.data(), m->h.tri.size() * 4);
    if (row_ptr) std::memcpy(row_ptr, m->h.row_ptr.data(), m->h.row_ptr.size() * 4);
    if (col) std::memcpy(col, m->h.col.data(), m->h.col.size() * 4);
    return SE_OK;
}

se_status se_mesh_neighbours(const se_mesh *m, int32_t *nb, double *l, double *lod) {
    if (!m) {
        set_error("se_mesh_neighbours: null mesh");
        return SE_ERR_ARG;
    }
    std::vector<int32_t> nb4;
    std::vector<double> vg;
    SE_TRY(build_visc_tables(m->h, nb4, vg));
    for (int64_t e = 0; e < m->h.ne; ++e)
        for (int j = 0; j < 3; ++j) {
            if (nb) nb[3 * e + j] = nb4[4 * e + j];
            if (l) l[3 * e + j] = vg[6 * e + 2 * j];
            if (lod) lod[3 * e + j] = vg[6 * e + 2 * j + 1];
        }
    return SE_OK;
}

se_status se_mesh_geometry(const se_mesh *m, double *Av, double *Ae, double *gN) {
    if (!m) {
        set_error("se_mesh_geometry: null mesh");
        return SE_ERR_ARG;
    }
    if (Av) std::memcpy(Av, m->h.Av.data(), m->h.nv * 8);
    if (Ae) std::memcpy(Ae, m->h.Ae.data(), m->h.ne * 8);
    if (gN) std::memcpy(gN, m->h.gN.data(), m->h.ne * 48);
    return SE_OK;
}

se_status se_batch_set_plan_impl(se_batch *b, int32_t tile, int32_t k_fused, int32_t block);
se_status se_batch_get_plan_impl(const se_batch *b, int32_t *tile, int32_t *k_fused, int32_t *block);
se_status se_batch_plan_stats_impl(const se_batch *b, int32_t tile, int32_t k_fused, int32_t block,
                                   se_plan_stats_t *stats);
se_status se_batch_faults_impl(se_batch *b, void *stream, uint32_t *bits);

se_status se_set_plan(void *obj, int32_t kind, int32_t tile, int32_t k_fused, int32_t block) {
    if (obj && kind == 1) return se_batch_set_plan_impl(static_cast<se_batch *>(obj), tile, k_fused, block);
    if (!obj || kind != 0) {
        set_error("se_set_plan: null object or unknown kind (0 mesh, 1 batch)");
        return SE_ERR_ARG;
    }
    se_mesh *m = static_cast<se_mesh *>(obj);
    if (m->device < 0) {   // host-only mesh: validate and remember the plan
        HostTiles ht;
        se_plan_stats_t st;
        std::vector<const HostMesh *> mem{&m->h};
        SE_TRY(plan_host(mem, {0, m->h.nv}, {0, m->h.ne}, tile, k_fused, block, ht, st));
        m->plan_T = tile;
        m->plan_K = k_fused;
        m->plan_block = block;
        return SE_OK;
    }
    DeviceGuard dg(m->device);
    std::unique_ptr<DevTiles> p;
    std::vector<const HostMesh *> mem{&m->h};
    SE_TRY(make_plan(mem, {0, m->h.nv}, {0, m->h.ne}, tile, k_fused, block, p));
    {
        std::lock_guard<std::mutex> lk(m->plan_mu);
        for (auto &d : m->dflt) d.reset();
        for (bool &b : m->no_own) b = false;
    }
    m->plan = std::move(p);
    m->plan_T = tile;
    m->plan_K = k_fused;
    m->plan_block = block;
    return SE_OK;
}

se_status se_get_plan(const void *obj, int32_t kind, int32_t *tile, int32_t *k_fused,
                      int32_t *block) {
    if (obj && kind == 1)
        return se_batch_get_plan_impl(static_cast<const se_batch *>(obj), tile, k_fused, block);
    if (!obj || kind != 0) {
        set_error("se_get_plan: null object or unsupported kind");
        return SE_ERR_ARG;
    }
    const se_mesh *m = static_cast<const se_mesh *>(obj);
    if (tile) *tile = m->plan_T;
    if (k_fused) *k_fused = m->plan_K;
    if (block) *block = m->plan_block;
    return SE_OK;
}

se_status se_plan_stats(const void *obj, int32_t kind, int32_t tile, int32_t k_fused,
                        int32_t block, se_plan_stats_t *stats) {
    if (obj && stats && kind == 1)
        return se_batch_plan_stats_impl(static_cast<const se_batch *>(obj), tile, k_fused, block,
                                        stats);
    if (!obj || !stats || kind != 0) {
        set_error("se_plan_stats: bad argument");
        return SE_ERR_ARG;
    }
    const se_mesh *m = static_cast<const se_mesh *>(obj);
    HostTiles ht;
    std::vector<const HostMesh *> mem{&m->h};
    return plan_host(mem, {0, m->h.nv}, {0, m->h.ne}, tile, k_fused, block, ht, *stats);
}

se_status se_workspace_bytes(const se_mesh *m, const se_params *p, int32_t nsub,
                             int32_t ckpt_every, size_t *bytes) {
    if (!m || !p || !bytes || nsub < 1) {
        set_error("se_workspace_bytes: bad argument");
        return SE_ERR_ARG;
    }
    const bool f32 = p->precision == SE_F32_MIXED;
    const Layout L = fwd_layout(m->h.nv, m->h.ne, f32, nsub, vol_width(m->h.nv),
                                p->scheme == SE_SCHEME_SESM, visc_on(p));
    *bytes = L.total;
    if (ckpt_every > 0) {
        const int32_t k = std::min(ckpt_every, nsub);
        *bytes = adj_layout(m->h.nv, m->h.ne, f32, nsub, k, L.total).total;
    }
    return SE_OK;
}

static se_status check_state(const se_state *st, const se_forcing *fo, const void *ws) {
    if (!st || !fo || !st->eta || !st->U || !fo->R || !fo->f || !fo->H0 || !ws) {
        set_error("null state, forcing or workspace array");
        return SE_ERR_ARG;
    }
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) {
        set_error("workspace must be 256-byte aligned");
        return SE_ERR_ARG;
    }
    return SE_OK;
}

// Access policy of the tile kernels for nv vertices: stream each tile's own tables and
// the write-back past the caches when one launch's working set exceeds the 256 MiB
// last-level cache (about 236 B per vertex in FP32, 356 in FP64; half more with the state of
// AB3-AM4 or the tables of the viscous term, wide); smaller ones stay cached from launch to
// launch and keep ordinary accesses.  60 substeps, us, ordinary / streamed:
//   SE FP32 900,000 vertices 797 / 849, 1,210,000 1118 / 1087, 1,380,000 1298 / 1198
//   SE FP64 550,482 795 / 839, 702,000 1049 / 1128, 801,000 1230 / 1240, 900,000 1417 / 1392
//   AB3-AM4 FP32 702,000 874 / 919, 801,000 1034 / 1024, 900,000 1170 / 1125
//   AB3-AM4 FP64 384,000 1022 / 1085, 524,288 1645 / 1590, 630,000 1984 / 1854
//   viscous FP32 702,000 2200 / 2274, 801,000 2505 / 2495, 900,000 2916 / 2787
//   viscous FP64 384,000 2351 / 2403, 524,288 3317 / 3228, 630,000 4045 / 3817
// (the line lay at half the cache for all forms).
static int32_t stream_policy(int64_t nv, bool f32, bool wide) {
    return (f32 ? 236.0 : 356.0) * (wide ? 1.5 : 1.0) * static_cast<double>(nv) >
           256.0 * 1024 * 1024;
}

// Launch arguments of the tile kernel on one mesh: plan tables, forcing, workspace
// (running sum, U^0 copy, volume partials); K substeps per launch, no average output.
static TileArgs tile_args(const se_mesh *m, const DevTiles &P, bool f32, const se_forcing *fo,
                          char *w, const Layout &L, const StepC &c) {
    TileArgs a{};
    a.nt = stream_policy(m->h.nv, f32, false);
    a.hdr = P.hdr.as<const TileHdrK>();
    a.lv_gid = P.lv_gid.as<const int32_t>();
    a.le_rec = P.le_rec.as<const uint32_t>();
    a.le_pos = P.le_pos.as<const uint32_t>();
    a.le_gid = P.le_gid.as<const int32_t>();
    a.se = P.se;
    a.sv = P.sv;
    a.cs_row = P.cs_row.as<const uint16_t>();
    a.lgeo = f32 ? P.geo32.p : P.geo64.p;
    a.lae = f32 ? P.ae32.p : P.ae64.p;
    a.lv_av = f32 ? P.lav32.p : P.lav64.p;
    a.mem = nullptr;
    a.c0 = c;
    a.R = fo->R;
    a.f = fo->f;
    a.H0 = fo->H0;
    a.W = fo->W;
    a.Av64 = m->d.Av64.as<const double>();
    a.sum = w + L.sum;
    a.U0c = w + L.U0c;
    a.Uavg = nullptr;
    a.vol_part = reinterpret_cast<double *>(w + L.vol);
    a.faults = m->d.faults.as<uint32_t>();
    a.K = P.K;
    a.ksub = P.K;
    a.ntiles = P.ntiles;
    a.xcd = 1;
    // tables loaded ahead of the header on launches of few tiles, which last as long as one
    // tile's chain of round trips: 60 substeps, us, after the header / ahead of it, 32 tiles
    // (2,048 vertices) FP32 92.5 / 90.5, FP64 96.7 / 92.1, viscous FP32 203 / 197, 113 tiles
    // (7,200) 94.3 / 92.4, 99.7 / 94.5, 207 / 202.  The price is the padding and the owned ids
    // that are read besides: tiles of 64 to 112 vertices gain up to 250 of them (16,000 vertices
    // FP64 100.2 / 94.7, 27,000 110.9 / 107.8), 250 tiles of 200 vertices lose (50,000 FP64
    // 130.4 / 136.1) and so do launches of more tiles than CUs (1,039 tiles FP32 578 / 585).
    // Up to 128 no mesh loses.
    a.early = P.ntiles <= 128 ? 1 : 0;
    a.cap_nv = P.max_nv;
    a.cap_ne = P.max_ne;
    a.cap_nvu = P.max_nvu;
    a.cap_cs = P.max_cs;
    a.ell = P.ell ? 1 : 0;
    return a;
}

se_status se_subcycle(se_mesh *m, const se_params *p, se_state *st, const se_forcing *fo,
                      int32_t nsub, double dt, void *ws, void *stream) {
    return sesub::subcycle_tile(m, p, st, fo, nsub, dt, ws, stream, true);
}

}  // extern "C"

// The tile-kernel subcycle behind se_subcycle and se_subcycle_noalloc.  With
// may_alloc false nothing is allocated: a missing plan or missing viscous tables are
// errors instead of being built here.
se_status sesub::subcycle_tile(se_mesh *m, const se_params *p, se_state *st,
                               const se_forcing *fo, int32_t nsub, double dt, void *ws,
                               void *stream, bool may_alloc) {
    SE_TRY(check_params(m, p, nsub, dt));
    const bool visc = visc_on(p);
    if (visc && p->scheme != SE_SCHEME_SE) {
        set_error("se_subcycle: the viscous term is implemented for SE_SCHEME_SE only");
        return SE_ERR_UNSUPPORTED;
    }
    SE_TRY(check_state(st, fo, ws));
    SE_TRY(check_device(m));
    DeviceGuard dg(m->device);
    const bool f32 = p->precision == SE_F32_MIXED;
    const bool sm = p->scheme == SE_SCHEME_SESM;
    DevTiles *PP = nullptr;
    SE_TRY(mesh_plan(m, (visc ? CL_VISC : sm ? CL_SESM : CL_FB) + (f32 ? 1 : 0), may_alloc,
                     static_cast<hipStream_t>(stream), &PP));
    if (!PP) {
        set_error("se_subcycle_noalloc: the mesh has no tile plan yet (se_set_plan, or one "
                  "se_subcycle call, makes one)");
        return SE_ERR_ARG;
    }
    DevTiles &P = *PP;
    if (!P.ok(f32, sm)) {
        set_error("se_subcycle: the current plan does not fit the register/LDS budget of this "
                  "precision and scheme (see se_plan_stats)");
        return SE_ERR_ARG;
    }
    const size_t es = f32 ? 4 : 8;
    size_t lds = P.lds(f32, sm);
    if (visc) {
        // two rings per substep
        lds = visc_lds(lds, f32, P.max_ne);
        if (!visc_fits(P, f32)) {
            set_error("se_subcycle: with the viscous term the plan needs k_fused >= 2, " +
                      std::to_string(lds) + " bytes of LDS within 160 KiB and at most " +
                      "3 / 1 (1024 threads) or 6 / 4 (512 threads) triangles per thread "
                      "(FP32 / FP64)");
            return SE_ERR_ARG;
        }
        if (!may_alloc && (!m->d.vnb.p || !P.vnb.p)) {
            set_error("se_subcycle_noalloc: the viscous tables of this mesh and plan are not "
                      "built yet (one se_subcycle call with the viscous term builds them)");
            return SE_ERR_ARG;
        }
        const bool built = P.vnb.p != nullptr;
        SE_TRY(ensure_visc(m));
        SE_TRY(ensure_tile_visc(m, P));
        if (!built && !m->plan) {
            // the tables of the plan that a later call of the other precision runs on when it
            // may not allocate (should they not fit, it is that call that reports it)
            DevTiles *any;
            {
                std::lock_guard<std::mutex> lk(m->plan_mu);
                any = m->dflt[CL_ANY].get();
            }
            if (any && any != &P && (visc_fits(*any, false) || visc_fits(*any, true)))
                (void)ensure_tile_visc(m, *any);
        }
    }
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t nv = m->h.nv, ne = m->h.ne;
    const Layout L = fwd_layout(nv, ne, f32, nsub, vol_width(nv), sm, visc);
    char *w = static_cast<char *>(ws);
    StepC c = make_step(p, nsub, dt);
    c.ntiles = P.ntiles;
    c.vol_off = 0;

    TileArgs a = tile_args(m, P, f32, fo, w, L, c);
    a.nt = stream_policy(nv, f32, sm || visc);
    a.Uavg = st->Uavg;
    a.ksub = visc ? P.K / 2 : P.K;
    void *eta_u = st->eta, *U_u = st->U;
    void *eta_w = w + L.eta_alt, *U_w = w + L.U_alt;
    const int nlaunch = (nsub + a.ksub - 1) / a.ksub;
    const int mode = sm ? 1 : (visc ? 2 : 0);
    if (visc) {
        // R - V(eta^0, U^0), read by every launch in place of R
        ViscArgs va = visc_args(m, f32, p, fo->H0, st->eta, st->U, w + L.vub);
        va.base = fo->R;
        va.sign = -1;
        va.out = w + L.vRb;
        HIP_TRY(launch_visc(f32, va, s), "se_subcycle viscous term");
        a.R = w + L.vRb;
        a.vnb = P.vnb.as<const uint32_t>();
        a.vgeo = f32 ? P.vgeo32.p : P.vgeo64.p;
        a.vA0 = p->visc_A0;
        a.vCv = p->visc_Cv;
    }
    HIP_TRY(prepare_tile(f32, mode, P.ept, P.block), "se_subcycle prepare");
    a.eta_u = eta_u;
    a.eta_w = eta_w;
    a.U_u = U_u;
    a.U_w = U_w;
    // The caller's state is read by the first launch and written by the last one, the
    // launches between alternate between two states in the workspace (the second one in
    // the plain path's flux array, 3 ne >= nv values, and in its copy of U^0): an odd
    // launch count needs no copy back and the caller's U serves as U^0 until the last
    // launch has read it (524,288 vertices FP32, 15 launches: two copies of 5.5 us less).
    // A single launch writes the workspace and is copied.
    a.direct = sm ? 0 : 1;
    a.U0c = U_u;
    void *se[3] = {eta_u, eta_w, w + L.phi}, *sU[3] = {U_u, U_w, w + L.U0c};
    for (int ch = 0; ch < nlaunch; ++ch) {
        a.chunk = ch;
        if (!sm) {
            const int in = ch == 0 ? 0 : 1 + ((ch - 1) & 1);
            const int out = ch + 1 == nlaunch && ch > 0 ? 0 : 1 + (ch & 1);
            a.eta_u = se[in];
            a.U_u = sU[in];
            a.eta_w = se[out];
            a.U_w = sU[out];
        } else {   // two sets in the workspace, launch ch writing set ch & 1
            for (int k = 0; k < 2; ++k) {
                const int set = (ch + 1 + k) & 1;
                for (int q = 0; q < 4; ++q) a.sm_v[k][q] = w + L.sv[4 * set + q];
                for (int q = 0; q < 3; ++q) a.sm_e[k][q] = w + L.se[3 * set + q];
            }
            if (ch == 0) {
                for (int q = 0; q < 3; ++q) a.sm_v[0][q] = eta_u;
                for (int q = 0; q < 2; ++q) a.sm_e[0][q] = U_u;
            }
        }
        HIP_TRY(launch_tile(f32, mode, P.ept, P.block, a, P.ntiles, lds, s), "se_subcycle launch");
    }
    if (sm) {
        // the last substep's transport update (pending) and the final elevation
        PlainArgs fa{};
        fa.nv = nv;
        fa.ne = ne;
        fa.tri = m->d.tri.as<const int32_t>();
        fa.geom = f32 ? m->d.geom32.p : m->d.geom64.p;
        fa.H0 = fo->H0;
        fa.R = fo->R;
        fa.f = fo->f;
        fa.eta = st->eta;
        fa.U = st->U;
        fa.eta1 = a.sm_v[1][0];
        fa.etaA = a.sm_v[1][3];
        fa.U1 = a.sm_e[1][0];
        fa.Uab = a.sm_e[1][2];
        fa.faults = m->d.faults.as<uint32_t>();
        fa.c = c;
        HIP_TRY(launch_sesm_fin(f32, fa, s), "se_subcycle final update");
    } else if (nlaunch == 1) {
        HIP_TRY(hipMemcpyAsync(eta_u, eta_w, nv * es, hipMemcpyDeviceToDevice, s), "copy eta");
        HIP_TRY(hipMemcpyAsync(U_u, U_w, 2 * ne * es, hipMemcpyDeviceToDevice, s), "copy U");
    }
    if (st->volume) {
        const int rows = (p->flags & SE_TRACK_VOLUME) ? nsub + 1 : 2;
        double add = 0.0;
        if (f32) {
            add = p->eta_ref * m->h.Av_total;
        }
        HIP_TRY(launch_vol_reduce(a.vol_part, P.ntiles, rows, add, st->volume, s), "volume");
    }
    return SE_OK;
}

extern "C" {

se_status se_subcycle_plain(se_mesh *m, const se_params *p, se_state *st, const se_forcing *fo,
                            int32_t nsub, double dt, void *ws, void *stream) {
    SE_TRY(check_params(m, p, nsub, dt));
    SE_TRY(check_state(st, fo, ws));
    SE_TRY(check_device(m));
    DeviceGuard dg(m->device);
    const bool f32 = p->precision == SE_F32_MIXED;
    const bool sesm = p->scheme == SE_SCHEME_SESM;
    const bool visc = visc_on(p);
    if (sesm && visc) {
        set_error("se_subcycle_plain: the viscous term is implemented for SE_SCHEME_SE only");
        return SE_ERR_UNSUPPORTED;
    }
    if (visc) SE_TRY(ensure_visc(m));
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t nv = m->h.nv, ne = m->h.ne;
    const Layout L = fwd_layout(nv, ne, f32, nsub, vol_width(nv), sesm, visc);
    char *w = static_cast<char *>(ws);
    PlainArgs a{};
    a.nv = nv;
    a.ne = ne;
    a.tri = m->d.tri.as<const int32_t>();
    a.row_ptr = m->d.row_ptr.as<const int32_t>();
    a.pcol = m->d.pcol.as<const int32_t>();
    a.geom = f32 ? m->d.geom32.p : m->d.geom64.p;
    a.H0 = fo->H0;
    a.R = fo->R;
    a.f = fo->f;
    a.W = fo->W;
    a.Av = f32 ? m->d.Av32.p : m->d.Av64.p;
    a.Av64 = m->d.Av64.as<const double>();
    a.eta = st->eta;
    a.U = st->U;
    a.phi = w + L.phi;
    a.sum = w + L.sum;
    a.U0c = w + L.U0c;
    a.Uavg = st->Uavg;
    a.vol_part = reinterpret_cast<double *>(w + L.vol);
    a.faults = m->d.faults.as<uint32_t>();
    a.c = make_step(p, nsub, dt);
    a.nblk_v = static_cast<int32_t>((nv + 255) / 256);
    if (sesm) {
        // histories start from the initial state
        const size_t es = f32 ? 4 : 8;
        a.eta1 = w + L.sv[0];
        a.eta2 = w + L.sv[1];
        a.etaA = w + L.sv[2];
        a.U1 = w + L.se[0];
        a.U2 = w + L.se[1];
        a.Uab = w + L.se[6];
        for (void *dst : {a.eta1, a.eta2})
            HIP_TRY(hipMemcpyAsync(dst, st->eta, nv * es, hipMemcpyDeviceToDevice, s), "history");
        for (void *dst : {a.U1, a.U2})
            HIP_TRY(hipMemcpyAsync(dst, st->U, 2 * ne * es, hipMemcpyDeviceToDevice, s), "history");
        for (int mm = 0; mm < nsub; ++mm) {
            a.m = mm;
            HIP_TRY(launch_sesm_step(f32, a, s), "se_subcycle_plain launch");
        }
    } else if (visc) {
        // R^hV of eq. (eq:viscosity_BT) at every substep, its initial value subtracted
        ViscArgs va = visc_args(m, f32, p, fo->H0, st->eta, st->U, w + L.vub);
        va.base = fo->R;
        va.sign = -1;
        va.out = w + L.vRb;
        HIP_TRY(launch_visc(f32, va, s), "se_subcycle_plain viscous term");
        va.base = w + L.vRb;
        va.sign = 1;
        va.out = w + L.vRe;
        a.R = w + L.vRe;
        for (int mm = 0; mm < nsub; ++mm) {
            a.m = mm;
            HIP_TRY(launch_visc(f32, va, s), "se_subcycle_plain viscous term");
            HIP_TRY(launch_plain_step(f32, a, s), "se_subcycle_plain launch");
        }
    } else {
        for (int mm = 0; mm < nsub; ++mm) {
            a.m = mm;
            HIP_TRY(launch_plain_step(f32, a, s), "se_subcycle_plain launch");
        }
    }
    if (st->volume) {
        const int rows = (p->flags & SE_TRACK_VOLUME) ? nsub + 1 : 2;
        double add = 0.0;
        if (f32) {
            add = p->eta_ref * m->h.Av_total;
        }
        HIP_TRY(launch_vol_reduce(a.vol_part, a.nblk_v, rows, add, st->volume, s), "volume");
    }
    return SE_OK;
}

// Tile tables of the trim for cap local triangles and vertices per tile, built at the first
// call that asks for them.
static se_status ensure_trim_tiles(se_mesh *m, int cap, const DevTrimTiles **out) {
    const auto it = m->d.trim_tiles.find(cap);
    if (it != m->d.trim_tiles.end()) {
        *out = it->second.get();
        return SE_OK;
    }
    TrimTiles tt;
    auto d = std::make_unique<DevTrimTiles>();
    if (build_trim_tiles(m->h, cap, kTrimTileOwn, cap, tt)) {
        SE_TRY(d->hdr.upload(tt.hdr.data(), tt.hdr.size() * 4));
        SE_TRY(d->lv.upload(tt.lv.data(), tt.lv.size() * 4));
        SE_TRY(d->le.upload(tt.le.data(), tt.le.size() * 4));
        SE_TRY(d->rloc.upload(tt.rloc.data(), tt.rloc.size() * 2));
        d->ntiles = tt.ntiles;
    }
    *out = d.get();
    m->d.trim_tiles[cap] = std::move(d);
    return SE_OK;
}

se_status se_trim_zstar(se_mesh *m, int32_t K, const double *H0, const double *eta_new,
                        const double *Uavg, const double *Ustar, const double *hn,
                        const double *h0, const double *W, double tau, double *U, double *hnew,
                        double *w, void *stream) {
    if (!m || !H0 || !eta_new || !Uavg || !Ustar || !hn || !h0 || !U || !hnew || !w) {
        set_error("se_trim_zstar: null argument");
        return SE_ERR_ARG;
    }
    if (K < 1 || K > 64 || !(tau > 0.0) || !std::isfinite(tau)) {
        set_error("se_trim_zstar: need 1 <= K <= 64 and a finite tau > 0");
        return SE_ERR_ARG;
    }
    SE_TRY(check_device(m));
    DeviceGuard dg(m->device);
    TrimArgs a{};
    a.nv = m->h.nv;
    a.ne = m->h.ne;
    a.K = K;
    a.tau = tau;
    a.tri = m->d.tri.as<const int32_t>();
    a.row_ptr = m->d.row_ptr.as<const int32_t>();
    a.pcol = m->d.pcol.as<const int32_t>();
    a.geom = m->d.geom64.as<const double>();
    a.Av = m->d.Av64.as<const double>();
    a.H0 = H0;
    a.eta_new = eta_new;
    a.Uavg = Uavg;
    a.Ustar = Ustar;
    a.hn = hn;
    a.h0 = h0;
    a.W = W;
    a.U = U;
    a.hnew = hnew;
    a.w = w;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    if (!m->d.slotS.p) {
        // sub-cell flux vectors S_k = -A_e grad N_k of every triangle, built on the host
        // and uploaded synchronously (visible to calls on any stream)
        const HostMesh &h = m->h;
        std::vector<double> S(6 * static_cast<size_t>(h.ne));
        for (int64_t e = 0; e < h.ne; ++e)
            for (int q = 0; q < 6; ++q) S[6 * e + q] = -h.Ae[e] * h.gN[6 * e + q];
        SE_TRY(m->d.slotS.upload(S.data(), S.size() * 8));
    }
    // the tile form (one launch), unless U is Ustar itself (a tile would overwrite
    // transports that a later tile still reads) or one vertex's row exceeds a tile
    const DevTrimTiles *T = nullptr;
    int cap = trim_tile_cap_e(K);
    if (U != Ustar) {
        SE_TRY(ensure_trim_tiles(m, cap, &T));
        if (T->ntiles == 0 && trim_tile_cap_wide(K) > 0) {
            cap = trim_tile_cap_wide(K);
            SE_TRY(ensure_trim_tiles(m, cap, &T));
        }
    }
    if (T && T->ntiles > 0) {
        a.tt_hdr = T->hdr.as<const int32_t>();
        a.tt_lv = T->lv.as<const int32_t>();
        a.tt_le = T->le.as<const int2>();
        a.tt_rloc = T->rloc.as<const uint16_t>();
        a.tt_ntiles = T->ntiles;
        a.tt_cap_v = cap;
        HIP_TRY(launch_trim_tile(a, m->d.slotS.as<const double>(), s), "se_trim_zstar launch");
        return SE_OK;
    }
    HIP_TRY(launch_trim(a, m->d.slotS.as<const double>(), s), "se_trim_zstar launch");
    return SE_OK;
}

// Neighbour tables of the viscous term, built on first use.
static se_status ensure_visc(se_mesh *m) {
    if (m->d.vnb.p) return SE_OK;
    std::vector<int32_t> nb4;
    std::vector<double> vg;
    SE_TRY(build_visc_tables(m->h, nb4, vg));
    std::vector<float> vg32(vg.begin(), vg.end());
    SE_TRY(m->d.vgeo64.upload(vg.data(), vg.size() * 8));
    SE_TRY(m->d.vgeo32.upload(vg32.data(), vg32.size() * 4));
    SE_TRY(m->d.vnb.upload(nb4.data(), nb4.size() * 4));
    return SE_OK;
}

// Tile-local neighbour tables of the viscous term for the mesh's current plan: for
// every local triangle, the local index of the triangle across each edge when it
// belongs to the tile (0xffff otherwise: a coast, or a neighbour beyond the loaded
// rings, which no updated triangle uses), and the edge geometry.
static se_status ensure_tile_visc(const se_mesh *m, DevTiles &P) {
    if (P.vnb.p) return SE_OK;
    std::vector<int32_t> nb4;
    std::vector<double> vg;
    SE_TRY(build_visc_tables(m->h, nb4, vg));
    const int64_t nle = static_cast<int64_t>(P.le_gid_host.size());
    std::vector<uint32_t> tnb(2 * nle);
    std::vector<double> tg64(P.ok64 ? 6 * nle : 0);   // of the precisions the plan runs in
    std::vector<float> tg32(P.ok32 ? 6 * nle : 0);
    std::vector<int32_t> eloc(m->h.ne, -1);
    for (int32_t t = 0; t < P.ntiles; ++t) {
        const int64_t off = static_cast<int64_t>(t) * P.se;
        const int32_t n = P.nE_host[static_cast<size_t>(t) * (P.K + 1) + P.K];
        for (int32_t q = 0; q < n; ++q) eloc[P.le_gid_host[off + q]] = q;
        for (int32_t q = 0; q < n; ++q) {
            const int64_t e = P.le_gid_host[off + q];
            uint32_t l3[3];
            for (int j = 0; j < 3; ++j) {
                const int32_t g = nb4[4 * e + j];
                l3[j] = (g >= 0 && eloc[g] >= 0) ? static_cast<uint32_t>(eloc[g]) : 0xffffu;
                for (int k = 0; k < 2; ++k) {
                    if (P.ok64) tg64[6 * (off + q) + 2 * j + k] = vg[6 * e + 2 * j + k];
                    if (P.ok32) tg32[6 * (off + q) + 2 * j + k] = static_cast<float>(vg[6 * e + 2 * j + k]);
                }
            }
            tnb[2 * (off + q)] = l3[0] | (l3[1] << 16);
            tnb[2 * (off + q) + 1] = l3[2] | (0xffffu << 16);
        }
        for (int32_t q = 0; q < n; ++q) eloc[P.le_gid_host[off + q]] = -1;
    }
    SE_TRY(P.vgeo64.upload(tg64.data(), tg64.size() * 8));
    SE_TRY(P.vgeo32.upload(tg32.data(), tg32.size() * 4));
    SE_TRY(P.vnb.upload(tnb.data(), tnb.size() * 4));
    return SE_OK;
}

static ViscArgs visc_args(const se_mesh *m, bool f32, const se_params *p, const void *H0,
                          const void *eta, const void *U, void *ubar) {
    ViscArgs va{};
    va.ne = m->h.ne;
    va.tri = m->d.tri.as<const int32_t>();
    va.nb = m->d.vnb.as<const int32_t>();
    va.vgeo = f32 ? m->d.vgeo32.p : m->d.vgeo64.p;
    va.geom = f32 ? m->d.geom32.p : m->d.geom64.p;
    va.H0 = H0;
    va.eta = eta;
    va.U = U;
    va.ubar = ubar;
    va.A0 = p->visc_A0;
    va.Cv = p->visc_Cv;
    va.eta_ref = f32 ? p->eta_ref : 0.0;
    va.linear_h = (p->flags & SE_LINEAR_H) ? 1 : 0;
    va.sign = 1;
    return va;
}

se_status se_barotropic_visc(se_mesh *m, int32_t precision, uint32_t flags, double eta_ref,
                             double A0, double Cv, const void *H0, const void *eta,
                             const void *U, void *V, void *ws, void *stream) {
    if (!m || !H0 || !eta || !U || !V || !ws) {
        set_error("se_barotropic_visc: null argument");
        return SE_ERR_ARG;
    }
    if (!(A0 >= 0.0) || !std::isfinite(A0) || !(Cv >= 0.0) || !std::isfinite(Cv) ||
        !std::isfinite(eta_ref)) {
        set_error("se_barotropic_visc: A0, Cv must be finite and >= 0, eta_ref finite");
        return SE_ERR_ARG;
    }
    if (precision != SE_F64 && precision != SE_F32_MIXED) {
        set_error("se_barotropic_visc: precision must be SE_F64 or SE_F32_MIXED");
        return SE_ERR_ARG;
    }
    SE_TRY(check_device(m));
    DeviceGuard dg(m->device);
    SE_TRY(ensure_visc(m));
    se_params p{};
    p.precision = precision;
    p.flags = flags & SE_LINEAR_H;
    p.eta_ref = eta_ref;
    p.visc_A0 = A0;
    p.visc_Cv = Cv;
    const bool f32 = precision == SE_F32_MIXED;
    ViscArgs va = visc_args(m, f32, &p, H0, eta, U, ws);
    va.out = V;
    HIP_TRY(launch_visc(f32, va, static_cast<hipStream_t>(stream)), "se_barotropic_visc launch");
    return SE_OK;
}

se_status se_forcing_assemble(se_mesh *m, int32_t K, const int32_t *nlev, const double *RA,
                     const double *RP, const double *RhV, const double *tau_s, const double *u,
                     double Cd, int32_t precision, void *R, void *stream) {
    if (!m || !R) {
        set_error("se_forcing_assemble: null mesh or output");
        return SE_ERR_ARG;
    }
    if (K < 1 || !(Cd >= 0.0) || !std::isfinite(Cd) || (Cd > 0.0 && !u)) {
        set_error("se_forcing_assemble: need K >= 1, a finite Cd >= 0, and u when Cd > 0");
        return SE_ERR_ARG;
    }
    if (precision != SE_F64 && precision != SE_F32_MIXED) {
        set_error("se_forcing_assemble: precision must be SE_F64 or SE_F32_MIXED");
        return SE_ERR_ARG;
    }
    if (static_cast<int64_t>(m->h.ne) * K > (int64_t(1) << 40)) {
        set_error("se_forcing_assemble: ne * K too large");
        return SE_ERR_ARG;
    }
    SE_TRY(check_device(m));
    DeviceGuard dg(m->device);
    ForcingArgs a{};
    a.ne = m->h.ne;
    a.K = K;
    a.out_f32 = precision == SE_F32_MIXED;
    a.Cd = Cd;
    a.nlev = nlev;
    a.RA = RA;
    a.RP = RP;
    a.RhV = RhV;
    a.u = u;
    a.tau_s = tau_s;
    a.R = R;
    a.faults = m->d.faults.as<uint32_t>();
    HIP_TRY(launch_forcing(a, static_cast<hipStream_t>(stream)), "se_forcing_assemble launch");
    return SE_OK;
}

se_status se_check_faults(void *obj, int32_t kind, void *stream, uint32_t *bits) {
    if (obj && bits && kind == 1) return se_batch_faults_impl(static_cast<se_batch *>(obj), stream, bits);
    if (!obj || !bits || kind != 0) {
        set_error("se_check_faults: bad argument");
        return SE_ERR_ARG;
    }
    se_mesh *m = static_cast<se_mesh *>(obj);
    SE_TRY(check_device(m));
    DeviceGuard dg(m->device);
    const hipStream_t s = static_cast<hipStream_t>(stream);
    HIP_TRY(hipStreamSynchronize(s), "se_check_faults sync");
    uint32_t v = 0;
    HIP_TRY(hipMemcpy(&v, m->d.faults.p, 4, hipMemcpyDeviceToHost), "se_check_faults copy");
    const uint32_t zero = 0;
    HIP_TRY(hipMemcpy(m->d.faults.p, &zero, 4, hipMemcpyHostToDevice), "se_check_faults reset");
    *bits = v;
    return SE_OK;
}


se_status se_subcycle_adjoint(se_mesh *m, const se_params *p, const void *eta0, const void *U0,
                              const se_forcing *fo, int32_t nsub, double dt, int32_t ckpt_every,
                              const void *lam_eta, const void *lam_U, const double *lam_Uavg,
                              void *g_eta0, void *g_U0, void *g_R, void *g_H0, void *ws,
                              void *stream) {
    SE_TRY(check_params(m, p, nsub, dt));
    if (p->scheme != SE_SCHEME_SE || visc_on(p)) {
        set_error("se_subcycle_adjoint: only the forward-backward scheme without the viscous "
                  "term has an adjoint");
        return SE_ERR_UNSUPPORTED;
    }
    if (!eta0 || !U0 || !fo || !fo->R || !fo->f || !fo->H0 || !ws) {
        set_error("se_subcycle_adjoint: null input, forcing or workspace");
        return SE_ERR_ARG;
    }
    if (ckpt_every < 1 || ckpt_every > nsub) {
        set_error("se_subcycle_adjoint: need 1 <= ckpt_every <= nsub");
        return SE_ERR_ARG;
    }
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) {
        set_error("workspace must be 256-byte aligned");
        return SE_ERR_ARG;
    }
    SE_TRY(check_device(m));
    DeviceGuard dg(m->device);
    const bool f32 = p->precision == SE_F32_MIXED;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t nv = m->h.nv, ne = m->h.ne;
    const size_t es = f32 ? 4 : 8;
    const Layout L = fwd_layout(nv, ne, f32, nsub, vol_width(nv));
    AdjLayout A = adj_layout(nv, ne, f32, nsub, ckpt_every, L.total);
    char *w = static_cast<char *>(ws);
    const size_t st_bytes = al((nv + 2 * ne) * es);
    auto st_eta = [&](size_t off) { return w + off; };
    auto st_U = [&](size_t off) { return w + off + nv * es; };

    // the caller's plan; else, once a forward subcycle has made a default, the adjoint's own;
    // else (it may not be made now, or none fits) the forward one's where it runs the reverse
    // kernel, or the one for every form
    const DevTiles *TP = m->plan.get();
    if (!TP) {
        bool planned;
        {
            std::lock_guard<std::mutex> lk(m->plan_mu);
            planned = m->dflt[CL_ANY] != nullptr;
        }
        DevTiles *own = nullptr;
        if (planned) SE_TRY(mesh_plan(m, CL_ADJ + (f32 ? 1 : 0), true, s, &own));
        std::lock_guard<std::mutex> lk(m->plan_mu);
        TP = own;
        if (!TP || !TP->adj_ready[f32 ? 1 : 0]) TP = m->dflt[CL_FB + (f32 ? 1 : 0)].get();
        if (!TP || !TP->adj_ready[f32 ? 1 : 0]) TP = m->dflt[CL_ANY].get();
    }
    const bool fwd_tiles = TP && TP->ok(f32, false) && TP->prepared[f32 ? 1 : 0];
    const bool rev_tiles = fwd_tiles && TP->adj_ready[f32 ? 1 : 0];
    // The reverse tile kernel reads the forward elevations alone, a fifth of a state or
    // less.  Where those of all substeps and two states for the forward launches to
    // alternate between fit the bytes that the checkpoints and segment buffers of this
    // ckpt_every take, the step is one segment: no substep runs forward twice and the
    // reverse launches are not cut at checkpoints (with two triangles per vertex so at any
    // ckpt_every up to about 180 substeps, on a strip of one triangle per vertex up to about
    // 60; 65,536 vertices FP64, M = 30, ckpt_every 5, one gradient: 220 -> 154 us).
    const size_t whole = al(static_cast<size_t>(nsub) * nv * es) + 2 * st_bytes;
    if (rev_tiles && A.nseg > 1 && A.ckpt + whole <= A.lam_eta) {
        A.k = nsub;
        A.nseg = 1;
        A.etraj = A.ckpt;
        A.traj[0] = A.lam_eta - 3 * st_bytes;   // slot 1 of either is all that is used
        A.traj[1] = A.lam_eta - 2 * st_bytes;
    }

    // forward substep (state update only) on the plain path
    PlainArgs fa{};
    fa.nv = nv;
    fa.ne = ne;
    fa.tri = m->d.tri.as<const int32_t>();
    fa.row_ptr = m->d.row_ptr.as<const int32_t>();
    fa.pcol = m->d.pcol.as<const int32_t>();
    fa.geom = f32 ? m->d.geom32.p : m->d.geom64.p;
    fa.H0 = fo->H0;
    fa.R = fo->R;
    fa.f = fo->f;
    fa.W = fo->W;
    fa.Av = f32 ? m->d.Av32.p : m->d.Av64.p;
    fa.Av64 = m->d.Av64.as<const double>();
    fa.phi = w + L.phi;
    fa.sum = w + L.sum;
    fa.U0c = w + L.U0c;
    fa.faults = m->d.faults.as<uint32_t>();
    fa.c = make_step(p, nsub, dt);
    fa.nblk_v = static_cast<int32_t>((nv + 255) / 256);
    fa.fwd_only = 1;
    // one forward substep from the state (se, sU) into the workspace state at off
    auto fstep = [&](const void *se, const void *sU, size_t off) -> se_status {
        fa.eta_src = se;
        fa.U_src = sU;
        fa.eta = st_eta(off);
        fa.U = st_U(off);
        HIP_TRY(launch_plain_step(f32, fa, s), "adjoint: forward substep");
        return SE_OK;
    };

    // 1. forward sweep storing a checkpoint every k substeps: state m (m = q k) in
    // checkpoint slot q, the caller's eta0, U0 standing for slot 0; the states between
    // checkpoints go to segment buffer 0 (no copies: each substep writes its result into
    // its slot).  The sweep stops at the last checkpoint: the states after it are
    // recomputed by the reverse sweep anyway.
    const int32_t k = A.k;
    auto ckpt_eta = [&](int32_t q) -> const void * { return q == 0 ? eta0 : st_eta(A.ckpt + st_bytes * q); };
    auto ckpt_U = [&](int32_t q) -> const void * { return q == 0 ? U0 : st_U(A.ckpt + st_bytes * q); };
    // state j of segment sg (j = 0: its checkpoint; else segment buffer sg mod 2)
    auto seg_off = [&](int32_t sg, int32_t j) { return A.traj[sg & 1] + st_bytes * j; };
    auto seg_eta = [&](int32_t sg, int32_t j) -> const void * {
        return j == 0 ? ckpt_eta(sg) : st_eta(seg_off(sg, j));
    };
    auto seg_U = [&](int32_t sg, int32_t j) -> const void * {
        return j == 0 ? ckpt_U(sg) : st_U(seg_off(sg, j));
    };
    if (fwd_tiles) {
        // The mesh has a tile plan for this precision: each segment runs as temporally
        // blocked launches from checkpoint q to checkpoint q + 1 (the tile path equals
        // the plain path bit for bit).  A segment is a subcycle of k substeps of this
        // dt_s; chunk i reads state B_i and writes B_{i+1} (B_0, B_n the checkpoints, the
        // others alternating between two free slots of the segment buffers).
        StepC c = fa.c;
        c.nsub = k;
        c.flags &= ~KF_TRACK_VOLUME;
        c.ntiles = TP->ntiles;
        c.vol_off = 0;
        TileArgs ta = tile_args(m, *TP, f32, fo, w, L, c);
        const size_t lds = TP->lds(f32, false);
        const int32_t nch = (k + TP->K - 1) / TP->K;
        for (int32_t q = 0; q + 1 < A.nseg; ++q) {
            for (int32_t i = 0; i < nch; ++i) {
                void *se = i == 0 ? const_cast<void *>(ckpt_eta(q)) : st_eta(seg_off((i - 1) & 1, 1));
                void *sU = i == 0 ? const_cast<void *>(ckpt_U(q)) : st_U(seg_off((i - 1) & 1, 1));
                void *de = i + 1 == nch ? st_eta(A.ckpt + st_bytes * (q + 1)) : st_eta(seg_off(i & 1, 1));
                void *dU = i + 1 == nch ? st_U(A.ckpt + st_bytes * (q + 1)) : st_U(seg_off(i & 1, 1));
                ta.direct = 1;
                ta.eta_u = se;
                ta.U_u = sU;
                ta.eta_w = de;
                ta.U_w = dU;
                ta.chunk = i;
                HIP_TRY(launch_tile(f32, 0, TP->ept, TP->block, ta, TP->ntiles, lds, s),
                        "adjoint: forward sweep");
            }
        }
    } else {
        const void *ce = eta0, *cU = U0;
        const int32_t last_ckpt = (A.nseg - 1) * k;
        for (int32_t n1 = 1; n1 <= last_ckpt; ++n1) {   // n1: index of the state produced
            const size_t dst = n1 % k == 0 ? A.ckpt + st_bytes * (n1 / k) : seg_off(0, n1 % k);
            SE_TRY(fstep(ce, cU, dst));
            ce = st_eta(dst);
            cU = st_U(dst);
        }
    }

    auto seg_len = [&](int32_t sg) { return std::min(nsub, sg * k + k) - sg * k; };
    AdjArgs aa{};
    aa.nv = nv;
    aa.ne = ne;
    aa.tri = fa.tri;
    aa.row_ptr = fa.row_ptr;
    aa.pcol = fa.pcol;
    aa.geom = fa.geom;
    aa.H0 = fo->H0;
    aa.Av = fa.Av;
    aa.f = fo->f;
    aa.lam_eta = w + A.lam_eta;
    aa.lam_U = w + A.lam_U;
    aa.lam_Uavg = lam_Uavg;
    aa.gR = g_R ? g_R : static_cast<void *>(w + A.gR);
    aa.gH0 = g_H0 ? g_H0 : static_cast<void *>(w + A.gH0);
    aa.psi = w + A.psi;
    aa.c = fa.c;
    aa.rM = 1.0 / static_cast<double>(nsub);
    aa.thrM = p->theta * aa.rM;

    if (rev_tiles) {
        // 2'. reverse sweep on the tile plan, segment by segment from the last.  A
        // segment's forward elevations are recomputed from its checkpoint on the tile
        // kernel (mode 3: each substep's owned elevations to the segment's trajectory
        // buffer, two buffers alternating by segment), its reverse substeps run up to K
        // per launch on the reverse tile kernel (the adjoint state alternating between
        // two buffers).  The recompute of segment sg - 1 shares the launches of the
        // reverse substeps of segment sg (independent work on disjoint arrays); only
        // the last segment's recompute runs alone.  The sweep's first launch starts from
        // the seeds and its last one writes the gradients of the initial state (the
        // seed and final kernels of the per-substep path folded in).
        const DevTiles &P = *TP;
        StepC c = fa.c;
        c.flags &= ~KF_TRACK_VOLUME;
        c.ntiles = P.ntiles;
        c.vol_off = 0;
        const size_t traj_bytes = al(static_cast<size_t>(k) * nv * es);
        auto traj_of = [&](int32_t sg) { return static_cast<void *>(w + A.etraj + (sg & 1) * traj_bytes); };
        AdjTileArgs ra{};
        ra.hdr = P.hdr.as<const TileHdrK>();
        ra.lv_gid = P.lv_gid.as<const int32_t>();
        ra.le_rec = P.le_rec.as<const uint32_t>();
        ra.le_pos = P.le_pos.as<const uint32_t>();
        ra.le_gid = P.le_gid.as<const int32_t>();
        ra.se = P.se;
        ra.sv = P.sv;
        ra.cs_row = P.cs_row.as<const uint16_t>();
        ra.lgeo = f32 ? P.geo32.p : P.geo64.p;
        ra.lae = f32 ? P.ae32.p : P.ae64.p;
        ra.lv_av = f32 ? P.lav32.p : P.lav64.p;
        ra.H0 = fo->H0;
        ra.f = fo->f;
        ra.traj_stride = nv;
        ra.lam_Uavg = lam_Uavg;
        ra.gR = aa.gR;
        ra.gH0 = aa.gH0;
        ra.c = fa.c;
        ra.rM = aa.rM;
        ra.thrM = aa.thrM;
        ra.K = P.K;
        ra.ntiles = P.ntiles;
        ra.xcd = 1;
        ra.ell = P.ell ? 1 : 0;
        ra.cap_nv = P.max_nv;
        ra.cap_ne = P.max_ne;
        ra.cap_nvu = P.max_nvu;
        ra.cap_cs = P.max_cs;
        void *lam_e[2] = {w + A.lam_eta, w + A.lam_eta2};
        void *lam_u[2] = {w + A.lam_U, w + A.lam_U2};
        int cur = 0;
        const size_t lds_f = P.lds(f32, false), lds_r = P.lds_adj[f32 ? 1 : 0];
        const size_t lds_p = std::max(lds_f, lds_r);
        // recompute launches of segment sg (none when it has a single substep)
        auto recompute = [&](int32_t sg) {
            std::vector<TileArgs> v;
            const int32_t len = seg_len(sg);
            if (len <= 1) return v;
            StepC cs = c;
            cs.nsub = len;
            TileArgs ta = tile_args(m, P, f32, fo, w, L, cs);
            ta.traj = traj_of(sg);
            ta.traj_stride = nv;
            const int32_t nch = (len + P.K - 1) / P.K;
            for (int32_t i = 0; i < nch; ++i) {
                void *se = i == 0 ? const_cast<void *>(ckpt_eta(sg)) : st_eta(seg_off((i - 1) & 1, 1));
                void *sU = i == 0 ? const_cast<void *>(ckpt_U(sg)) : st_U(seg_off((i - 1) & 1, 1));
                void *de = st_eta(seg_off(i & 1, 1));
                void *dU = st_U(seg_off(i & 1, 1));
                ta.direct = 1;
                ta.eta_u = se;
                ta.U_u = sU;
                ta.eta_w = de;
                ta.U_w = dU;
                ta.chunk = i;
                v.push_back(ta);
            }
            return v;
        };
        for (const TileArgs &ta : recompute(A.nseg - 1))
            HIP_TRY(launch_tile(f32, 3, P.ept, P.block, ta, P.ntiles, lds_f, s),
                    "adjoint: last segment recompute");
        for (int32_t sg = A.nseg - 1; sg >= 0; --sg) {
            const std::vector<TileArgs> rec = sg > 0 ? recompute(sg - 1) : std::vector<TileArgs>();
            ra.eta_s0 = ckpt_eta(sg);
            ra.traj = traj_of(sg);
            size_t i = 0;
            for (int32_t s_hi = seg_len(sg); s_hi > 0; ++i) {
                const int32_t cntr = std::min(P.K, s_hi);
                const bool first = sg == A.nseg - 1 && i == 0, last = sg == 0 && s_hi == cntr;
                ra.cnt = cntr;
                ra.s_hi = s_hi;
                ra.seed = first ? 1 : 0;
                ra.lam_eta_in = first ? lam_eta : lam_e[cur];
                ra.lam_U_in = first ? lam_U : lam_u[cur];
                ra.lam_eta_out = lam_e[cur ^ 1];
                ra.lam_U_out = lam_u[cur ^ 1];
                ra.fin = last ? 1 : 0;
                ra.g_eta0 = last ? g_eta0 : nullptr;
                ra.g_U0 = last ? g_U0 : nullptr;
                if (i < rec.size())
                    HIP_TRY(launch_adj_tile_pair(f32, P.ept, P.block, ra, rec[i], lds_p, s),
                            "adjoint: reverse substeps and recompute");
                else
                    HIP_TRY(launch_adj_tile(f32, P.ept, P.block, ra, lds_r, s),
                            "adjoint: reverse substeps");
                cur ^= 1;
                s_hi -= cntr;
            }
            for (; i < rec.size(); ++i)
                HIP_TRY(launch_tile(f32, 3, P.ept, P.block, rec[i], P.ntiles, lds_f, s),
                        "adjoint: segment recompute");
        }
        return SE_OK;
    }
    HIP_TRY(launch_adj_init(f32, aa, lam_eta, lam_U, s), "adjoint: init");

    // 2. reverse sweep, segment by segment.  Segment sg (substeps m0 .. m1 - 1) needs its
    // states m0 + 1 .. m1 - 1, recomputed from its checkpoint into segment buffer sg mod 2.
    // The last segment is recomputed alone; every other segment's recompute runs in the
    // same launches as the reverse substeps of the segment after it (independent work on
    // disjoint buffers), which halves the chain of dependent launches.
    {
        const int32_t sg = A.nseg - 1;
        for (int32_t j = 1; j < seg_len(sg); ++j)
            SE_TRY(fstep(seg_eta(sg, j - 1), seg_U(sg, j - 1), seg_off(sg, j)));
    }
    for (int32_t sg = A.nseg - 1; sg >= 0; --sg) {
        const int32_t nrev = seg_len(sg);                 // reverse substeps of sg
        const int32_t nrec = sg > 0 ? seg_len(sg - 1) - 1 : 0;   // recompute of sg - 1
        for (int32_t i = 0; i < std::max(nrev, nrec); ++i) {
            const bool rev = i < nrev, rec = i < nrec;
            if (rev) aa.eta_m = seg_eta(sg, nrev - 1 - i);
            if (rec) {
                fa.eta_src = seg_eta(sg - 1, i);
                fa.U_src = seg_U(sg - 1, i);
                fa.eta = st_eta(seg_off(sg - 1, i + 1));
                fa.U = st_U(seg_off(sg - 1, i + 1));
            }
            if (rev && rec)
                HIP_TRY(launch_adj_pair(f32, aa, fa, s), "adjoint: reverse substep and recompute");
            else if (rev)
                HIP_TRY(launch_adj_step(f32, aa, s), "adjoint: reverse substep");
            else
                HIP_TRY(launch_plain_step(f32, fa, s), "adjoint: recompute");
        }
    }
    HIP_TRY(launch_adj_final(f32, aa, g_eta0, g_U0, s), "adjoint: final");
    return SE_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Batched ensemble: a disjoint union of member meshes sharing one tile table
// ---------------------------------------------------------------------------
struct se_batch {
    int device = 0;
    std::vector<sesub::HostMesh> h;
    std::vector<int64_t> voff, eoff;
    int64_t nv = 0, ne = 0;
    std::vector<double> atot;            // per member total area
    sesub::DevBuf Av64, Av32, faults;
    int32_t plan_T = 768, plan_K = 4, plan_block = 512;
    struct Graph {
        std::vector<uint64_t> key;
        hipGraph_t g = nullptr;
        hipGraphExec_t x = nullptr;
    };
    // What the calls of one precision run on: the plan (the caller's, one for both precisions,
    // or a default of that precision) and what follows from it and the last configuration
    struct Exec {
        std::shared_ptr<sesub::DevTiles> plan;
        std::vector<int32_t> mtiles, mtile_first;   // tiles per member, the first of them
        sesub::DevBuf table, lists;
        std::vector<sesub::StepC> table_host;
        std::vector<int32_t> list_off;   // per launch offset into lists (size nlaunch + 1)
        // one-launch epilogue of a call: volume rows of every member, final states that
        // ended in the workspace copied back (per configuration, host copies to compare)
        sesub::DevBuf voltab, cpytab;
        std::vector<sesub::VolMember> voltab_host;
        std::vector<sesub::CopyRange> cpytab_host;
        std::vector<Graph> graphs;
        void drop_graphs() {
            for (auto &gr : graphs) {
                if (gr.x) (void)hipGraphExecDestroy(gr.x);
                if (gr.g) (void)hipGraphDestroy(gr.g);
            }
            graphs.clear();
        }
        ~Exec() { drop_graphs(); }
    } exec[2];                           // FP64, FP32
};

namespace sesub {
namespace {

std::vector<const HostMesh *> batch_members(const se_batch *b) {
    std::vector<const HostMesh *> v;
    for (const auto &m : b->h) v.push_back(&m);
    return v;
}

void batch_use_plan(se_batch *b, se_batch::Exec &x, const std::shared_ptr<DevTiles> &p) {
    const size_t n = b->h.size();
    x.mtiles.assign(n, 0);
    x.mtile_first.assign(n, -1);
    for (size_t t = 0; t < p->hdr_host.size(); ++t) {
        const int mb = p->hdr_host[t].member;
        if (x.mtile_first[mb] < 0) x.mtile_first[mb] = static_cast<int32_t>(t);
        x.mtiles[mb]++;
    }
    x.plan = p;
    x.table_host.clear();   // forces a new schedule
    x.drop_graphs();
}

// Default plan of a batch, chosen at its first call from the vertices of all members and
// the call's precision, among the plans that run in both: about one 512-thread tile per CU
// with many rings while the members together are that small, else two per CU.  24 basins
// of 3,000 to 40,000 vertices (513,187 in all) FP32: 512,2,512 1045, 352,5,512 722 us per
// call cold; FP64 1927, 256,4,512 1234; eight of 2,000 to 8,000 (36,883) 256,4,512 236 and
// 283, 128,8,512 196 and 233.
//
// One default per precision, so that a call runs on the same plan whichever precision came
// first (24 basins FP64 after FP32: 1,324 us on the FP32 plan, 1,054 on its own).  Where no
// plan may be made (a stream under capture) or none finds memory, the other precision's
// stands in: a default runs in both.
se_status batch_exec(se_batch *b, bool f32, hipStream_t s, se_batch::Exec **out) {
    se_batch::Exec &x = b->exec[f32 ? 1 : 0], &other = b->exec[f32 ? 0 : 1];
    *out = &x;
    if (x.plan) return SE_OK;
    if (other.plan && s) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
            *out = &other;
            return SE_OK;
        }
    }
    std::vector<PlanCand> cand;
    if (b->nv <= 75000) {
        const int32_t T = std::max<int32_t>(64, static_cast<int32_t>((b->nv + 287) / 288 + 7) / 8 * 8);
        for (int32_t K : {8, 6, 5}) cand.push_back({T, K, 512, 4, 0});
    }
    if (f32) {
        cand.push_back({352, 5, 512, 4, 0});
        cand.push_back({320, 5, 512, 4, 0});
        cand.push_back({448, 4, 512, 4, 0});
    }
    cand.push_back({256, 4, 512, 3, 0});
    cand.push_back({256, 4, 512, 4, 0});
    for (const PlanCand &c : {PlanCand{768, 4, 512, 8, 0}, PlanCand{512, 4, 512, 8, 0},
                              PlanCand{512, 2, 512, 8, 0}, PlanCand{256, 4, 512, 8, 0},
                              PlanCand{256, 2, 256, 8, 0}, PlanCand{128, 2, 256, 8, 0},
                              PlanCand{64, 1, 256, 8, 0}})
        cand.push_back(c);
    for (const auto &c : cand) {
        HostTiles ht;
        se_plan_stats_t st;
        if (plan_host(batch_members(b), b->voff, b->eoff, c.T, c.K, c.block, ht, st) != SE_OK)
            continue;
        if (!st.ok_f32 || !st.ok_f64 || st.tri_per_thread > c.ept) continue;
        if (other.plan && other.plan->T == c.T && other.plan->K == c.K && other.plan->block == c.block) {
            batch_use_plan(b, x, other.plan);
            return SE_OK;
        }
        std::unique_ptr<DevTiles> p;
        const se_status rc = upload_plan(batch_members(b), b->voff, b->eoff, c.T, c.K, c.block, ht, st, 3, p);
        if (rc == SE_OK) {
            batch_use_plan(b, x, std::move(p));
            if (!other.plan) {
                b->plan_T = c.T;
                b->plan_K = c.K;
                b->plan_block = c.block;
            }
        } else if (other.plan) {
            batch_use_plan(b, x, other.plan);
        } else {
            return rc;
        }
        return SE_OK;
    }
    set_error("no default plan fits this batch");
    return SE_ERR_ARG;
}

int64_t batch_vol_rows(const se_params *p, const int32_t *nsub, size_t i) {
    return (p->flags & SE_TRACK_VOLUME) ? nsub[i] + 1 : 2;
}

struct BatchLayout {
    size_t eta_alt, U_alt, sum, U0c, vol, total;
    std::vector<int64_t> vol_off;   // per member offset (elements) into vol partials
};

BatchLayout batch_layout(const se_batch *b, bool f32, const se_params *p, const int32_t *nsub) {
    const size_t s = f32 ? 4 : 8;
    BatchLayout L{};
    size_t o = 0;
    L.eta_alt = o;
    o += al(b->nv * s);
    L.U_alt = o;
    o += al(2 * b->ne * s);
    L.sum = o;
    o += al(16 * b->ne);
    L.U0c = o;
    o += al(2 * b->ne * s);
    L.vol = o;
    int64_t acc = 0;
    for (size_t i = 0; i < b->h.size(); ++i) {
        L.vol_off.push_back(acc);
        acc += batch_vol_rows(p, nsub, i) * ((b->h[i].nv + 63) / 64);
    }
    o += al(acc * 8);
    L.total = o;
    return L;
}

}  // namespace
}  // namespace sesub

extern "C" {

se_status se_batch_create(se_mesh *const *members, int32_t n, se_batch **out) {
    if (!members || n < 1 || !out) {
        set_error("se_batch_create: need n >= 1 members and an output pointer");
        return SE_ERR_ARG;
    }
    *out = nullptr;
    auto b = std::make_unique<se_batch>();
    b->device = members[0] ? members[0]->device : -1;
    b->voff.push_back(0);
    b->eoff.push_back(0);
    for (int32_t i = 0; i < n; ++i) {
        if (!members[i] || members[i]->device != b->device) {
            set_error("se_batch_create: null member or members on different devices");
            return SE_ERR_ARG;
        }
        b->h.push_back(members[i]->h);
        b->voff.push_back(b->voff.back() + members[i]->h.nv);
        b->eoff.push_back(b->eoff.back() + members[i]->h.ne);
    }
    b->nv = b->voff.back();
    b->ne = b->eoff.back();
    if (b->nv >= (int64_t(1) << 31) || b->ne >= (int64_t(1) << 30)) {
        set_error("se_batch_create: batch too large for 32-bit indices");
        return SE_ERR_ARG;
    }
    std::vector<double> av;
    av.reserve(b->nv);
    for (const auto &m : b->h) {
        b->atot.push_back(m.Av_total);
        av.insert(av.end(), m.Av.begin(), m.Av.end());
    }
    if (b->device >= 0) {
        DeviceGuard dg(b->device);
        SE_TRY(b->Av64.upload(av.data(), av.size() * 8));
        std::vector<float> av32(av.begin(), av.end());
        SE_TRY(b->Av32.upload(av32.data(), av32.size() * 4));
        const uint32_t zero = 0;
        SE_TRY(b->faults.upload(&zero, 4));
    }
    *out = b.release();
    return SE_OK;
}

void se_batch_destroy(se_batch *b) {
    if (!b) return;
    if (b->device < 0) {
        delete b;
        return;
    }
    DeviceGuard dg(b->device);
    delete b;
}

se_status se_batch_info(const se_batch *b, int64_t *nv_total, int64_t *ne_total,
                        int64_t *vert_offset, int64_t *elem_offset) {
    if (!b) {
        set_error("se_batch_info: null batch");
        return SE_ERR_ARG;
    }
    if (nv_total) *nv_total = b->nv;
    if (ne_total) *ne_total = b->ne;
    if (vert_offset) std::memcpy(vert_offset, b->voff.data(), b->voff.size() * 8);
    if (elem_offset) std::memcpy(elem_offset, b->eoff.data(), b->eoff.size() * 8);
    return SE_OK;
}

se_status se_batch_workspace_bytes(const se_batch *b, const se_params *p, const int32_t *nsub,
                                   size_t *bytes) {
    if (!b || !p || !nsub || !bytes) {
        set_error("se_batch_workspace_bytes: bad argument");
        return SE_ERR_ARG;
    }
    for (size_t i = 0; i < b->h.size(); ++i)
        if (nsub[i] < 1) {
            set_error("se_batch_workspace_bytes: nsub must be >= 1");
            return SE_ERR_ARG;
        }
    *bytes = batch_layout(b, p->precision == SE_F32_MIXED, p, nsub).total;
    return SE_OK;
}

se_status se_subcycle_batched(se_batch *b, const se_params *p, se_state *st, const se_forcing *fo,
                              const int32_t *nsub, const double *dt, int use_graph, void *ws,
                              void *stream) {
    if (!b || !p || !nsub || !dt) {
        set_error("se_subcycle_batched: null argument");
        return SE_ERR_ARG;
    }
    if (p->scheme != SE_SCHEME_SE || visc_on(p)) {
        set_error("se_subcycle_batched: only the forward-backward scheme without the viscous "
                  "term is batched");
        return SE_ERR_UNSUPPORTED;
    }
    SE_TRY(check_state(st, fo, ws));
    if (b->device < 0) {
        set_error("host-only batch cannot run kernels");
        return SE_ERR_ARG;
    }
    const size_t n = b->h.size();
    // per-member validation (CFL uses each member's own spectral bound)
    for (size_t i = 0; i < n; ++i) {
        se_mesh probe;
        probe.h.mu_max = b->h[i].mu_max;
        SE_TRY(check_params(&probe, p, nsub[i], dt[i]));
    }
    const hipStream_t s = static_cast<hipStream_t>(stream);
    if (use_graph && s == nullptr) {
        set_error("se_subcycle_batched: graph capture needs a non-default stream");
        return SE_ERR_ARG;
    }
    DeviceGuard dg(b->device);
    const bool f32 = p->precision == SE_F32_MIXED;
    se_batch::Exec *x = nullptr;
    SE_TRY(batch_exec(b, f32, s, &x));
    const DevTiles &P = *x->plan;
    if (!(f32 ? P.ok32 : P.ok64)) {
        set_error("se_subcycle_batched: plan does not fit this precision");
        return SE_ERR_ARG;
    }
    const BatchLayout L = batch_layout(b, f32, p, nsub);
    const int32_t K = P.K;

    // member constants and launch offsets (balance the active tiles per launch)
    std::vector<StepC> tab(n);
    std::vector<int32_t> Lm(n), order(n);
    int32_t Lmax = 0;
    for (size_t i = 0; i < n; ++i) {
        Lm[i] = (nsub[i] + K - 1) / K;
        Lmax = std::max(Lmax, Lm[i]);
        order[i] = static_cast<int32_t>(i);
    }
    std::sort(order.begin(), order.end(), [&](int32_t i, int32_t j) {
        return Lm[i] != Lm[j] ? Lm[i] > Lm[j] : x->mtiles[i] > x->mtiles[j];
    });
    std::vector<int64_t> load(Lmax, 0);
    std::vector<int32_t> off(n, 0);
    for (int32_t i : order) {
        int32_t best = 0;
        int64_t best_peak = -1;
        for (int32_t o = 0; o + Lm[i] <= Lmax; ++o) {
            int64_t peak = 0;
            for (int32_t c = o; c < o + Lm[i]; ++c) peak = std::max(peak, load[c]);
            if (best_peak < 0 || peak < best_peak) {
                best_peak = peak;
                best = o;
            }
        }
        off[i] = best;
        for (int32_t c = best; c < best + Lm[i]; ++c) load[c] += x->mtiles[i];
    }
    for (size_t i = 0; i < n; ++i) {
        tab[i] = make_step(p, nsub[i], dt[i]);
        tab[i].ntiles = x->mtiles[i];
        tab[i].vol_off = L.vol_off[i];
        tab[i].chunk0 = off[i];
    }
    const bool same = x->table_host.size() == n &&
                      std::memcmp(x->table_host.data(), tab.data(), n * sizeof(StepC)) == 0;
    if (!same) {
        // new configuration: upload constants and per-launch tile lists
        HIP_TRY(hipStreamSynchronize(s), "batched: sync before table update");
        std::vector<int32_t> lists;
        std::vector<int32_t> loff{0};
        for (int32_t c = 0; c < Lmax; ++c) {
            for (size_t i = 0; i < n; ++i)
                if (c >= off[i] && c < off[i] + Lm[i])
                    for (int32_t t = 0; t < x->mtiles[i]; ++t) lists.push_back(x->mtile_first[i] + t);
            loff.push_back(static_cast<int32_t>(lists.size()));
        }
        SE_TRY(x->table.upload(tab.data(), n * sizeof(StepC)));
        SE_TRY(x->lists.upload(lists.data(), std::max<size_t>(lists.size(), 1) * 4));
        x->list_off = loff;
        x->table_host = tab;
        x->drop_graphs();
    }
    // epilogue tables: volume rows per member, and the word ranges of the members
    // whose last chunk wrote the workspace buffers (an odd number of chunks)
    const size_t es = f32 ? 4 : 8;
    std::vector<VolMember> vt;
    int32_t vrows = 0;
    for (size_t i = 0; i < n; ++i) {
        const int32_t rows = static_cast<int32_t>(batch_vol_rows(p, nsub, i));
        VolMember vm{};
        vm.part_off = L.vol_off[i];
        vm.out_off = vrows;
        vm.width = x->mtiles[i];
        vm.row0 = vrows;
        vm.add = f32 ? p->eta_ref * b->atot[i] : 0.0;
        vt.push_back(vm);
        vrows += rows;
    }
    std::vector<CopyRange> ct;
    int64_t cwords = 0;
    const int64_t wpe = static_cast<int64_t>(es / 4);   // 32-bit words per value
    for (size_t i = 0; i < n; ++i) {
        if (Lm[i] % 2 == 0) continue;
        CopyRange re{b->voff[i] * wpe, cwords, 0, 0};
        ct.push_back(re);
        cwords += b->h[i].nv * wpe;
        CopyRange ru{2 * b->eoff[i] * wpe, cwords, 1, 0};
        ct.push_back(ru);
        cwords += 2 * b->h[i].ne * wpe;
    }
    auto differs = [](const auto &x, const auto &y) {
        return x.size() != y.size() ||
               (!x.empty() && std::memcmp(x.data(), y.data(), x.size() * sizeof(x[0])) != 0);
    };
    if (differs(vt, x->voltab_host) || differs(ct, x->cpytab_host)) {
        HIP_TRY(hipStreamSynchronize(s), "batched: sync before epilogue table update");
        x->drop_graphs();
        SE_TRY(x->voltab.upload(vt.data(), vt.size() * sizeof(VolMember)));
        if (ct.empty())
            SE_TRY(x->cpytab.alloc(sizeof(CopyRange)));   // never read (no ranges)
        else
            SE_TRY(x->cpytab.upload(ct.data(), ct.size() * sizeof(CopyRange)));
        x->voltab_host = vt;
        x->cpytab_host = ct;
    }
    char *w = static_cast<char *>(ws);
    TileArgs a{};
    a.nt = stream_policy(b->nv, f32, false);
    a.hdr = P.hdr.as<const TileHdrK>();
    a.lv_gid = P.lv_gid.as<const int32_t>();
    a.le_rec = P.le_rec.as<const uint32_t>();
    a.le_pos = P.le_pos.as<const uint32_t>();
    a.le_gid = P.le_gid.as<const int32_t>();
    a.se = P.se;
    a.sv = P.sv;
    a.cs_row = P.cs_row.as<const uint16_t>();
    a.lgeo = f32 ? P.geo32.p : P.geo64.p;
    a.lae = f32 ? P.ae32.p : P.ae64.p;
    a.lv_av = f32 ? P.lav32.p : P.lav64.p;
    a.mem = x->table.as<const StepC>();
    a.R = fo->R;
    a.f = fo->f;
    a.H0 = fo->H0;
    a.W = fo->W;
    a.Av64 = b->Av64.as<const double>();
    a.sum = w + L.sum;
    a.U0c = w + L.U0c;
    a.Uavg = st->Uavg;
    a.vol_part = reinterpret_cast<double *>(w + L.vol);
    a.faults = b->faults.as<uint32_t>();
    a.K = K;
    a.ksub = K;
    a.xcd = 1;
    a.cap_nv = P.max_nv;
    a.cap_ne = P.max_ne;
    a.cap_nvu = P.max_nvu;
    a.cap_cs = P.max_cs;
    a.ell = P.ell ? 1 : 0;
    a.eta_u = st->eta;
    a.eta_w = w + L.eta_alt;
    a.U_u = st->U;
    a.U_w = w + L.U_alt;
    const size_t lds = f32 ? P.lds_bytes32 : P.lds_bytes64;
    HIP_TRY(prepare_tile(f32, 0, P.ept, P.block), "batched prepare");

    auto enqueue = [&]() -> se_status {
        for (int32_t c = 0; c < Lmax; ++c) {
            const int32_t cnt = x->list_off[c + 1] - x->list_off[c];
            if (cnt == 0) continue;
            a.chunk = c;
            a.tile_list = x->lists.as<const int32_t>() + x->list_off[c];
            a.ntiles = cnt;
            HIP_TRY(launch_tile(f32, 0, P.ept, P.block, a, cnt, lds, s), "batched launch");
        }
        HIP_TRY(launch_copy_ranges(reinterpret_cast<const uint32_t *>(w + L.eta_alt),
                                   static_cast<uint32_t *>(st->eta),
                                   reinterpret_cast<const uint32_t *>(w + L.U_alt),
                                   static_cast<uint32_t *>(st->U),
                                   x->cpytab.as<const CopyRange>(),
                                   static_cast<int32_t>(x->cpytab_host.size()), cwords, s),
                "batched copy of final states");
        if (st->volume)
            HIP_TRY(launch_vol_reduce_batch(a.vol_part, x->voltab.as<const VolMember>(),
                                            static_cast<int32_t>(n), vrows, st->volume, s),
                    "batched volume");
        return SE_OK;
    };

    if (!use_graph) return enqueue();
    std::vector<uint64_t> key = {
        reinterpret_cast<uint64_t>(st->eta), reinterpret_cast<uint64_t>(st->U),
        reinterpret_cast<uint64_t>(st->Uavg), reinterpret_cast<uint64_t>(st->volume),
        reinterpret_cast<uint64_t>(fo->R), reinterpret_cast<uint64_t>(fo->f),
        reinterpret_cast<uint64_t>(fo->H0), reinterpret_cast<uint64_t>(fo->W),
        reinterpret_cast<uint64_t>(ws), reinterpret_cast<uint64_t>(s),
        static_cast<uint64_t>(p->precision), static_cast<uint64_t>(p->flags)};
    for (auto &gr : x->graphs) {
        if (gr.key == key) {
            HIP_TRY(hipGraphLaunch(gr.x, s), "batched graph launch");
            return SE_OK;
        }
    }
    se_batch::Graph gr;
    gr.key = key;
    HIP_TRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal), "begin capture");
    const se_status es_ = enqueue();
    hipGraph_t g = nullptr;
    const hipError_t ee = hipStreamEndCapture(s, &g);
    if (es_ != SE_OK) {
        if (g) (void)hipGraphDestroy(g);
        return es_;
    }
    if (ee != hipSuccess) return hip_fail(ee, "end capture");
    gr.g = g;
    HIP_TRY(hipGraphInstantiate(&gr.x, g, nullptr, nullptr, 0), "graph instantiate");
    x->graphs.push_back(gr);
    HIP_TRY(hipGraphLaunch(gr.x, s), "batched graph launch");
    return SE_OK;
}


se_status se_batch_set_plan_impl(se_batch *b, int32_t tile, int32_t k_fused, int32_t block) {
    if (b->device < 0) {
        HostTiles ht;
        se_plan_stats_t st;
        SE_TRY(plan_host(batch_members(b), b->voff, b->eoff, tile, k_fused, block, ht, st));
        b->plan_T = tile;
        b->plan_K = k_fused;
        b->plan_block = block;
        return SE_OK;
    }
    DeviceGuard dg(b->device);
    std::unique_ptr<DevTiles> p;
    SE_TRY(make_plan(batch_members(b), b->voff, b->eoff, tile, k_fused, block, p));
    const std::shared_ptr<DevTiles> sp = std::move(p);
    for (se_batch::Exec &x : b->exec) batch_use_plan(b, x, sp);
    b->plan_T = tile;
    b->plan_K = k_fused;
    b->plan_block = block;
    return SE_OK;
}

se_status se_batch_get_plan_impl(const se_batch *b, int32_t *tile, int32_t *k_fused,
                                 int32_t *block) {
    if (tile) *tile = b->plan_T;
    if (k_fused) *k_fused = b->plan_K;
    if (block) *block = b->plan_block;
    return SE_OK;
}

se_status se_batch_plan_stats_impl(const se_batch *b, int32_t tile, int32_t k_fused,
                                   int32_t block, se_plan_stats_t *stats) {
    HostTiles ht;
    return plan_host(batch_members(b), b->voff, b->eoff, tile, k_fused, block, ht, *stats);
}

se_status se_batch_faults_impl(se_batch *b, void *stream, uint32_t *bits) {
    if (b->device < 0) {
        set_error("host-only batch has no fault word");
        return SE_ERR_ARG;
    }
    DeviceGuard dg(b->device);
    const hipStream_t s = static_cast<hipStream_t>(stream);
    HIP_TRY(hipStreamSynchronize(s), "se_check_faults sync");
    uint32_t v = 0;
    HIP_TRY(hipMemcpy(&v, b->faults.p, 4, hipMemcpyDeviceToHost), "se_check_faults copy");
    const uint32_t zero = 0;
    HIP_TRY(hipMemcpy(b->faults.p, &zero, 4, hipMemcpyHostToDevice), "se_check_faults reset");
    *bits = v;
    return SE_OK;
}

}  // extern "C"
