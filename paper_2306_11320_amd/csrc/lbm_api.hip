// Host side of the C ABI declared in include/lbm.h: parameter validation,
// workspace carving, tile tables, HIP graph capture of step sequences,
// diagnostics and state transfer.  All lattice arithmetic runs in the kernels
// of lbm_kernels.hip.
#include "lbm.h"
#include "lbm_internal.hpp"

#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_TRY(expr)                                                                       \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess) return fail(LBM_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

constexpr size_t kAlign = 256;
// Nodes per row boundary: FP32 rows start on 64-byte boundaries of a
// population run, FP64 rows are packed with no gap; rows of lattices that runs
// can step are packed in both (see make_layout).
int row_align(size_t rsz) { return rsz == 8 ? 1 : 16; }
size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

constexpr double W9[9] = {4.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0, 1.0 / 9.0,
                          1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0};

struct Layout {
    int nx, ny, pitch;
    long long plane;        // elements per plane
    size_t pop_off[2];      // byte offsets of time levels A and B
    size_t jprev_off;
    size_t twall_off;       // byte offset of the wall-temperature tables
    int tw_stride;          // entries per side
    int tile_off[lbm::kTileCount], tile_cnt[lbm::kTileCount];
};

size_t real_size(uint32_t prec) { return prec == LBM_FP64 ? sizeof(double) : sizeof(float); }

int validate(const lbm_params& p)
{
    if (p.abi_version != LBM_ABI_VERSION) return fail(LBM_EINVAL, "abi_version %u != %u", p.abi_version, LBM_ABI_VERSION);
    if (p.nx < 3 || p.ny < 3) return fail(LBM_EINVAL, "lattice %ux%u smaller than 3x3", p.nx, p.ny);
    if (p.nx > (uint32_t)INT_MAX || p.ny > (uint32_t)INT_MAX)
        return fail(LBM_EINVAL, "lattice %ux%u: sizes must fit a signed 32-bit integer", p.nx, p.ny);
    // node offsets within a level are 32-bit byte offsets in the kernels
    const uint64_t word = p.precision == LBM_FP64 ? 8 : 4, row = (uint64_t)row_align(word);
    if (((uint64_t)(p.nx + row - 1) / row * row * p.ny + lbm::kBlock - 1) / lbm::kBlock * lbm::kBlock * lbm::kPlanes *
            word >= (1ull << 32))
        return fail(LBM_EINVAL, "lattice too large (%ux%u): a time level must stay below 4 GiB", p.nx, p.ny);
    if (p.precision != LBM_FP64 && p.precision != LBM_FP32_DEV) return fail(LBM_EINVAL, "unknown precision %u", p.precision);
    for (int s = 0; s < 4; ++s)
        if (p.bc[s] > LBM_BC_OUTLET) return fail(LBM_EINVAL, "unknown boundary kind %u on side %d", p.bc[s], s);
    if ((p.bc[0] == LBM_BC_PERIODIC) != (p.bc[1] == LBM_BC_PERIODIC))
        return fail(LBM_EINVAL, "x sides: periodic paired with a non-periodic side");
    if ((p.bc[2] == LBM_BC_PERIODIC) != (p.bc[3] == LBM_BC_PERIODIC))
        return fail(LBM_EINVAL, "y sides: periodic paired with a non-periodic side");
    if (p.grad_mode > 1) return fail(LBM_EINVAL, "grad_mode must be 0 or 1");
    if (p.collision != LBM_BGK && p.collision != LBM_TRT) return fail(LBM_EINVAL, "unknown collision %u", p.collision);
    if (p.force_form != LBM_FORCE_EQ11 && p.force_form != LBM_FORCE_POTENTIAL)
        return fail(LBM_EINVAL, "unknown force_form %u", p.force_form);
    if (p.collision == LBM_TRT && !(p.trt_magic > 0)) return fail(LBM_EINVAL, "trt_magic must be positive");
    if (p.n_bubbles > 4) return fail(LBM_EINVAL, "at most 4 tracked regions");
    if (!(p.rho_l > 0 && p.rho_h > 0)) return fail(LBM_EINVAL, "densities must be positive");
    if (!(p.mu_l > 0 && p.mu_h > 0)) return fail(LBM_EINVAL, "viscosities must be positive (tau_g > 1/2)");
    if (!(p.lambda_l > 0 && p.lambda_h > 0)) return fail(LBM_EINVAL, "conductivities must be positive (tau_h > 1/2)");
    if (!(p.rhocp_l > 0 && p.rhocp_h > 0)) return fail(LBM_EINVAL, "heat capacitances must be positive");
    if (!(p.mobility > 0)) return fail(LBM_EINVAL, "mobility must be positive (tau_phi > 1/2)");
    if (!(p.W > 0)) return fail(LBM_EINVAL, "interface width must be positive");
    // The destination blend of Eq. 28, h_i <- [h*_i + (rho c_p - 1) h_i] / rho c_p,
    // is a convex combination only for rho c_p >= 1: accepted, with a warning
    // left in the thread's message text.
    if (p.rhocp_l < 1.0 || p.rhocp_h < 1.0)
        (void)fail(LBM_OK, "warning: heat capacitance below 1 (%g, %g): the blend of Eq. 28 is not convex",
                   p.rhocp_l, p.rhocp_h);
    return LBM_OK;
}

// Step kernel of a set of lattices: 0 BGK only; 1 some lattice relaxes with
// two relaxation times; 2 some lattice uses the potential form of the
// capillary force.
int step_variant(const lbm_params* ps, int n)
{
    int v = 0;
    for (int k = 0; k < n; ++k) {
        if (ps[k].collision == LBM_TRT && v < 1) v = 1;
        if (ps[k].force_form == LBM_FORCE_POTENTIAL) v = 2;
    }
    return v;
}

// Whether the run tile ids step the lattice in runs (else in its tiles).
bool runs_for(const lbm_params& p, int variant)
{
    return variant < 2 && p.bc[0] == LBM_BC_PERIODIC && p.nx >= (uint32_t)lbm::kRunMinNx &&
           p.nx <= (uint32_t)lbm::kRunMaxNx;
}

Layout make_layout(const lbm_params& p, size_t rsz, int variant, size_t& cursor)
{
    Layout L{};
    L.nx = (int)p.nx;
    L.ny = (int)p.ny;
    // Rows are not padded to whole blocks: a row whose width is not a multiple
    // of the block shares its last block with the next row, so no slot that
    // no node owns is moved (measured on the batched sweep, FP64: 1.15 ->
    // 1.07 ms per step).  In FP32, tiles on rows whose starts are not 8-byte
    // aligned were measured up to 10% slower; there rows start on 64-byte
    // boundaries (at most 15 slots between rows, written as zeros by the
    // step), except in lattices that runs can step: packed rows keep a run's
    // nodes contiguous in memory, so every wavefront of a run reads whole
    // aligned runs of 64 values (width 221: 51.5 -> 45.5 ps per node).
    L.pitch = runs_for(p, variant) ? (int)p.nx : (int)align_up(p.nx, (size_t)row_align(rsz));
    L.plane = (long long)align_up(align_up((size_t)L.pitch * p.ny, lbm::kBlock), kAlign / rsz);
    const size_t level = (size_t)lbm::kPlanes * L.plane * rsz;
    L.pop_off[0] = cursor;
    cursor = align_up(cursor + level, kAlign);
    L.pop_off[1] = cursor;
    cursor = align_up(cursor + level, kAlign);
    L.jprev_off = cursor;
    cursor = align_up(cursor + 2 * (size_t)L.plane * rsz, kAlign);
    // wall temperatures at s = -kTwPad/2 ... max(nx, ny) + kTwPad/2 - 1/2 in
    // steps of 1/2, for each of the four sides
    L.tw_stride = 2 * (L.nx > L.ny ? L.nx : L.ny) + 2 * lbm::kTwPad;
    L.twall_off = cursor;
    cursor = align_up(cursor + 4 * (size_t)L.tw_stride * rsz, kAlign);
    return L;
}

int tiles_of(const Layout& L, const lbm_params& p, int variant, int t)
{
    const int rn = lbm::run_nodes(t);
    if (rn && runs_for(p, variant)) return (int)(((long long)L.nx * L.ny + rn - 1) / rn);
    const int tx = lbm::kTileTX[t], ty = lbm::kTileTY[t];
    return ((L.nx + tx - 1) / tx) * ((L.ny + ty - 1) / ty);
}

template <typename real>
lbm::Inst<real> make_inst(const lbm_params& p, const Layout& L, char* ws)
{
    lbm::Inst<real> I{};
    I.pop[0] = reinterpret_cast<real*>(ws + L.pop_off[0]);
    I.pop[1] = reinterpret_cast<real*>(ws + L.pop_off[1]);
    I.jprev = reinterpret_cast<real*>(ws + L.jprev_off);
    for (int l = 0; l < 2; ++l)
        for (int q = 0; q < 27; ++q) I.qbase[l][q] = I.pop[l] + lbm::pop_index(q, 0);
    I.jbase[0] = I.jprev;
    I.jbase[1] = I.jprev + L.plane;
    I.nx = L.nx;
    I.ny = L.ny;
    I.pitch = L.pitch;
    I.plane = L.plane;
    I.grad_mode = (int)p.grad_mode;
    I.collision = (int)p.collision;
    I.force_form = (int)p.force_form;
    I.trt_magic = (real)p.trt_magic;
    for (int s = 0; s < 4; ++s) I.bc[s] = (int)p.bc[s];
    const double phi0 = p.phi0_dev, T0 = p.T0_dev;
    I.phi0 = (real)phi0;
    I.T0 = (real)T0;
    // xi(phi) = xi_l (1 - phi)/2 + xi_h (1 + phi)/2 = xi_a + xi_b phi
    I.rho_a = (real)(0.5 * (p.rho_l + p.rho_h));
    I.rho_b = (real)(0.5 * (p.rho_h - p.rho_l));
    I.mu_a = (real)(0.5 * (p.mu_l + p.mu_h));
    I.mu_b = (real)(0.5 * (p.mu_h - p.mu_l));
    I.lam_a = (real)(0.5 * (p.lambda_l + p.lambda_h));
    I.lam_b = (real)(0.5 * (p.lambda_h - p.lambda_l));
    I.rcp_a = (real)(0.5 * (p.rhocp_l + p.rhocp_h));
    I.rcp_b = (real)(0.5 * (p.rhocp_h - p.rhocp_l));
    I.sigma_ref = (real)p.sigma_ref;
    I.sigma_T = (real)p.sigma_T;
    I.sigma_TT = (real)p.sigma_TT;
    I.dTref = (real)(T0 - p.T_ref);
    I.W2 = (real)(p.W * p.W);
    I.pref = (real)(3.0 * std::sqrt(2.0) * p.W / 4.0);
    I.inv_W2 = (real)(1.0 / (p.W * p.W));
    I.inv_s2W = (real)(1.0 / (std::sqrt(2.0) * p.W));
    const double tau_phi = 0.5 + 3.0 * p.mobility;  // M = c_s^2 (tau_phi - 1/2)
    I.inv_tau_phi = (real)(1.0 / tau_phi);
    I.fac_phi = (real)(1.0 - 0.5 / tau_phi);
    I.Gx = (real)p.Gx;
    I.Gy = (real)p.Gy;
    I.twall = reinterpret_cast<const real*>(ws + L.twall_off);
    I.tw_stride = L.tw_stride;
    I.u_in = (real)p.u_in_mean;
    I.phi_in_d = (real)(p.phi_in - phi0);
    I.T_in_d = (real)(p.T_in - T0);
    return I;
}

// Wall temperatures relative to T0 at s = (j - kTwPad) / 2 along each side,
// T_w(s) = Tw_mean + Tw_amp cos(Tw_k s) + Tw_slope s, for the boundary rules
// of the step kernel; copied into the lattice's table (the stream is
// synchronized before the host copy is freed).
template <typename real>
hipError_t put_wall_table(const lbm_params& p, const Layout& L, char* ws, hipStream_t s)
{
    std::vector<real> t(4 * (size_t)L.tw_stride);
    for (int side = 0; side < 4; ++side)
        for (int j = 0; j < L.tw_stride; ++j) {
            const double x = 0.5 * (j - lbm::kTwPad);
            const double Tw = p.Tw_mean[side] + p.Tw_amp[side] * std::cos(p.Tw_k[side] * x) + p.Tw_slope[side] * x;
            t[(size_t)side * L.tw_stride + j] = (real)(Tw - p.T0_dev);
        }
    hipError_t e = hipMemcpyAsync(ws + L.twall_off, t.data(), t.size() * sizeof(real), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    return e;
}

uint64_t params_hash(const std::vector<lbm_params>& ps)
{
    uint64_t h = 1469598103934665603ull;  // FNV-1a
    for (const auto& p : ps) {
        const unsigned char* b = reinterpret_cast<const unsigned char*>(&p);
        for (size_t i = 0; i < sizeof(p); ++i) {
            h ^= b[i];
            h *= 1099511628211ull;
        }
    }
    return h;
}

}  // namespace

struct lbm_ctx {
    uint32_t prec = 0;
    int n = 0;
    int tile = 0;
    int graph_steps = 64;
    int grid = 0;
    // step kernel: 0 BGK only; 1 some lattice relaxes with two relaxation
    // times; 2 some lattice uses the potential form of the capillary force
    int variant = 0;
    // some lattice is stepped in runs by the run tile ids (else those ids
    // repeat the tiles of their TX x TY shape)
    bool has_runs = false;
    hipStream_t stream = nullptr;
    char* ws = nullptr;
    size_t ws_bytes = 0;
    std::vector<lbm_params> params;
    std::vector<Layout> lay;
    std::vector<char> h_insts;  // host copy of the device Inst array
    void* d_insts = nullptr;
    lbm::Tile* d_tiles[lbm::kTileCount] = {};
    int ntiles[lbm::kTileCount] = {};
    bool cut[lbm::kTileCount] = {};  // the table holds interior tiles that are not whole
    double* d_partials = nullptr;
    double* d_result = nullptr;
    int64_t step = 0;
    hipGraphExec_t gexec = nullptr;
    int gexec_steps = 0;
    std::vector<double> bx, by;  // per instance, 4 tracked centroids
};

namespace {

size_t inst_size(uint32_t prec) { return prec == LBM_FP64 ? sizeof(lbm::Inst<double>) : sizeof(lbm::Inst<float>); }

// Carves the workspace; fills layouts and the offsets of the shared tables.
size_t plan(const lbm_params* ps, int n, std::vector<Layout>* lay, size_t* off_insts, size_t off_tiles[],
            size_t* off_partials, size_t* off_result)
{
    const uint32_t prec = ps[0].precision;
    const size_t rsz = real_size(prec);
    size_t cursor = 0;
    std::vector<Layout> L;
    int tot[lbm::kTileCount] = {};
    const int variant = step_variant(ps, n);
    for (int k = 0; k < n; ++k) {
        Layout l = make_layout(ps[k], rsz, variant, cursor);
        for (int t = 0; t < lbm::kTileCount; ++t) {
            l.tile_off[t] = tot[t];
            l.tile_cnt[t] = tiles_of(l, ps[k], variant, t);
            tot[t] += l.tile_cnt[t];
        }
        L.push_back(l);
    }
    *off_insts = cursor;
    cursor = align_up(cursor + (size_t)n * inst_size(prec), kAlign);
    int maxt = 1;
    for (int t = 0; t < lbm::kTileCount; ++t) {
        off_tiles[t] = cursor;
        cursor = align_up(cursor + (size_t)tot[t] * sizeof(lbm::Tile), kAlign);
        if (tot[t] > maxt) maxt = tot[t];
    }
    *off_partials = cursor;
    cursor = align_up(cursor + (size_t)maxt * lbm::D_COUNT * sizeof(double), kAlign);
    *off_result = cursor;
    cursor = align_up(cursor + lbm::D_COUNT * sizeof(double), kAlign);
    if (lay) *lay = L;
    return cursor;
}

void drop_graph(lbm_ctx* c)
{
    if (c->gexec) {
        (void)hipGraphExecDestroy(c->gexec);
        c->gexec = nullptr;
        c->gexec_steps = 0;
    }
}

int launch_one(lbm_ctx* c, int src)
{
    HIP_TRY(lbm::launch_step((int)c->prec, c->tile, c->d_insts, c->d_tiles[c->tile], c->ntiles[c->tile],
                             c->cut[c->tile], c->grid, src, c->variant, c->stream));
    return LBM_OK;
}

int capture(lbm_ctx* c)
{
    drop_graph(c);
    hipGraph_t g = nullptr;
    HIP_TRY(hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
    int rc = LBM_OK;
    for (int s = 0; s < c->graph_steps && rc == LBM_OK; ++s) rc = launch_one(c, s & 1);
    hipError_t e = hipStreamEndCapture(c->stream, &g);
    if (rc != LBM_OK) {
        if (g) (void)hipGraphDestroy(g);
        return rc;
    }
    if (e != hipSuccess) return fail(LBM_EHIP, "hipStreamEndCapture: %s", hipGetErrorString(e));
    e = hipGraphInstantiate(&c->gexec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) return fail(LBM_EHIP, "hipGraphInstantiate: %s", hipGetErrorString(e));
    c->gexec_steps = c->graph_steps;
    return LBM_OK;
}

// Tile of a new context (the tile tables exist).  Figures: us per step; r = nx
// mod 64.  Two things count besides the columns a shape leaves idle:
// * a last column of tiles with at most 8 nodes a wavefront (4 columns of a 32-wide
//   tile, 8 of a wider one) makes a step 1 to 2 us longer, of at most 16 about
//   0.3, in every precision and form (the cause was not found: the loads and
//   stores are those of any cut tile);
// * a launch of at most one workgroup per CU takes the time of its slowest tile, a
//   larger one that of the CU with the most.
// The choices:
// * batches whose populations outgrow the 256 MB Infinity Cache, all of lattices
//   that runs can step: runs of 512 nodes in FP32 (droplets of width 128-256:
//   290 MB 66 against 82 with 64 x 4 tiles, 890 MB 191 against 236; 180 MB 34.4
//   against 31.1), of 256 in FP64 (360 MB 89.0 against 90.7, 1.8 GB 397 against
//   430; 190 MB 42.0 against 36.4);
// * 32 x 8 where 64-wide tiles leave half a tile of every row idle.  FP64, r in 1 ..
//   32: if a CU gets fewer tiles than of 64 x 4, and at most four (a sixteenth of
//   the CUs with one more does not count): 200 x 800 15.3 against 19.6, 160 x 1200 16.3
//   against 19.1, 352 x 704 20.9 against 22.2, 258 x 900 21.2 against 21.9, 333 x 555
//   17.3 against 17.9, 390 x 600 21.0 against 22.4; as many: 260 x 700 20.8 against 17.6, 270 x
//   700 19.2 against 18.4, 150 x 1300 19.1 against 18.0, 390 x 1600 64.7 against 60.9; more
//   than four: 280 x 1100 26.3 against 25.5, 340 x 1200 32.1 against 30.9, 352 x 1408
//   37.3 against 36.5 (64 x 4 has a BGK kernel of its own for cut tiles there; TRT 260 x
//   1040 25.6 against 29.0).  Up to six columns of 64 also if a CU gets at most two
//   (160 x 320 7.8 against 8.7, 140 x 560 10.9 against 11.2; 130 x 500 11.3 both), with TRT
//   if it gets fewer, however many, and if r is in 5 .. 8 (200 x 900 TRT 20.2 against 22.4, BGK 18.9
//   against 19.5).  FP32, r = 32 up to six columns: 32 x 8 tiles are then whole
//   (160 x 320 6.1 against 6.5, 288 x 900 11.7 against 13.6, 352 x 1408 19.9 against 20.6;
//   416 x 1600 25.2 against 25.1; 221 x 884 11.9 against 10.3).  The potential form,
//   whose second ring is smaller around 32 x 8 tiles, takes them at any width: FP32,
//   r = 32: 352 x 704 14.3 against 19.1, 480 x 1600 37.3 against 40.8, 544 x 1600 42.5
//   against 43.8; FP64, r in 1 .. 32: 221 x 884 24.8 against 27.0, 480 x 1600 89.6 against
//   97.7, 600 x 1200 87.9 against 87.6; and in FP64 up to six columns also for r above
//   32 (104 x 256 10.1 against 10.6, 250 x 500 15.2 against 15.7, 300 x 256 13.5 against
//   14.3; 432 x 900 43.6 against 43.2, 440 x 1600 87.0 against 86.7) except 33 .. 36, a
//   last column of 4 nodes and less (100 x 400 13.0 against 11.1, 36 x 256 11.9 against
//   10.1, 292 x 900 32.9 against 32.4, 355 x 700 33.7 against 31.3; but 225 x 900 26.2
//   against 27.1);
// * FP64: else 64 x 4;
// * FP32: 64 x 8 when one round of resident workgroups covers every tile
//   (fewer ring reloads; 256 x 1024 +1.8%), else 64 x 4 (later rounds overlap
//   earlier ones; 512 x 2048 +2.3%), and where those are at most one per CU
//   (64 x 32 5.6 against 5.8, 128 x 512 6.28 against 6.32; 140 x 560 7.5 against
//   7.0) unless their last column has 16 nodes or fewer (130 x 260 7.7
//   against 7.0, 200 x 256 8.5 against 6.8, 140 x 280 6.7 against 6.4);
// * FP32 with the potential form in one round: 128 x 4 instead of 64 x 8 where
//   rows do not start on whole lines (nx not whole in 16: a 128-wide tile reads five lines for
//   four, a 64-wide three for two), as long as it needs no more workgroups per CU and
//   its last column has more than 8 nodes (221 x 884 12.8 against 13.5, 200 x 600
//   11.3 against 12.4, 140 x 280 8.6 against 9.0, 140 x 700 10.5 against 11.2; but
//   more per CU: 140 x 560 10.3 against 9.5, 140 x 1200 17.4 against 12.6, 270 x 700 18.3
//   against 12.9; few nodes: 130 x 260 10.1 against 9.1); where they do, beyond one
//   workgroup per CU only (208 x 600 11.1 against 11.4, 240 x 900 13.0 against 13.3;
//   112 x 256 8.2 against 7.9).
int default_tile(const lbm_ctx* c)
{
    const bool fp64 = c->prec == LBM_FP64, pot = c->variant == 2;
    size_t bytes = 0;
    bool runs = c->n > 1, halves = true, few8 = true, six_all = true, few16 = false, wide = true, lines = false;
    for (int k = 0; k < c->n; ++k) {
        const int nx = c->lay[k].nx, r = nx % 64, last = nx % 128;
        const bool six = nx <= 6 * 64;
        bytes += 2 * (size_t)lbm::kPlanes * c->lay[k].plane * real_size(c->prec);
        runs = runs && runs_for(c->params[k], c->variant);
        six_all = six_all && six;
        if (fp64) halves = halves && ((r >= 1 && r <= 32) || (pot && r > 36 && six));
        else halves = halves && r == 32 && (pot || six);
        few8 = few8 && r >= 5 && r <= 8;
        few16 = few16 || (r >= 1 && r <= 16);
        wide = wide && nx % 32 != 0 && !(last >= 1 && last <= 8);
        lines = lines || nx % 16 == 0;
    }
    if (runs && bytes > ((size_t)256 << 20)) return fp64 ? 7 : 6;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    auto per_cu = [&](int t, int slack = 0) { return (c->ntiles[t] - slack + cus - 1) / cus; };
    if (fp64 && !pot) {
        const int p = per_cu(2, cus / 16);
        const bool fewer = p < per_cu(0) && (p <= 4 || (six_all && c->variant == 1));
        halves = halves && (fewer || (six_all && (few8 || per_cu(2) <= 2)));
    }
    if (halves) return 2;
    if (fp64) return 0;
    if (!pot && !few16 && c->ntiles[0] <= cus) return 0;
    auto resident = [&](int t) {  // whether one round holds every tile of shape t
        int n = 0;
        return lbm::step_occupancy((int)c->prec, t, c->variant, &n) != hipSuccess || n < 1 || c->ntiles[t] <= n * cus;
    };
    if (!resident(3)) return 0;
    return pot && wide && per_cu(5) <= per_cu(3) && !(lines && per_cu(3) == 1) && resident(5) ? 5 : 3;
}

int init_common(int n, const lbm_params* ps, const double* const* phi0, const double* const* ux0,
                const double* const* uy0, const double* const* T0, void* d_ws, size_t ws_bytes, void* stream,
                lbm_ctx** out)
{
    if (!out) return fail(LBM_EINVAL, "out is NULL");
    *out = nullptr;
    if (n < 1 || !ps || !phi0 || !ux0 || !uy0 || !T0 || !d_ws) return fail(LBM_EINVAL, "NULL argument or n < 1");
    if (reinterpret_cast<uintptr_t>(d_ws) % kAlign) return fail(LBM_EINVAL, "workspace not 256-byte aligned");
    for (int k = 0; k < n; ++k) {
        int rc = validate(ps[k]);
        if (rc) return rc;
        if (ps[k].precision != ps[0].precision) return fail(LBM_EINVAL, "lattice %d: precision differs", k);
        if (!phi0[k] || !ux0[k] || !uy0[k] || !T0[k]) return fail(LBM_EINVAL, "lattice %d: NULL field", k);
    }
    std::vector<Layout> lay;
    size_t off_insts, off_tiles[lbm::kTileCount], off_part, off_res;
    const size_t need = plan(ps, n, &lay, &off_insts, off_tiles, &off_part, &off_res);
    if (ws_bytes < need) return fail(LBM_ENOSPACE, "workspace %zu bytes < %zu needed", ws_bytes, need);

    lbm_ctx* c = new (std::nothrow) lbm_ctx();
    if (!c) return fail(LBM_EINVAL, "out of host memory");
    c->prec = ps[0].precision;
    c->n = n;
    c->stream = static_cast<hipStream_t>(stream);
    c->ws = static_cast<char*>(d_ws);
    c->ws_bytes = ws_bytes;
    c->params.assign(ps, ps + n);
    c->variant = step_variant(ps, n);
    for (int k = 0; k < n; ++k) c->has_runs = c->has_runs || runs_for(ps[k], c->variant);
    c->lay = lay;
    c->d_insts = c->ws + off_insts;
    c->d_partials = reinterpret_cast<double*>(c->ws + off_part);
    c->d_result = reinterpret_cast<double*>(c->ws + off_res);
    c->bx.assign(4 * (size_t)n, 0.0);
    c->by.assign(4 * (size_t)n, 0.0);
    const size_t isz = inst_size(c->prec);
    c->h_insts.resize((size_t)n * isz);
    for (int k = 0; k < n; ++k) {
        if (c->prec == LBM_FP64) {
            auto I = make_inst<double>(ps[k], lay[k], c->ws);
            std::memcpy(c->h_insts.data() + k * isz, &I, isz);
        } else {
            auto I = make_inst<float>(ps[k], lay[k], c->ws);
            std::memcpy(c->h_insts.data() + k * isz, &I, isz);
        }
        for (int b = 0; b < 4; ++b) {
            c->bx[4 * k + b] = ps[k].bubble_x[b];
            c->by[4 * k + b] = ps[k].bubble_y[b];
        }
    }
    auto bail = [&](int rc) {
        delete c;
        return rc;
    };
    hipError_t e = hipMemcpyAsync(c->d_insts, c->h_insts.data(), c->h_insts.size(), hipMemcpyHostToDevice, c->stream);
    if (e != hipSuccess) return bail(fail(LBM_EHIP, "copy of lattice constants: %s", hipGetErrorString(e)));
    for (int k = 0; k < n; ++k) {
        e = c->prec == LBM_FP64 ? put_wall_table<double>(ps[k], lay[k], c->ws, c->stream)
                                : put_wall_table<float>(ps[k], lay[k], c->ws, c->stream);
        if (e != hipSuccess) return bail(fail(LBM_EHIP, "copy of wall temperatures: %s", hipGetErrorString(e)));
    }
    // tile tables for every compiled shape, ordered by lattice then row-major
    // tiles (or runs in node order)
    for (int t = 0; t < lbm::kTileCount; ++t) {
        std::vector<lbm::Tile> tl;
        for (int k = 0; k < n; ++k) {
            const int tx = lbm::kTileTX[t], ty = lbm::kTileTY[t];
            const int nx = lay[k].nx, ny = lay[k].ny;
            const int rn = lbm::run_nodes(t);
            if (rn && runs_for(ps[k], c->variant)) {
                const long long nn = (long long)nx * ny;
                for (long long n0 = 0; n0 < nn; n0 += rn) {
                    const long long last = (n0 + rn < nn ? n0 + rn : nn) - 1;
                    // interior: no node of the first or last row
                    const bool inner = n0 / nx >= 1 && last / nx <= ny - 2;
                    tl.push_back(lbm::Tile{k, (int)n0, 0, lbm::kTileRun | (inner ? lbm::kTileInterior : 0)});
                }
                continue;
            }
            const bool px = ps[k].bc[0] == LBM_BC_PERIODIC, py = ps[k].bc[2] == LBM_BC_PERIODIC;
            for (int y = 0; y < ny; y += ty)
                for (int x = 0; x < nx; x += tx) {
                    const bool whole = x + tx <= nx && y + ty <= ny;
                    // wrap-only: in a periodic direction one wrap must reach
                    // every point of the tile and its ring (tile no longer
                    // than the lattice)
                    const bool inx = px ? (nx >= 3 && tx <= nx) : (x >= 1 && x + tx <= nx - 1);
                    const bool iny = py ? (ny >= 3 && ty <= ny) : (y >= 1 && y + ty <= ny - 1);
                    // whether the tile or its ring crosses a side that is neither periodic nor a wall
                    const bool cross[4] = {x == 0, x + tx >= nx, y == 0, y + ty >= ny};
                    bool walls = true;
                    for (int s = 0; s < 4; ++s)
                        if (cross[s] && (ps[k].bc[s] == LBM_BC_INLET || ps[k].bc[s] == LBM_BC_OUTLET)) walls = false;
                    tl.push_back(lbm::Tile{k, x, y, (inx && iny ? lbm::kTileInterior : 0) |
                                                        (whole ? lbm::kTileWhole : 0) | (walls ? lbm::kTileWalls : 0)});
                }
        }
        c->d_tiles[t] = reinterpret_cast<lbm::Tile*>(c->ws + off_tiles[t]);
        c->ntiles[t] = (int)tl.size();
        for (const lbm::Tile& tile : tl)
            if ((tile.flags & (lbm::kTileInner | lbm::kTileRun)) == lbm::kTileInterior) c->cut[t] = true;
        e = hipMemcpyAsync(c->d_tiles[t], tl.data(), tl.size() * sizeof(lbm::Tile), hipMemcpyHostToDevice, c->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) return bail(fail(LBM_EHIP, "copy of tile table: %s", hipGetErrorString(e)));
    }
    c->tile = default_tile(c);
    // equilibrium populations: fields are staged in the lattice's level B
    for (int k = 0; k < n; ++k) {
        const size_t nn = (size_t)lay[k].nx * lay[k].ny;
        double* staged = reinterpret_cast<double*>(c->ws + lay[k].pop_off[1]);
        const double* src[4] = {phi0[k], ux0[k], uy0[k], T0[k]};
        for (int q = 0; q < 4; ++q) {
            e = hipMemcpyAsync(staged + q * nn, src[q], nn * sizeof(double), hipMemcpyHostToDevice, c->stream);
            if (e != hipSuccess) return bail(fail(LBM_EHIP, "copy of initial fields: %s", hipGetErrorString(e)));
        }
        lbm::InitArgs ia{ps[k].phi0_dev, ps[k].T0_dev, 0.5 * (ps[k].rho_l + ps[k].rho_h),
                         0.5 * (ps[k].rho_h - ps[k].rho_l), 0, 0};
        e = lbm::launch_init((int)c->prec, static_cast<char*>(c->d_insts) + k * isz, (long long)nn, staged, ia, 0,
                             c->stream);
        if (e != hipSuccess) return bail(fail(LBM_EHIP, "init kernel: %s", hipGetErrorString(e)));
        // the staging must be consumed before the next lattice reuses memory
        e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) return bail(fail(LBM_EHIP, "init: %s", hipGetErrorString(e)));
    }
    // (phi u) of the previous level := (phi u) now, so the first time derivative is zero
    constexpr int ft = lbm::kMacroTile;
    e = lbm::launch_fields((int)c->prec, ft, c->d_insts, c->d_tiles[ft], c->ntiles[ft], 0, nullptr,
                           nullptr, nullptr, nullptr, nullptr, 0, 1, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return bail(fail(LBM_EHIP, "initial (phi u): %s", hipGetErrorString(e)));
    *out = c;
    return LBM_OK;
}

// Tile of the field kernel on one lattice: 64 x 4, but in FP32 64 x 8 where those
// are at most two per CU and either the potential form has its second ring to
// load (221 x 884 8.9 -> 7.9 us, 256 x 1024 8.5 -> 7.7, 100 x 400 6.5 -> 6.2; beyond, 400 x
// 1600 19.6 against 19.8) or 64 x 4 tiles are more than three per CU (221 x 884 6.6 -> 6.3,
// 256 x 1024 6.3 -> 6.0; 250 x 700, 700 tiles, 6.1 against 6.2; beyond, 512 x 2048 20.7
// against 21.7).  FP64: 64 x 4 (221 x 884 11.2 against 12.0).
int field_tile(const lbm_ctx* c, const Layout& L)
{
    const bool fewer = c->variant == 2 || L.tile_cnt[lbm::kMacroTile] > 3 * 256;
    return c->prec == LBM_FP32_DEV && fewer && L.tile_cnt[lbm::kFieldTile] <= 2 * 256 ? lbm::kFieldTile : lbm::kMacroTile;
}

int check_instance(const lbm_ctx* c, int k)
{
    if (!c) return fail(LBM_EINVAL, "context is NULL");
    if (k < 0 || k >= c->n) return fail(LBM_EINVAL, "instance %d out of range [0, %d)", k, c->n);
    return LBM_OK;
}

}  // namespace

extern "C" {

size_t lbm_workspace_bytes(const lbm_params* p) { return lbm_workspace_bytes_batch(p, 1); }

size_t lbm_workspace_bytes_batch(const lbm_params* p, int n)
{
    if (!p || n < 1) return 0;
    for (int k = 0; k < n; ++k)
        if (validate(p[k]) != LBM_OK) return 0;
    size_t a, b[lbm::kTileCount], d, e;
    return plan(p, n, nullptr, &a, b, &d, &e);
}

int lbm_init(const lbm_params* p, const double* phi0, const double* ux0, const double* uy0, const double* T0,
             void* d_workspace, size_t ws_bytes, void* hip_stream, lbm_ctx** out)
{
    return init_common(1, p, &phi0, &ux0, &uy0, &T0, d_workspace, ws_bytes, hip_stream, out);
}

int lbm_init_batch(int n, const lbm_params* params, const double* const* phi0, const double* const* ux0,
                   const double* const* uy0, const double* const* T0, void* d_workspace, size_t ws_bytes,
                   void* hip_stream, lbm_ctx** out)
{
    return init_common(n, params, phi0, ux0, uy0, T0, d_workspace, ws_bytes, hip_stream, out);
}

int lbm_instances(const lbm_ctx* c) { return c ? c->n : 0; }

int lbm_step(lbm_ctx* c, int64_t n)
{
    if (!c) return fail(LBM_EINVAL, "context is NULL");
    if (n < 0) return fail(LBM_EINVAL, "negative step count");
    while (n > 0) {
        if (c->graph_steps > 0 && (c->step & 1) == 0 && n >= c->graph_steps) {
            if (!c->gexec) {
                int rc = capture(c);
                if (rc) return rc;
            }
            HIP_TRY(hipGraphLaunch(c->gexec, c->stream));
            c->step += c->gexec_steps;
            n -= c->gexec_steps;
        } else {
            int rc = launch_one(c, (int)(c->step & 1));
            if (rc) return rc;
            c->step += 1;
            n -= 1;
        }
    }
    return LBM_OK;
}

int lbm_fields_instance(lbm_ctx* c, int instance, void* d_phi, void* d_ux, void* d_uy, void* d_T, void* d_p,
                        int out_dtype)
{
    int rc = check_instance(c, instance);
    if (rc) return rc;
    if (out_dtype != LBM_OUT_F64 && out_dtype != LBM_OUT_F32) return fail(LBM_EINVAL, "unknown output dtype");
    const Layout& L = c->lay[instance];
    const int ft = field_tile(c, L);
    HIP_TRY(lbm::launch_fields((int)c->prec, ft, c->d_insts, c->d_tiles[ft] + L.tile_off[ft],
                               L.tile_cnt[ft], (int)(c->step & 1), d_phi, d_ux, d_uy, d_T, d_p,
                               out_dtype == LBM_OUT_F32, 0, c->stream));
    return LBM_OK;
}

int lbm_reinit_fields(lbm_ctx* c, int instance, const void* d_phi, const void* d_ux, const void* d_uy,
                      const void* d_T, const void* d_p, int in_dtype, int mode)
{
    int rc = check_instance(c, instance);
    if (rc) return rc;
    if (!d_phi || !d_ux || !d_uy || !d_T) return fail(LBM_EINVAL, "NULL field");
    if (in_dtype != LBM_OUT_F64 && in_dtype != LBM_OUT_F32) return fail(LBM_EINVAL, "unknown input dtype");
    if (mode != LBM_REINIT_EQUILIBRIUM && mode != LBM_REINIT_SHIFT) return fail(LBM_EINVAL, "unknown reinit mode");
    const Layout& L = c->lay[instance];
    const lbm_params& p = c->params[instance];
    const long long n = (long long)L.nx * L.ny;
    const int lvl = (int)(c->step & 1);
    const size_t isz = inst_size(c->prec);
    const void* inst = static_cast<char*>(c->d_insts) + instance * isz;
    const int ft = field_tile(c, L);
    const lbm::Tile* tiles = c->d_tiles[ft] + L.tile_off[ft];
    // the other time level is free until the next step: it holds the staged
    // new fields (planes 0..4) and, when shifting, the current ones (5..9)
    double* staged = reinterpret_cast<double*>(c->ws + L.pop_off[lvl ^ 1]);
    HIP_TRY(lbm::launch_stage(d_phi, d_ux, d_uy, d_T, d_p, in_dtype == LBM_OUT_F32, n, staged, c->stream));
    if (mode == LBM_REINIT_SHIFT)
        HIP_TRY(lbm::launch_fields((int)c->prec, ft, c->d_insts, tiles, L.tile_cnt[ft], lvl, staged + 5 * n,
                                   staged + 6 * n, staged + 7 * n, staged + 8 * n, staged + 9 * n, 0, 0, c->stream));
    lbm::InitArgs ia{p.phi0_dev, p.T0_dev, 0.5 * (p.rho_l + p.rho_h), 0.5 * (p.rho_h - p.rho_l), d_p != nullptr,
                     mode == LBM_REINIT_SHIFT};
    HIP_TRY(lbm::launch_init((int)c->prec, inst, n, staged, ia, lvl, c->stream));
    HIP_TRY(lbm::launch_fields((int)c->prec, ft, c->d_insts, tiles, L.tile_cnt[ft], lvl, nullptr, nullptr,
                               nullptr, nullptr, nullptr, 0, 1, c->stream));
    return LBM_OK;
}

int lbm_fields(lbm_ctx* c, void* d_phi, void* d_ux, void* d_uy, void* d_T, void* d_p, int out_dtype)
{
    return lbm_fields_instance(c, 0, d_phi, d_ux, d_uy, d_T, d_p, out_dtype);
}

int lbm_diagnostics_instance(lbm_ctx* c, int instance, lbm_diag* out)
{
    int rc = check_instance(c, instance);
    if (rc) return rc;
    if (!out) return fail(LBM_EINVAL, "out is NULL");
    const Layout& L = c->lay[instance];
    const lbm_params& p = c->params[instance];
    lbm::DiagArgs a{};
    a.n_bubbles = (int)p.n_bubbles;
    for (int b = 0; b < 4; ++b) {
        a.bx[b] = c->bx[4 * instance + b];
        a.by[b] = c->by[4 * instance + b];
    }
    a.rcp_a = 0.5 * (p.rhocp_l + p.rhocp_h);
    a.rcp_b = 0.5 * (p.rhocp_h - p.rhocp_l);
    constexpr int ft = lbm::kMacroTile;
    HIP_TRY(lbm::launch_diag((int)c->prec, c->d_insts, c->d_tiles[ft] + L.tile_off[ft],
                             L.tile_cnt[ft], (int)(c->step & 1), a, c->d_partials, c->d_result, c->stream));
    double r[lbm::D_COUNT];
    HIP_TRY(hipMemcpyAsync(r, c->d_result, sizeof(r), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    std::memset(out, 0, sizeof(*out));
    out->step = c->step;
    out->mass_phi = r[lbm::D_MASS];
    out->vol_light = r[lbm::D_VOL];
    out->heat = r[lbm::D_HEAT];
    out->sum_neg = r[lbm::D_SNEG];
    out->max_u = r[lbm::D_MAXU];
    out->n_nonfinite = (int64_t)r[lbm::D_NONFIN];
    out->n_neg = (int64_t)r[lbm::D_NNEG];
    if (out->sum_neg != 0.0) {
        out->u_r = r[lbm::D_SUY] / out->sum_neg;
        out->ux_r = r[lbm::D_SUX] / out->sum_neg;
        out->xc = r[lbm::D_SX] / out->sum_neg;
        out->yc = r[lbm::D_SY] / out->sum_neg;
    }
    for (int b = 0; b < (int)p.n_bubbles; ++b) {
        const double* q = r + lbm::D_BUB + 5 * b;
        out->bub_sum[b] = q[0];
        if (q[0] != 0.0) {
            out->bub_x[b] = q[1] / q[0];
            out->bub_y[b] = q[2] / q[0];
            out->bub_ux[b] = q[3] / q[0];
            out->bub_uy[b] = q[4] / q[0];
            c->bx[4 * instance + b] = out->bub_x[b];
            c->by[4 * instance + b] = out->bub_y[b];
        } else {
            out->bub_x[b] = c->bx[4 * instance + b];
            out->bub_y[b] = c->by[4 * instance + b];
        }
    }
    if (out->n_nonfinite > 0 || !(out->max_u <= 0.5))
        return fail(LBM_EUNSTABLE, "unstable: %lld non-finite nodes, max |u| = %g", (long long)out->n_nonfinite,
                    out->max_u);
    return LBM_OK;
}

int lbm_diagnostics(lbm_ctx* c, lbm_diag* out) { return lbm_diagnostics_instance(c, 0, out); }

int lbm_destroy(lbm_ctx* c)
{
    if (!c) return LBM_OK;
    hipError_t e = hipStreamSynchronize(c->stream);
    drop_graph(c);
    delete c;
    if (e != hipSuccess) return fail(LBM_EHIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
    return LBM_OK;
}

const char* lbm_last_error(void) { return g_err.c_str(); }

// ---- state transfer ----

namespace {
// One of f, g, h (q0 = kF, kG, kH) or jprev (q0 < 0) of a lattice between its
// level `lvl` and a host array, through the other time level as FP64 device
// scratch (free until the next step; 9 FP64 values per node fit the 27 words of
// a level in either precision).
int transfer(lbm_ctx* c, int instance, int lvl, int q0, double* host, int in)
{
    const Layout& L = c->lay[instance];
    const lbm_params& p = c->params[instance];
    const long long nn = (long long)L.nx * L.ny;
    const size_t bytes = (size_t)nn * (q0 < 0 ? 2 : 9) * sizeof(double);
    static_assert(9 * sizeof(double) <= lbm::kPlanes * sizeof(float), "scratch level");
    double* buf = reinterpret_cast<double*>(c->ws + L.pop_off[lvl ^ 1]);
    const void* inst = static_cast<char*>(c->d_insts) + instance * inst_size(c->prec);
    lbm::StateShift sh{};
    for (int k = 0; k < 9; ++k) sh.v[k] = W9[k] * (q0 == lbm::kF ? p.phi0_dev : (q0 == lbm::kH ? p.T0_dev : 0.0));
    if (in) HIP_TRY(hipMemcpyAsync(buf, host, bytes, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(lbm::launch_state((int)c->prec, inst, nn, lvl, q0, sh, buf, in, c->stream));
    if (!in) HIP_TRY(hipMemcpyAsync(host, buf, bytes, hipMemcpyDeviceToHost, c->stream));
    return LBM_OK;
}

// Lattices of at most this many nodes are transferred whole and converted on the
// host instead: two copies each way instead of four with a kernel each (set and
// get in FP32: 24 x 24 95 us against 205, 64 x 32 160 against 245, 64 x 64 246 against
// 279).
constexpr long long kSmallState = 4096;

int transfer_small(lbm_ctx* c, int instance, int lvl, double* const (&pops)[3], double* jprev, int in)
{
    const Layout& L = c->lay[instance];
    const lbm_params& p = c->params[instance];
    const size_t rsz = real_size(c->prec), plane_b = (size_t)L.plane * rsz, level_b = lbm::kPlanes * plane_b;
    const bool any = pops[0] || pops[1] || pops[2], all = pops[0] && pops[1] && pops[2];
    const std::unique_ptr<char[]> lev(new (std::nothrow) char[level_b + 2 * plane_b]());
    if (!lev) return fail(LBM_EINVAL, "out of host memory");
    char *jp = lev.get() + level_b, *d_lev = c->ws + L.pop_off[lvl], *d_jp = c->ws + L.jprev_off;
    // populations that are not given keep their values
    if (any && !(in && all)) HIP_TRY(hipMemcpyAsync(lev.get(), d_lev, level_b, hipMemcpyDeviceToHost, c->stream));
    if (jprev && !in) HIP_TRY(hipMemcpyAsync(jp, d_jp, 2 * plane_b, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    // one plane of a host array; at(n): its element in dev of node number n
    auto plane = [&](char* dev, auto at, double* host, double sh) {
        for (int j = 0; j < L.ny; ++j)
            for (int i = 0; i < L.nx; ++i, ++host) {
                const size_t e = (size_t)at((long long)j * L.pitch + i);
                if (c->prec == LBM_FP64) {
                    double& v = reinterpret_cast<double*>(dev)[e];
                    if (in) v = *host - sh;
                    else *host = v + sh;
                } else {
                    float& v = reinterpret_cast<float*>(dev)[e];
                    if (in) v = (float)(*host - sh);
                    else *host = (double)v + sh;
                }
            }
    };
    const double rest[3] = {p.phi0_dev, 0.0, p.T0_dev};
    const size_t nn = (size_t)L.nx * L.ny;
    for (int q = 0; q < 3; ++q)
        for (int k = 0; pops[q] && k < 9; ++k)
            plane(lev.get(), [&](long long n) { return lbm::pop_index(9 * q + k, n); }, pops[q] + k * nn, W9[k] * rest[q]);
    for (int q = 0; jprev && q < 2; ++q)
        plane(jp + q * plane_b, [](long long n) { return n; }, jprev + q * nn, 0.0);
    if (in && any) HIP_TRY(hipMemcpyAsync(d_lev, lev.get(), level_b, hipMemcpyHostToDevice, c->stream));
    if (in && jprev) HIP_TRY(hipMemcpyAsync(d_jp, jp, 2 * plane_b, hipMemcpyHostToDevice, c->stream));
    if (in) HIP_TRY(hipStreamSynchronize(c->stream));
    return LBM_OK;
}

// The given ones of f, g, h and (phi u) between level `lvl` and host arrays;
// synchronizes.
int transfer_state(lbm_ctx* c, int instance, int lvl, double* f, double* g, double* h, double* jprev, int in)
{
    const Layout& L = c->lay[instance];
    if ((long long)L.nx * L.ny <= kSmallState) return transfer_small(c, instance, lvl, {f, g, h}, jprev, in);
    int rc;
    if (f && (rc = transfer(c, instance, lvl, lbm::kF, f, in))) return rc;
    if (g && (rc = transfer(c, instance, lvl, lbm::kG, g, in))) return rc;
    if (h && (rc = transfer(c, instance, lvl, lbm::kH, h, in))) return rc;
    if (jprev && (rc = transfer(c, instance, lvl, -1, jprev, in))) return rc;
    HIP_TRY(hipStreamSynchronize(c->stream));
    return LBM_OK;
}
}  // namespace

int lbm_get_state(lbm_ctx* c, int instance, double* f, double* g, double* h, double* jprev, int64_t* step)
{
    int rc = check_instance(c, instance);
    if (rc) return rc;
    if ((rc = transfer_state(c, instance, (int)(c->step & 1), f, g, h, jprev, 0))) return rc;
    if (step) *step = c->step;
    return LBM_OK;
}

int lbm_set_state(lbm_ctx* c, int instance, const double* f, const double* g, const double* h, const double* jprev,
                  int64_t step)
{
    int rc = check_instance(c, instance);
    if (rc) return rc;
    if (step < 0) return fail(LBM_EINVAL, "negative step");
    if (c->n > 1 && (step & 1) != (c->step & 1))
        return fail(LBM_EINVAL, "batched lattices share one time level: step parity must stay %lld",
                    (long long)(c->step & 1));
    const Layout& L = c->lay[instance];
    // the current level is the one the new step count points at; copy the
    // other populations across if the parity changes
    const int old_lvl = (int)(c->step & 1), new_lvl = (int)(step & 1);
    if (old_lvl != new_lvl)
        HIP_TRY(hipMemcpyAsync(c->ws + L.pop_off[new_lvl], c->ws + L.pop_off[old_lvl],
                               (size_t)lbm::kPlanes * L.plane * real_size(c->prec), hipMemcpyDeviceToDevice, c->stream));
    if ((rc = transfer_state(c, instance, new_lvl, const_cast<double*>(f), const_cast<double*>(g),
                             const_cast<double*>(h), const_cast<double*>(jprev), 1)))
        return rc;
    c->step = step;
    return LBM_OK;
}

namespace {
struct CkptHeader {
    char magic[8];
    uint32_t version, prec;
    int32_t n, pad;
    int64_t step;
    uint64_t hash;
    double bx[4], by[4];
};
size_t ckpt_payload(const lbm_ctx* c, int k)
{
    const size_t rsz = real_size(c->prec);
    return ((size_t)lbm::kPlanes + 2) * c->lay[k].plane * rsz;
}
}  // namespace

size_t lbm_checkpoint_bytes(const lbm_ctx* c)
{
    if (!c) return 0;
    size_t b = 0;
    for (int k = 0; k < c->n; ++k) b += sizeof(CkptHeader) + ckpt_payload(c, k);
    return b;
}

int lbm_checkpoint_save(lbm_ctx* c, void* host_buf, size_t bytes)
{
    if (!c || !host_buf) return fail(LBM_EINVAL, "NULL argument");
    if (bytes < lbm_checkpoint_bytes(c)) return fail(LBM_EINVAL, "checkpoint buffer too small");
    char* p = static_cast<char*>(host_buf);
    const uint64_t hsh = params_hash(c->params);
    const size_t rsz = real_size(c->prec);
    const int lvl = (int)(c->step & 1);
    for (int k = 0; k < c->n; ++k) {
        const Layout& L = c->lay[k];
        CkptHeader hd{};
        std::memcpy(hd.magic, "LBMCKPT3", 8);
        hd.version = LBM_ABI_VERSION;
        hd.prec = c->prec;
        hd.n = c->n;
        hd.step = c->step;
        hd.hash = hsh;
        for (int b = 0; b < 4; ++b) {
            hd.bx[b] = c->bx[4 * k + b];
            hd.by[b] = c->by[4 * k + b];
        }
        std::memcpy(p, &hd, sizeof(hd));
        p += sizeof(hd);
        const size_t level_b = (size_t)lbm::kPlanes * L.plane * rsz;
        HIP_TRY(hipMemcpyAsync(p, c->ws + L.pop_off[lvl], level_b, hipMemcpyDeviceToHost, c->stream));
        HIP_TRY(hipMemcpyAsync(p + level_b, c->ws + L.jprev_off, 2 * (size_t)L.plane * rsz, hipMemcpyDeviceToHost,
                               c->stream));
        p += ckpt_payload(c, k);
    }
    HIP_TRY(hipStreamSynchronize(c->stream));
    return LBM_OK;
}

int lbm_checkpoint_load(lbm_ctx* c, const void* host_buf, size_t bytes)
{
    if (!c || !host_buf) return fail(LBM_EINVAL, "NULL argument");
    if (bytes != lbm_checkpoint_bytes(c)) return fail(LBM_EINVAL, "checkpoint size %zu != %zu", bytes,
                                                      lbm_checkpoint_bytes(c));
    const char* p = static_cast<const char*>(host_buf);
    const uint64_t hsh = params_hash(c->params);
    const size_t rsz = real_size(c->prec);
    CkptHeader first{};
    std::memcpy(&first, p, sizeof(first));
    if (std::memcmp(first.magic, "LBMCKPT3", 8) || first.hash != hsh || first.prec != c->prec || first.n != c->n)
        return fail(LBM_EINVAL, "checkpoint of another format, or written by a context with different parameters");
    const int lvl = (int)(first.step & 1);
    for (int k = 0; k < c->n; ++k) {
        const Layout& L = c->lay[k];
        CkptHeader hd{};
        std::memcpy(&hd, p, sizeof(hd));
        p += sizeof(hd);
        for (int b = 0; b < 4; ++b) {
            c->bx[4 * k + b] = hd.bx[b];
            c->by[4 * k + b] = hd.by[b];
        }
        const size_t level_b = (size_t)lbm::kPlanes * L.plane * rsz;
        HIP_TRY(hipMemcpyAsync(c->ws + L.pop_off[lvl], p, level_b, hipMemcpyHostToDevice, c->stream));
        HIP_TRY(hipMemcpyAsync(c->ws + L.jprev_off, p + level_b, 2 * (size_t)L.plane * rsz, hipMemcpyHostToDevice,
                               c->stream));
        p += ckpt_payload(c, k);
    }
    HIP_TRY(hipStreamSynchronize(c->stream));
    c->step = first.step;
    return LBM_OK;
}

// ---- launch configuration ----

int lbm_tile_count(void) { return lbm::kTileCount; }

int lbm_tile_shape(int id, int* tx, int* ty)
{
    if (id < 0 || id >= lbm::kTileCount) return fail(LBM_EINVAL, "tile id %d out of range", id);
    // runs: tx = nodes per run, ty = 0
    const int rn = lbm::run_nodes(id);
    if (tx) *tx = rn ? rn : lbm::kTileTX[id];
    if (ty) *ty = rn ? 0 : lbm::kTileTY[id];
    return LBM_OK;
}

int lbm_set_tile(lbm_ctx* c, int id)
{
    if (!c) return fail(LBM_EINVAL, "context is NULL");
    if (id < 0 || id >= lbm::kTileCount) return fail(LBM_EINVAL, "tile id %d out of range", id);
    if (c->tile != id) {
        drop_graph(c);
        c->tile = id;
        if (c->n > 1) c->grid = 0;
    }
    return LBM_OK;
}

int lbm_get_tile(const lbm_ctx* c) { return c ? c->tile : -1; }

int lbm_set_graph_steps(lbm_ctx* c, int steps)
{
    if (!c) return fail(LBM_EINVAL, "context is NULL");
    if (steps < 0 || (steps & 1)) return fail(LBM_EINVAL, "graph steps must be even and >= 0");
    drop_graph(c);
    c->graph_steps = steps;
    return LBM_OK;
}

int lbm_set_grid(lbm_ctx* c, int workgroups)
{
    if (!c) return fail(LBM_EINVAL, "context is NULL");
    if (workgroups < 0) return fail(LBM_EINVAL, "negative grid");
    drop_graph(c);
    c->grid = workgroups > c->ntiles[c->tile] ? c->ntiles[c->tile] : workgroups;
    return LBM_OK;
}

int lbm_copy_probe(const void* d_src, void* d_dst, size_t bytes, void* hip_stream)
{
    if (!d_src || !d_dst || bytes == 0 || bytes % 16) return fail(LBM_EINVAL, "copy probe: bad arguments");
    if ((reinterpret_cast<uintptr_t>(d_src) | reinterpret_cast<uintptr_t>(d_dst)) % 16)
        return fail(LBM_EINVAL, "copy probe: buffers must be 16-byte aligned");
    HIP_TRY(lbm::launch_copy(d_src, d_dst, bytes, static_cast<hipStream_t>(hip_stream)));
    return LBM_OK;
}

int lbm_autotune(lbm_ctx* c, int steps_per_trial, int* best_tile, int* best_grid, float* best_ms)
{
    if (!c) return fail(LBM_EINVAL, "context is NULL");
    if (steps_per_trial < 1) return fail(LBM_EINVAL, "steps_per_trial must be >= 1");
    int dev = 0, cus = 0;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    // Each trial replays a captured graph of G steps, as lbm_step does: the
    // graph of a configuration is captured and replayed once untimed, then
    // replayed once timed (plain launches would time the launch path of
    // small lattices rather than their kernels).
    const int saved_graph = c->graph_steps;
    const int G = steps_per_trial + (steps_per_trial & 1);
    drop_graph(c);
    c->graph_steps = G;
    float best = 1e30f;
    int bt = c->tile, bg = c->grid;
    // untimed steps first: the first candidate must not be timed on a cold
    // device (clocks and caches)
    int rc = lbm_step(c, G > 8 ? G : 8);
    if (rc == LBM_OK) {
        hipError_t e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) rc = fail(LBM_EHIP, "autotune warm-up: %s", hipGetErrorString(e));
    }
    for (int t = 0; t < lbm::kTileCount && rc == LBM_OK; ++t) {
        if (lbm::run_nodes(t) && !c->has_runs) continue;
        int grids[3] = {0, 0, 0}, ng = 1;
        if (c->n > 1) {
            int per_cu = 1;
            if (lbm::step_occupancy((int)c->prec, t, c->variant, &per_cu) != hipSuccess || per_cu < 1) per_cu = 1;
            const int resident = per_cu * (cus > 0 ? cus : 256);
            grids[0] = resident < c->ntiles[t] ? resident : c->ntiles[t];
            grids[1] = 2 * resident < c->ntiles[t] ? 2 * resident : c->ntiles[t];
            grids[2] = c->ntiles[t];
            ng = 3;
        }
        for (int q = 0; q < ng && rc == LBM_OK; ++q) {
            c->tile = t;
            c->grid = grids[q];
            drop_graph(c);
            // an even step count starts a graph; the untimed replay captures it
            if (c->step & 1) rc = lbm_step(c, 1);
            if (rc == LBM_OK) rc = lbm_step(c, G);
            if (rc) break;
            hipError_t e = hipEventRecord(e0, c->stream);
            if (e == hipSuccess) rc = lbm_step(c, G);
            if (rc) break;
            if (e == hipSuccess) e = hipEventRecord(e1, c->stream);
            if (e == hipSuccess) e = hipEventSynchronize(e1);
            float ms = 0.f;
            if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
            if (e != hipSuccess) {
                rc = fail(LBM_EHIP, "autotune timing: %s", hipGetErrorString(e));
                break;
            }
            ms /= (float)G;
            if (ms < best) {
                best = ms;
                bt = t;
                bg = grids[q];
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    drop_graph(c);
    c->tile = bt;
    c->grid = bg;
    c->graph_steps = saved_graph;
    if (rc) return rc;
    if (best_tile) *best_tile = bt;
    if (best_grid) *best_grid = bg;
    if (best_ms) *best_ms = best;
    return LBM_OK;
}

int lbm_get_grid(const lbm_ctx* c) { return c ? c->grid : -1; }

size_t lbm_bytes_per_update(int precision)
{
    const size_t rsz = precision == LBM_FP64 ? 8 : 4;
    return (2 * lbm::kPlanes + 4) * rsz;
}

}  // extern "C"
