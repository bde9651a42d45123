// Host-side sizing of the launches: element sizes, which recompute kernel a
// checkpoint interval takes and its scratch, and the feedback model's table
// layout and block counts.  Plain host code (no kernels), shared by the entry
// points and the launchers.
#include "fb_launch.hpp"
#include "jd_launch.hpp"

namespace jd {

size_t real_size(int prec) { return prec == JD_FP64 ? sizeof(double) : sizeof(float); }

template <typename Real, int D>
static int max_K() { return RecomputeShape<Real, D>::R * RecomputeShape<Real, D>::S; }

template <typename Real, int D>
static int reg_R() { return RecomputeShape<Real, D>::R; }

// Longest checkpoint interval of the register kernel, and the longest it
// sweeps with one regeneration of each step (K <= R: one sub-segment).
static int register_max_K(int prec, int D) {
    if (prec == JD_FP64)
        return D == 1 ? max_K<double, 1>() : D == 2 ? max_K<double, 2>()
             : D == 4 ? max_K<double, 4>() : max_K<double, 8>();
    return D == 1 ? max_K<float, 1>() : D == 2 ? max_K<float, 2>()
         : D == 4 ? max_K<float, 4>() : max_K<float, 8>();
}
static int register_single_K(int prec, int D) {
    if (prec == JD_FP64)
        return D == 1 ? reg_R<double, 1>() : D == 2 ? reg_R<double, 2>()
             : D == 4 ? reg_R<double, 4>() : reg_R<double, 8>();
    return D == 1 ? reg_R<float, 1>() : D == 2 ? reg_R<float, 2>()
         : D == 4 ? reg_R<float, 4>() : reg_R<float, 8>();
}

// The segment kernel (one regeneration, workspace scratch) where the register
// kernel would regenerate every step twice at d = 8, and wherever K exceeds
// the register kernel's buffers.  At d <= 4 a second regeneration costs less
// than writing and reading back the states.
bool recompute_uses_segments(int prec, int D, int K) {
    return K > register_max_K(prec, D) || (D == 8 && K > register_single_K(prec, D));
}

size_t seg_scratch_bytes(const HostProblem& p, const HostRun& r) {
    if (r.mode != JD_RECOMPUTE || !recompute_uses_segments(r.prec, p.D, r.K))
        return 0;
    return (size_t)seg_blocks(r) * (size_t)r.K * (size_t)p.d * kBlock * real_size(r.prec);
}

bool recompute_supported(const HostProblem& p, const HostRun& r) {
    return r.K >= 1 && seg_scratch_bytes(p, r) <= kSegScratchMax;
}

// ---------------------------------------------------------------------------
// The feedback model.

FbTable fb_table_layout(const FbHost& p) {
    FbTable t;
    auto up = [](size_t x) { return (x + 63) / 64 * 64; };
    t.mu = 0;
    t.zd = up((size_t)p.N * p.nx * p.nvp);
    t.ks = t.zd + up((size_t)(p.N + 1) * 2);
    t.sd = t.ks + 64;
    t.count = t.sd + up((size_t)(p.N + 1) * 2);
    return t;
}

size_t fb_mom_count(const FbHost& p, const HostRun& r) {
    return (size_t)(p.N + 1) * (size_t)fb_partial_blocks(p, r) * 4;
}

size_t fb_svar_count(const FbHost& p) { return (size_t)(p.N + 1) * 2 + 4; }

int fb_ring_groups(int np) { return np <= kBlock ? 1 : 8; }

// Where the small-count kernels (fb_small.hip) take over, 50 steps of the
// 10 x 10 grid on an MI355X.
//
// Forward: a row kernel's time grows with the slots it computes (a segment's
// halos included), the lane kernels' stays flat up to one wave per SIMD
// (65536 particles) and, for rings of more than 256 particles, one workgroup per
// CU.  Row / lane, FP32: 36 / 144 us at 2000 particles, 117 / 134 at 49152, 132 / 134
// at 57344; FP64 42 / 250, 224 / 242, 255 / 242.  Rings of 8..256, by computed slots:
// FP32 114 / 144 at 26900, 155 / 144 at 47600, 174 / 144 at 53800; FP64 182 / 242 at 23600, 336 /
// 242 at 47100.  Rings of 500 and 2000: FP32 267 / 334 at 96000, 345 / 334 at 128000;
// FP64 850 / 1084 at 128000, 1054 / 1084 at 160000.  Jump-adapted grid (0.18 jumps per
// interval): FP32 68 / 205 at 2000, 159 / 199 at 28672, 198 / 199 at 32768 (at 0.93
// per interval 235 / 232); FP64 93 / 378 at 2000, 340 / 378 at 28672, 380 / 378 at 32768.
static int64_t fb_small_forward_max(const FbHost& p, const HostRun& r) {
    if (p.np > 1 && p.G > 1)
        return r.prec == JD_FP64 ? 147456 : 114688;
    if (p.grid == 1)
        return 28672;
    if (p.np > 1)
        return r.prec == JD_FP64 ? 32768 : 40960;
    return 49152;
}
// Adjoint, split / one kernel: FP32 33 / 162 us at 2000 particles, 72 / 163 at
// 32768, 118 / 169 at 65536 (the whole gradient 260 / 267), 171 / 172 at 100000 (309 /
// 287); FP64 139 / 230 at 32768, 201 / 233 at 48000, 265 / 236 at 64000.  Rings of
// more than 256: FP32 363 / 454 at 200000, 447 / 458 at 256000; FP64 894 / 1080 at
// 200000, 1107 / 1083 at 256000.  Jump-adapted grid: FP32 65 / 364 at 2000, 240 / 368 at
// 49152, 351 / 370 at 65536 (100 steps: 371 / 507 at 49152, 514 / 507 at 65536); FP64 86 / 515
// at 2000, 355 / 515 at 32768, 421 / 515 at 36864 (300 steps 1786 / 1675).
// Jump-adapted grid: a block with a particle past its jump stack (32 entries) is swept
// by the general kernel as well, so the split is taken up to 16 expected jumps (past
// the stack: 1 particle in 10^4).
constexpr double kFbSmallJumps = 16.0;
static int64_t fb_small_adjoint_max(const FbHost& p, const HostRun& r) {
    if (p.np > 1 && p.G > 1)
        return 200000;
    if (p.grid == 1)
        return p.rate * p.T > kFbSmallJumps ? 0 : r.prec == JD_FP64 ? 32768 : 49152;
    return r.prec == JD_FP64 ? 49152 : 65536;
}
// The coefficients of all particle-steps stay in the workspace.
constexpr size_t kFbSmallMaxBytes = (size_t)1 << 30;

// Values of one slot that the split adjoint keeps: per step its coefficients
// and weight, on the jump-adapted grid per sub-step.
static size_t fb_small_cells(const FbHost& p) {
    return (size_t)p.N + (p.grid == 1 ? kFbJumpStates : 0);
}
bool fb_small_adjoint_ok(const FbHost& p, const HostRun& r) {
    return r.mode == JD_STORE && r.M <= fb_small_adjoint_max(p, r) &&
           (size_t)r.ldm * fb_small_cells(p) * (kFbSmallCoef + 1) * real_size(r.prec) <=
               kFbSmallMaxBytes;
}

// The row forward leaves the empty slots of a ring workgroup unwritten, which
// only the split adjoint masks.
bool fb_small_forward_ok(const FbHost& p, const HostRun& r) {
    if (p.np > 1 && !fb_small_adjoint_ok(p, r))
        return false;
    const int slots = fb_row_slots(p);
    return fb_row_plan(p, r, slots).blocks * slots <= fb_small_forward_max(p, r);
}

// A row forward's time hardly grows up to 8192 particles (50 steps, the whole call: FP32
// 36 us at 2000 particles, 42 at 8192, 57 at 16384, FP64 43 / 58 / 91; jump-adapted
// grid 67 / 78 / 105 and 93 / 119 / 209), so up to four trials of a line search share one
// launch.  Ten iterations of 2000 particles x 50 on the jump-adapted grid, 28 trials:
// 3.78 ms with a launch per trial, 2.16 with four in one.
int fb_trials(const FbHost& p, const HostRun& r) {
    if (p.np > 1 || !fb_small_forward_ok(p, r))
        return 1;
    const int64_t n = 8192 / r.ldm;
    return n < 1 ? 1 : n > kLsTrials ? kLsTrials : (int)n;
}

FbSmall fb_small_layout(const FbHost& p, const HostRun& r) {
    FbSmall s{};
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    size_t off = 0;
    const bool adj = fb_small_adjoint_ok(p, r);
    const bool rings = p.np > 1 && adj;  // segments' state between launches
    s.state = off;
    off += rings ? up((size_t)2 * 4 * r.M * real_size(r.prec)) : 0;
    s.acc = off;
    off += rings ? up((size_t)r.M * sizeof(double)) : 0;
    s.start = off;
    off += adj && p.grid == 1 ? up((size_t)r.ldm * p.N) : 0;
    const size_t cells = (size_t)r.ldm * fb_small_cells(p) * real_size(r.prec);
    s.coef = off;
    off += adj ? up(cells * kFbSmallCoef) : 0;
    s.wgt = off;
    off += adj ? up(cells) : 0;
    s.total = off;
    return s;
}

FbRowPlan fb_row_plan(const FbHost& p, const HostRun& r, int slots) {
    FbRowPlan q{};
    q.steps = p.N;
    if (p.np == 1) {
        q.blocks = r.ldm / slots;
    } else if (p.np <= slots) {
        q.rings = slots / p.np;
        q.blocks = (p.nsys + q.rings - 1) / q.rings;
    } else {
        // a quarter of the slots as halo on either side: half the work is own
        q.halo = slots / 4;
        q.steps = 2 * q.halo;
        q.own = slots - 2 * q.halo;
        q.nseg = (p.np + q.own - 1) / q.own;
        q.blocks = p.nsys * q.nseg;
    }
    return q;
}

int fb_forward_blocks(const FbHost& p, const HostRun& r) {
    if (fb_small_forward_ok(p, r))
        return (int)fb_row_plan(p, r, fb_row_slots(p)).blocks;
    return p.np == 1 ? r.nblk : r.nblk / p.G;
}

// Several groups per block divide the per-step gradient partials but cost
// registers.  Measured on 2^20 x 500: FP64 paths 31.1 / 28.9 ms for 1 / 2
// groups (16.2 / 15.5 / 18.3 ms for 1 / 2 / 4 on FP32 paths while these used
// the FP64 matrix cores); FP32 paths on the FP32 matrix cores with velocity
// transposes of the compiled row width fit five waves per SIMD with one group:
// 10.8 ms against 11.3 ms for two (four waves) and 11.0 ms for two forced to
// five waves (spills).  Rings keep their own G (whole rings per block); the
// jump-adapted adjoint runs one group.
int fb_adjoint_groups(const FbHost& p, const HostRun& r) {
    if (p.np > 1)
        return p.G;
    return p.grid == 0 && r.prec == JD_FP64 && r.nblk >= 2048 ? 2 : 1;
}

int fb_partial_blocks(const FbHost& p, const HostRun& r) {
    if (p.np > 1 && fb_small_adjoint_ok(p, r))
        return p.G == 1 ? r.nblk : r.nblk / 2;  // two 256-slot groups per column
    const int G = fb_adjoint_groups(p, r);
    return (r.nblk + G - 1) / G;
}

}  // namespace jd
