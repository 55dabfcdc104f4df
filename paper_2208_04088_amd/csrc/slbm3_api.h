// Host side of the three-dimensional step (slbm3_* in include/slbm3.h).
// Included at the end of slbm.hip: it shares that translation unit's error
// reporting (fail, HIP_TRY, slbm_last_error) and DeviceGuard.
#include "slbm3.h"
#include "step3_kernel.h"

// How k3_march goes through a box and whether it takes its steps (march_of).
struct March3 {
    bool on = false;
    int rows = 1, nch = 1, nyt = 1, depth = 1, mtiles = 1, slots = 256;
};

struct slbm3_s {
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int nx = 0, ny = 0, nz = 0;
    long long plane = 0;             // sites
    long long stride = 0;            // elements between planes of the population and U buffers
    int precision = SLBM_FP64;
    size_t esize = 8;
    int px = 1;
    int wkind[2] = {0, 0};
    double wval[2][3] = {{0, 0, 0}, {0, 0, 0}};   // lattice units
    double wq[2] = {0.5, 0.5};
    // time profiles: the walls' (RAMP: ramp length in steps, else 0) and the
    // general geometry's ramp slots (slot 0: constant)
    double wramp[2] = {0.0, 0.0};
    double slot_ramp[slbm3_dev::kProfileSlots3] = {};
    int norder = 0;
    double lamL = 0, muL = 1.0 / 3.0, tau = 0.55, FL[3] = {0, 0, 0};
    double dt_user = 1, s_sigma = 1, s_v = 1, rho_user = 1;
    void* buf[2] = {nullptr, nullptr};
    int cur = 0;
    bool local = true;
    double* U = nullptr;
    void* dens = nullptr;
    // the walls' parts (wall_parts3), one block: k3_march reads [cur], writes the other
    void* wall[2] = {nullptr, nullptr};
    bool wall_fresh = false;              // wall[cur] belongs to the current state
    unsigned int* diverged = nullptr;
    double* scratch = nullptr;       // planes of doubles, on demand (host readouts, initial fields)
    int scratch_planes = 0;
    int64_t step = 0;
    // general geometry: site flags, first link record of each site, records
    bool geo = false;
    uint32_t* flags = nullptr;
    int32_t* bidx = nullptr;
    void* links = nullptr;
    // per link record: (A, s_kappa) of the rule (k3_step, k3_links_ext); k3_march
    // reads one and writes the other (lval_at)
    void* lval[2] = {nullptr, nullptr};
    int32_t* rowrec = nullptr;       // per 64-site chunk of a row: first record
    int32_t* wrec = nullptr;         // per workgroup of k3_step: first record
    int32_t* elink = nullptr;        // the records whose Neumann data are extrapolated
    int64_t n_ext = 0;
    uint64_t geo_hash = 0;           // the geometry a checkpoint must match (mask and cut links, or the walls)
    int64_t n_links = 0;
    size_t link_bytes = 0;
    March3 march;
};

namespace {

using namespace slbm3_dev;

// Which of the two lists of rule values belongs to the current state: with
// k3_march the one of the state's buffer, so that a state is one place whatever
// led there (a step from local populations, which reads none, writes in place
// what the next step reads); without it the first.
int lval_at(const slbm3_s* h) { return h->march.on ? h->cur ^ (h->local ? 1 : 0) : 0; }

template <typename real>
Step3Args<real> make_args3(const slbm3_s* h, int src)
{
    Step3Args<real> a{};
    a.src = (const real*)h->buf[src];
    a.dst = (real*)h->buf[src ^ 1];
    a.U = h->U;
    a.dens = (real*)h->dens;
    a.diverged = h->diverged;
    a.plane = h->plane;
    a.stride = h->stride;
    a.nx = h->nx; a.ny = h->ny; a.nz = h->nz;
    a.px = h->px;
    a.local = h->local ? 1 : 0;
    a.ntiles = ((h->nx + 63) / 64) * h->ny * h->nz;
    // backwards where the second pass would find little of the first one's
    // state in the caches: not small boxes with cut links, which it lets end on
    // the rows with the longest work.  us per step, forward and backward:
    //   fp32 slab   64^3 18.3 18.1   80^3 36.4 34.7   (96^3 and more: k3_march)   fp64 slab  60^3 30.0 29.5
    //   fp32 porous 100^3 (176 MB) 54.7 53.2   128^3 102.9 102.6   150^3 238 225   180^3 360 351
    //   fp64 porous  90^3 (240 MB) 73.8 73.2   120^3 206 195
    //   fp64 solid with a cavity and a crack  45x38x41 16.5 16.8   60^3 (72 MB) 26.7 28.4
    a.back = !h->geo || h->plane * (long long)((2 * kQ + 1) * sizeof(real) + 24) > 125000000 ? 1 : 0;
    // time profiles at the step of the state the pulls read (the previous
    // step's post-collision state) and of the state this step produces
    const double n_pull = h->step >= 1 ? (double)(h->step - 1) : 0.0, n_next = (double)h->step;
    auto ramp = [](double n, double len) { return len > 0.0 ? std::min(n / len, 1.0) : 1.0; };
    for (int k = 0; k < kProfileSlots3; ++k) {
        a.pf_pull[k] = (real)ramp(n_pull, h->slot_ramp[k]);
        a.pf_next[k] = (real)ramp(n_next, h->slot_ramp[k]);
    }
    for (int s = 0; s < 2; ++s) {
        a.wkind[s] = h->wkind[s];
        for (int k = 0; k < 3; ++k) a.wval[s][k] = (real)(h->wval[s][k] * ramp(n_pull, h->wramp[s]));
        // section 4.2: a site behind x along the cut link exists unless nx = 1
        const bool behind = h->nx >= 2;
        const double q = h->wq[s];
        a.wkap[s] = (real)(behind ? (1.0 - 2.0 * q) / (1.0 + 2.0 * q) : 0.0);
        a.wbeta[s] = (real)(behind ? 2.0 / (1.0 + 2.0 * q) : 1.0);
        a.wq1[s] = (real)(1.0 + q);
        a.wq[s] = (real)q;
        a.wext[s] = behind && h->norder == 1 && h->wkind[s] == SLBM_NEUMANN ? 1 : 0;
        a.wskap[s] = h->wkind[s] == SLBM_DIRICHLET ? a.wkap[s] : -a.wkap[s];
        for (int k = 0; k < 3; ++k) a.wval_next[s][k] = (real)(h->wval[s][k] * ramp(n_next, h->wramp[s]));
    }
    a.wsrc = (const real*)h->wall[h->cur];
    a.wdst = (real*)h->wall[h->cur ^ 1];
    a.omega = (real)(1.0 / h->tau);
    a.omega_h = (real)(1.0 - 0.5 / h->tau);
    a.ml = (real)(h->muL - h->lamL);
    a.lm = (real)(h->lamL - h->muL);
    for (int k = 0; k < 3; ++k) a.F[k] = (real)h->FL[k];
    a.flags = h->flags;
    a.bidx = h->bidx;
    a.links = (const Link3<real>*)h->links;
    a.lval = (real*)h->lval[lval_at(h)];
    a.lval_next = (real*)h->lval[lval_at(h) ^ 1];
    a.rowrec = h->rowrec;
    a.nlinks = (int)h->n_links;
    a.wrec = h->wrec;
    return a;
}

// The cut links of a general geometry as the kernels read them: per-site
// flags (bit i - 1: link i cut; kVoid3: void), each cut site's first record,
// and the records sorted by site and direction, in lattice units.  Validates
// what slbm3_create documents; the host arrays are the caller's.
struct Geo3 {
    std::vector<int> gslot;          // per group: its time-profile slot
    std::vector<double> slot_ramp;   // per slot: ramp length in steps (0: constant)
    std::vector<uint32_t> flags;
    std::vector<int32_t> bidx;
    std::vector<Link3<double>> recs;
    std::vector<double> skap;        // per record: kappa (Dirichlet), -kappa (Neumann) or 0 (ext)
    std::vector<int32_t> elink;      // the ext records
    std::vector<int32_t> wrec;       // per workgroup of k3_step: its first record, then the count
    std::vector<int32_t> rowrec;     // per 64-site chunk of a row: its first record, then the count
    uint64_t hash = 0;               // FNV-1a of the mask and of each cut link's site, direction, q,
                                     // groups and normals, in record order
};

// 64-bit FNV-1a, fed value by value (no struct padding enters it).
struct Fnv64 {
    uint64_t h = 0xcbf29ce484222325ull;
    void bytes(const void* p, size_t n)
    {
        const unsigned char* c = (const unsigned char*)p;
        for (size_t i = 0; i < n; ++i) h = (h ^ c[i]) * 0x100000001b3ull;
    }
    template <typename T> void put(T v) { bytes(&v, sizeof v); }
};

int build_geo3(const slbm3_params* p, const slbm3_s* h, Geo3& g)
{
    const long long n = h->plane;
    const int nx = h->nx, ny = h->ny, nz = h->nz;
    if (p->n_links < 0 || (p->n_links > 0 && !p->links)) return fail(SLBM_E_INVAL, "links: null array");
    if (p->n_groups < 0 || (p->n_groups > 0 && !p->groups)) return fail(SLBM_E_INVAL, "groups: null array");
    if (p->n_links > 18LL * n) return fail(SLBM_E_INVAL, "more links than a box has");
    if (p->n_links > (int64_t)INT_MAX - 255)
        return fail(SLBM_E_UNSUPPORTED, "more than 2^31 - 256 cut links (records are indexed with 32 bits)");
    for (int k = 0; k < p->n_groups; ++k) {
        const slbm3_bc_group& gr = p->groups[k];
        if (gr.kind != SLBM_DIRICHLET && gr.kind != SLBM_NEUMANN)
            return fail(SLBM_E_INVAL, "group %d: kind must be SLBM_DIRICHLET or SLBM_NEUMANN", k);
        if (!std::isfinite(gr.value[0]) || !std::isfinite(gr.value[1]) || !std::isfinite(gr.value[2]) ||
            !std::isfinite(gr.pressure))
            return fail(SLBM_E_INVAL, "group %d: values must be finite", k);
        if (gr.profile != SLBM_PROFILE_STEP && gr.profile != SLBM_PROFILE_RAMP)
            return fail(SLBM_E_INVAL, "group %d: profile must be SLBM_PROFILE_STEP or SLBM_PROFILE_RAMP", k);
        if (gr.profile == SLBM_PROFILE_RAMP && !(gr.ramp_time > 0.0))
            return fail(SLBM_E_INVAL, "group %d: ramp time must be positive", k);
    }
    // each group's time-profile slot: 0 for STEP, one slot per distinct ramp time
    g.gslot.assign((size_t)p->n_groups, 0);
    g.slot_ramp.assign(kProfileSlots3, 0.0);
    {
        int nslots = 1;
        for (int k = 0; k < p->n_groups; ++k) {
            if (p->groups[k].profile != SLBM_PROFILE_RAMP) continue;
            const double len = p->groups[k].ramp_time / h->dt_user;
            int sl = 1;
            while (sl < nslots && g.slot_ramp[(size_t)sl] != len) ++sl;
            if (sl == nslots) {
                if (nslots == kProfileSlots3)
                    return fail(SLBM_E_UNSUPPORTED, "more than %d distinct ramp times", kProfileSlots3 - 1);
                g.slot_ramp[(size_t)nslots++] = len;
            }
            g.gslot[(size_t)k] = sl;
        }
    }
    g.flags.assign((size_t)n, 0u);
    for (long long s = 0; s < n; ++s)
        if (!p->mask[s]) g.flags[s] = kVoid3;
    auto far_site = [&](long long s, int i) {
        const long long x = s % nx, y = (s / nx) % ny, z = s / ((long long)nx * ny);
        const long long fx = (x + kCX[i] + nx) % nx, fy = (y + kCY[i] + ny) % ny, fz = (z + kCZ[i] + nz) % nz;
        return (fz * ny + fy) * nx + fx;
    };
    for (int64_t l = 0; l < p->n_links; ++l) {
        const slbm3_link& L = p->links[l];
        if (L.site < 0 || (long long)L.site >= n) return fail(SLBM_E_INVAL, "link %lld: site out of range", (long long)l);
        if (L.dir < 1 || L.dir > 18) return fail(SLBM_E_INVAL, "link %lld: direction must be in 1..18", (long long)l);
        if (!p->mask[L.site]) return fail(SLBM_E_INVAL, "link %lld: starts at a void site", (long long)l);
        if (!(L.q > 0.0 && L.q <= 1.0)) return fail(SLBM_E_INVAL, "link %lld: q must be in (0, 1]", (long long)l);
        if (L.group < 0 || L.group >= p->n_groups) return fail(SLBM_E_INVAL, "link %lld: group out of range", (long long)l);
        const double nn = std::sqrt(L.normal[0] * L.normal[0] + L.normal[1] * L.normal[1] + L.normal[2] * L.normal[2]);
        if (!(std::fabs(nn - 1.0) <= 1e-9)) return fail(SLBM_E_INVAL, "link %lld: normal is not a unit vector", (long long)l);
        if (L.group2 < -1 || L.group2 >= p->n_groups)
            return fail(SLBM_E_INVAL, "link %lld: second group out of range", (long long)l);
        if (L.group2 >= 0) {
            const double* m2 = L.normal2;
            const double n2 = std::sqrt(m2[0] * m2[0] + m2[1] * m2[1] + m2[2] * m2[2]);
            if (!(std::fabs(n2 - 1.0) <= 1e-9))
                return fail(SLBM_E_INVAL, "link %lld: second normal is not a unit vector", (long long)l);
            const double d = L.normal[0] * m2[0] + L.normal[1] * m2[1] + L.normal[2] * m2[2];
            if (!(std::fabs(d) <= 1e-9))
                return fail(SLBM_E_INVAL, "link %lld: the two faces' normals are not orthogonal", (long long)l);
            if (g.gslot[(size_t)L.group] != g.gslot[(size_t)L.group2])
                return fail(SLBM_E_INVAL, "link %lld: the two faces of an edge need the same time profile", (long long)l);
        }
        const uint32_t bit = 1u << (L.dir - 1);
        if (g.flags[L.site] & bit) return fail(SLBM_E_INVAL, "link %lld: listed twice", (long long)l);
        g.flags[L.site] |= bit;
    }
    // a link into the material crosses a crack: the link back is listed too
    for (int64_t l = 0; l < p->n_links; ++l) {
        const slbm3_link& L = p->links[l];
        const long long f = far_site(L.site, L.dir);
        if (p->mask[f] && !(g.flags[f] & (1u << (opp3(L.dir) - 1))))
            return fail(SLBM_E_INVAL, "link %lld: ends in the material but the link back (the crack's other face) "
                                      "is not listed", (long long)l);
    }
    // every link from the material into the void is listed: planes of z on
    // several host threads, each site's 18 neighbours through the 9 rows
    // around it; the first offending site (lowest index) is reported
    {
        const int nthreads = (int)std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
        std::vector<long long> first((size_t)nthreads, -1);
        std::vector<int> first_dir((size_t)nthreads, 0);
        auto scan = [&](int t) {
            for (int z = t; z < nz; z += nthreads) {
                for (int y = 0; y < ny; ++y) {
                    const uint8_t* row[3][3];
                    for (int dz = -1; dz <= 1; ++dz)
                        for (int dy = -1; dy <= 1; ++dy)
                            row[dz + 1][dy + 1] = p->mask + (((long long)((z + dz + nz) % nz) * ny + (y + dy + ny) % ny) * nx);
                    const long long base = ((long long)z * ny + y) * nx;
                    for (int x = 0; x < nx; ++x) {
                        if (!p->mask[base + x]) continue;
                        const uint32_t fl = g.flags[base + x];
                        const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
                        for (int i = 1; i < kQ; ++i) {
                            const int fx = kCX[i] < 0 ? xm : (kCX[i] > 0 ? xp : x);
                            if (!row[kCZ[i] + 1][kCY[i] + 1][fx] && !(fl & (1u << (i - 1)))) {
                                if (first[t] < 0 || base + x < first[t]) {
                                    first[t] = base + x;
                                    first_dir[t] = i;
                                }
                                break;
                            }
                        }
                        if (first[t] >= 0) break;
                    }
                    if (first[t] >= 0) break;
                }
                if (first[t] >= 0) break;              // later planes of this thread have higher indices
            }
        };
        std::vector<std::thread> pool;
        for (int t = 1; t < nthreads; ++t) pool.emplace_back(scan, t);
        scan(0);
        for (std::thread& th : pool) th.join();
        long long bad = -1;
        int bad_dir = 0;
        for (int t = 0; t < nthreads; ++t)
            if (first[t] >= 0 && (bad < 0 || first[t] < bad)) {
                bad = first[t];
                bad_dir = first_dir[t];
            }
        if (bad >= 0) return fail(SLBM_E_INVAL, "site %lld: link %d into the void is not listed", bad, bad_dir);
    }
    // records sorted by site, then direction (the kernel walks a site's cut
    // bits upwards from its first record)
    std::vector<int64_t> order((size_t)p->n_links);
    for (int64_t l = 0; l < p->n_links; ++l) order[(size_t)l] = l;
    std::sort(order.begin(), order.end(), [&](int64_t u, int64_t v) {
        const slbm3_link &A = p->links[u], &B = p->links[v];
        return A.site != B.site ? A.site < B.site : A.dir < B.dir;
    });
    {
        Fnv64 f;
        for (long long i = 0; i < n; ++i) f.put((uint8_t)(p->mask[i] != 0));   // any nonzero is material
        for (int64_t l : order) {
            const slbm3_link& L = p->links[l];
            f.put(L.site); f.put(L.dir); f.put(L.q); f.put(L.group); f.put(L.group2);
            for (int k = 0; k < 3; ++k) { f.put(L.normal[k]); f.put(L.normal2[k]); }
        }
        g.hash = f.h;
    }
    g.bidx.assign((size_t)n, 0);
    g.recs.resize(order.size());
    g.skap.resize(order.size());
    for (size_t r = 0; r < order.size(); ++r) {
        const slbm3_link& L = p->links[order[r]];
        if (r == 0 || p->links[order[r - 1]].site != L.site) g.bidx[L.site] = (int32_t)r;
        // a link through the edge of two faces: the Dirichlet face wins
        const bool two = L.group2 >= 0;
        const bool d1 = p->groups[L.group].kind == SLBM_DIRICHLET;
        const bool d2 = two && p->groups[L.group2].kind == SLBM_DIRICHLET;
        const slbm3_bc_group& gr = p->groups[(!d1 && d2) ? L.group2 : L.group];
        const int i = L.dir, ib = opp3(i);
        // section 4.2: no site behind x when the opposite link is cut too
        const bool thin = (g.flags[L.site] >> (ib - 1)) & 1u;
        const double q = L.q;
        const double kap = thin ? 0.0 : (1.0 - 2.0 * q) / (1.0 + 2.0 * q);
        const double bet = thin ? 1.0 : 2.0 / (1.0 + 2.0 * q);
        const double w = w3(i);
        const double c[3] = {(double)kCX[i], (double)kCY[i], (double)kCZ[i]};
        const double c2 = c[0] * c[0] + c[1] * c[1] + c[2] * c[2];
        Link3<double>& R = g.recs[r];
        R.kap = kap;
        R.bet2 = 2.0 * bet;
        R.q1 = 1.0 + q;
        R.q = q;
        for (int k = 0; k < 6; ++k) R.B[k] = 0.0;
        R.K = 0.0;
        if (gr.kind == SLBM_DIRICHLET) {
            const double cv = (c[0] * gr.value[0] + c[1] * gr.value[1] + c[2] * gr.value[2]) / h->s_v;
            R.c0 = bet * 6.0 * w * cv;
        } else {
            // the constants of e = c0 drho_bd + B:P_b - K (the record's
            // comment): sigma* = Pi sigma_b Pi + N, with N fixed by the
            // traction(s).  One face: Pi = I - n n, N = n t + t n - (t.n) n n.
            // Two faces (an edge): Pi = e e with e = n_A x n_B, and N holds the
            // rows of n_A and n_B in the frame (n_A, n_B, e), their shear
            // averaged.
            const double* n = L.normal;
            double t[3], A[3][3], Pi[3][3], N[3][3], T[3][3], B0[3][3];
            for (int k = 0; k < 3; ++k) t[k] = (gr.value[k] - gr.pressure * n[k]) / h->s_sigma;
            for (int u = 0; u < 3; ++u)
                for (int v = 0; v < 3; ++v) A[u][v] = c[u] * c[v] - (u == v ? 1.0 / 3.0 : 0.0);
            if (!two) {
                const double tn = t[0] * n[0] + t[1] * n[1] + t[2] * n[2];
                for (int u = 0; u < 3; ++u)
                    for (int v = 0; v < 3; ++v) {
                        Pi[u][v] = (u == v ? 1.0 : 0.0) - n[u] * n[v];
                        N[u][v] = n[u] * t[v] + t[u] * n[v] - tn * n[u] * n[v];
                    }
            } else {
                const slbm3_bc_group& g2r = p->groups[L.group2];
                const double* nb = L.normal2;
                double tb[3];
                for (int k = 0; k < 3; ++k) tb[k] = (g2r.value[k] - g2r.pressure * nb[k]) / h->s_sigma;
                const double e[3] = {n[1] * nb[2] - n[2] * nb[1], n[2] * nb[0] - n[0] * nb[2], n[0] * nb[1] - n[1] * nb[0]};
                auto dot = [](const double* a_, const double* b_) { return a_[0] * b_[0] + a_[1] * b_[1] + a_[2] * b_[2]; };
                const double* u3[3] = {n, nb, e};
                double S[3][3] = {{dot(t, n), 0.5 * (dot(t, nb) + dot(tb, n)), dot(t, e)},
                                  {0.5 * (dot(t, nb) + dot(tb, n)), dot(tb, nb), dot(tb, e)},
                                  {dot(t, e), dot(tb, e), 0.0}};
                for (int u = 0; u < 3; ++u)
                    for (int v = 0; v < 3; ++v) {
                        Pi[u][v] = e[u] * e[v];
                        double acc = 0.0;
                        for (int X = 0; X < 3; ++X)
                            for (int Y = 0; Y < 3; ++Y) acc += S[X][Y] * u3[X][u] * u3[Y][v];
                        N[u][v] = acc;
                    }
            }
            for (int u = 0; u < 3; ++u)
                for (int v = 0; v < 3; ++v) T[u][v] = A[u][0] * Pi[0][v] + A[u][1] * Pi[1][v] + A[u][2] * Pi[2][v];
            for (int u = 0; u < 3; ++u)
                for (int v = 0; v < 3; ++v) B0[u][v] = Pi[u][0] * T[0][v] + Pi[u][1] * T[1][v] + Pi[u][2] * T[2][v];
            double NA = 0.0;
            for (int u = 0; u < 3; ++u)
                for (int v = 0; v < 3; ++v) NA += N[u][v] * A[u][v];
            const double trB = B0[0][0] + B0[1][1] + B0[2][2];
            const double lm = h->lamL - h->muL;
            R.c0 = w * (2.5 - 1.5 * c2) + 4.5 * w * lm * (trB - c2 + 1.0);
            R.B[0] = 4.5 * w * B0[0][0];
            R.B[1] = 4.5 * w * B0[1][1];
            R.B[2] = 4.5 * w * B0[2][2];
            R.B[3] = 9.0 * w * B0[0][1];
            R.B[4] = 9.0 * w * B0[0][2];
            R.B[5] = 9.0 * w * B0[1][2];
            R.K = 4.5 * w * NA;
        }
        const int ext = gr.kind == SLBM_NEUMANN && h->norder == 1 && !thin ? 1 : 0;
        R.meta = link3_meta(i, ib, gr.kind, ext, kCX[i], kCY[i], kCZ[i], g.gslot[(size_t)(&gr - p->groups)]);
        R.site = L.site;
        g.skap[r] = ext ? 0.0 : (gr.kind == SLBM_DIRICHLET ? kap : -kap);
        if (ext) g.elink.push_back((int32_t)r);
    }
    // k3_step's workgroups take four 64-site row chunks each, a contiguous
    // range of sites from the first site of their first chunk
    {
        const long long chunks = (nx + 63) / 64, ntiles = chunks * ny * nz, nwg = (ntiles + 3) / 4;
        g.wrec.resize((size_t)nwg + 1);
        size_t r = 0;
        for (long long w = 0; w < nwg; ++w) {
            const long long t = 4 * w, row = t / chunks;
            const long long first = row * nx + 64 * (t % chunks);
            while (r < g.recs.size() && g.recs[r].site < first) ++r;
            g.wrec[(size_t)w] = (int32_t)r;
        }
        g.wrec[(size_t)nwg] = (int32_t)g.recs.size();
        g.rowrec.resize((size_t)ntiles + 1);
        r = 0;
        for (long long t = 0; t < ntiles; ++t) {
            const long long first = t / chunks * nx + 64 * (t % chunks);
            while (r < g.recs.size() && g.recs[r].site < first) ++r;
            g.rowrec[(size_t)t] = (int32_t)r;
        }
        g.rowrec[(size_t)ntiles] = (int32_t)g.recs.size();
    }
    return SLBM_OK;
}

// The records in the handle's precision.
template <typename real>
std::vector<Link3<real>> cast_links3(const std::vector<Link3<double>>& in)
{
    std::vector<Link3<real>> out(in.size());
    for (size_t r = 0; r < in.size(); ++r) {
        const Link3<double>& A = in[r];
        Link3<real>& B = out[r];
        B.kap = (real)A.kap; B.bet2 = (real)A.bet2; B.q1 = (real)A.q1; B.q = (real)A.q; B.c0 = (real)A.c0;
        for (int k = 0; k < 6; ++k) B.B[k] = (real)A.B[k];
        B.K = (real)A.K;
        B.meta = A.meta;
        B.site = A.site;
    }
    return out;
}

// Elements from one plane of a population or displacement buffer to the
// next: the plane rounded up to 4096 sites, then to an odd multiple of 4096,
// so that a power-of-two box does not start all its planes on one channel.
long long plane_stride(long long plane)
{
    long long q = (plane + 4095) / 4096;
    if ((q & 1) == 0) q += 1;
    return q * 4096;
}

int grid3(const slbm3_s* h)
{
    const long long tiles = (long long)((h->nx + 63) / 64) * h->ny * h->nz;
    const long long wg = (tiles + 3) / 4;
    const long long unit = 8LL * xcd_group_size3(h->geo);   // xcd_group3 permutes whole units
    return (int)((wg + unit - 1) / unit * unit);
}

// The extrapolating rules (general geometry, GEO, which implies PX; the other
// cut links' parts come from the previous k3_step), read by both pulls, and
// the density pass, which a step or a readout follows.
template <typename real, bool PX, bool GEO>
Step3Args<real> launch3_density(slbm3_s* h)
{
    const Step3Args<real> a = make_args3<real>(h, h->cur);
    if (GEO && !h->local && h->n_ext > 0)
        hipLaunchKernelGGL((k3_links_ext<real>), dim3((unsigned)((h->n_ext + 255) / 256)), dim3(256), 0, h->stream, a,
                           (const int32_t*)h->elink, (int)h->n_ext);
    hipLaunchKernelGGL((k3_density<real, PX, GEO>), dim3(grid3(h)), dim3(256), 0, h->stream, a);
    return a;
}

// `what`: 0 step, 2 init from scratch.
template <typename real, bool PX, bool GEO>
int launch3(slbm3_s* h, int what)
{
    const dim3 grid(grid3(h)), blk(256);
    if (what == 2) {
        Step3Args<real> a = make_args3<real>(h, h->cur);
        a.dst = (real*)h->buf[h->cur];
        hipLaunchKernelGGL((k3_set_dens<real>), dim3((unsigned)((h->plane + 255) / 256)), blk, 0, h->stream, a,
                           (const double*)h->scratch);
        hipLaunchKernelGGL((k3_init<real, PX, GEO>), grid, blk, 0, h->stream, a, (const double*)h->scratch);
    } else {
        const Step3Args<real> a = launch3_density<real, PX, GEO>(h);
        hipLaunchKernelGGL((k3_step<real, PX, GEO>), grid, blk, 0, h->stream, a);
    }
    HIP_TRY(hipGetLastError());
    return SLBM_OK;
}

int launch3_any(slbm3_s* h, int what);

// What a step goes through: both buffers and the displacement.
long long state_bytes3(const slbm3_s* h) { return h->plane * (2 * kQ * (long long)h->esize + 24); }

// Whether k3_march stores past the caches: once the state exceeds the 256 MB
// memory-side cache; below, the next launch finds what plain stores left in it.
// Boxes with cut links are above it wherever k3_march takes them.  us per step of
// slabs, streamed and plain:
//   fp32  96^3 (155 MB) 54 43   112^3 (247 MB) 80 56   116^3 (274 MB) 81 80   128^3 99 102   160^3 196 204
//   fp64  64^3 (85 MB) 27 25    90^3 (239 MB) 82 56    90x130x70 (268 MB) 90 93   96^3 77 82   128^3 175 181
// Rows that are not whole lines (64 bytes) share theirs with the next, and a line
// stored past the caches in two parts costs more than one; in single precision
// plain stores win from some 450 MB:
//   114x128x128 (329 MB) 100 102   120x150x150 (475 MB) 134 146   190x150x150 (752 MB) 235 224   114x192x192 (740 MB) 265 236
//   180x152x152 (732 MB) 275 242   300x256x256 (3.5 GB) 1099 1027   255x256x256 1029 964
// (double precision streams: 120x150x150 213 231, 300x256x256 1709 1759, 250x200x200 902 876).
constexpr long long kRaggedBytes = 450000000;
bool streamed3(const slbm3_s* h)
{
    const long long b = state_bytes3(h);
    return b > kCacheBytes && !(h->precision == SLBM_FP32 && h->nx % 16 != 0 && b > kRaggedBytes);
}

// Planes a k3_march workgroup marches through, for `tiles` tiles of rows over
// nz planes: a workgroup takes depth + 2 planes' time and a little to start,
// and the chip runs `slots` of them at once, so the depth that needs the
// fewest plane times in whole rounds (among depths that cost about the same
// the smaller: the last round ends more evenly; 256^3 slab 685 us at 32, 693 at
// 64).
int march_depth(long long tiles, int nz, int slots)
{
    int best = 1;
    long long cost = -1;
    for (int d = 1; d <= std::min(nz, 64); ++d) {
        const long long wgs = tiles * ((nz + d - 1) / d), c = 6 * ((wgs + slots - 1) / slots * (d + 3)) + d;
        if (cost < 0 || c < cost) { cost = c; best = d; }
    }
    return best;
}

// Whether the cut links leave k3_march's workgroups about equally long.  A wave
// takes a plane's links of its row 64 at a time, and the waves of the other rows
// wait for it: 0.15 of a plane's time each.  A plane face along z puts 320 links
// into one row of a tile, plane after plane, and the launch lasts as long as
// those tiles.  The launch's time by that over its time with equal rows; us per
// step, two launches and one (blocks of material in void):
//   fp32  1024x8x1024 1.51 577 687   512x34x256 1.57 277 402   128x128x256 1.50 258 317   192^3 1.57 423 454
//         256^3 1.57 1014 1228   1024x66x512 1.22 1987 2000
//   fp64  1024x8x1024 1.57 1065 1748   128x128x256 1.58 483 650   192^3 1.37 784 866   256^3 1.26 1886 1945
//         1024x66x512 1.18 3721 3445
// (porous solids of every density and round holes: up to 1.16, one launch faster).
bool even_links3(const slbm3_s* h, const Geo3& g, const March3& m)
{
    const int nseg = (h->nz + m.depth - 1) / m.depth;
    double sum = 0, base = 0, most = 0;
    for (int seg = 0; seg < nseg; ++seg)
        for (int yt = 0; yt < m.nyt; ++yt)
            for (int ch = 0; ch < m.nch; ++ch) {
                const int z1 = std::min(h->nz, (seg + 1) * m.depth), y1 = std::min(h->ny, (yt + 1) * m.rows);
                double wait = 0;
                for (int z = seg * m.depth; z < z1; ++z) {
                    int longest = 1, all = 0;
                    for (int y = yt * m.rows; y < y1; ++y) {
                        const size_t t = ((size_t)z * h->ny + y) * m.nch + ch;
                        const int n = (g.rowrec[t + 1] - g.rowrec[t] + 63) / 64;
                        longest = std::max(longest, n);
                        all += n;
                    }
                    wait += longest - std::max(1.0, (double)all / m.rows);
                }
                const double planes = z1 - seg * m.depth + 3;
                sum += planes + 0.15 * wait;
                base += planes;
                most = std::max(most, planes + 0.15 * wait);
            }
    const double mean = sum / m.mtiles, rounds = std::max(1.0, (double)m.mtiles / m.slots);
    return rounds * mean + std::min(2.0, rounds) * (most - mean) <= 1.25 * rounds * base / m.mtiles;
}

// How k3_march goes through the box, and whether it takes its steps (but for
// the first one from a state that is read in place: after creation or initial
// fields).  Formed once, at creation.
//
// Not a mask without cut links, not walls whose Neumann data are extrapolated
// (they read a second site) or that share one site.  And only boxes large
// enough: below, a workgroup's few planes in series (2.6 us each in single, 5 us
// in double precision) take longer than the two launches, whose every load is
// independent.  us per step, two launches and one:
//   fp32 slab  64^3 19 24   200x60x40 30 34   90x130x70 47 43   96^3 52 43   128^3 123 99   256^3 897 686
//   fp32 per.  64^3 15 21   200x60x40 24 28   90x130x70 37 40   96^3 39 35   128^3 110 94   256^3 897 672
//   fp64 slab  40^3 17 20   64^3 32 25        90x130x70 87 90   96^3 106 77  128^3 228 175
//   fp64 per.  40^3 13 16   64^3 24 22        90x130x70 73 87   96^3 91 75   128^3 205 169   256^3 1669 1230
// Nor boxes so thin that most of what the workgroups go through is halo, or most
// of the chip waits in the last round of them: `useful` is the share of the row
// planes of whole rounds that are stepped.  useful, two launches and one:
//   fp32 slab  1024x1x1024 .31 48 80   1024x1024x1 .27 47 68   3000x17x17 .33 41 48   400x9x240 .33 43 52
//              2048x2048x2 .40 449 471   1024x200x4 .42 40 38   1024x512x3 .48 75 77   1024x1024x4 .53 233 217
//   fp64 slab  1024x1024x2 .36 212 235   1024x200x4 .35 72 84   1024x64x4 .33 26 28   3000x17x17 .41 80 85
//              128x64x32 .40 29 24   500x30x17 .40 27 24   1024x1024x3 .45 317 316   1024x1024x4 .48 435 399
// and two rows between walls (512x2x512 fp64 45 51, 700x2x700 97 106; periodic 41 33, 94 77).
// Nor, in single precision, boxes of several chunks whose rows are not whole lines
// (64 bytes) and end in a short chunk: a chunk's 64 lanes cost the same however many
// hold sites, and lines that two rows share are written in parts.  Up to the
// caches' size, and again between where the two launches fall out of them and
// where the parts cost more, one launch is still faster.  lanes (the share that
// hold sites), state, two launches and one, slab and periodic:
//   130x100x100 .68 229 MB 69 61, 56 51     66x150x150 .52 261 MB 90 111, 70 95     150x100x100 .78 264 MB 79 90, 68 84
//   98x136x136 .77 319 MB 117 109, 105 101  136x120x120 .71 345 MB 126 115, 111 108  100x150x150 .78 396 MB 140 130, 129 121
//   130x150x150 .68 515 MB 187 203, 173 194   90x200x200 .70 634 MB 227 261, 210 251   98x208x208 .77 746 MB 267 285, 259 275
//   140x230x230 .73 1303 MB 468 495, 461 488  108x288x288 .84 1577 MB 526 547, 555 522  257x256x256 .80 983 1025, 1010 1012
//   rows that fill their chunks  114x192x192 .89 740 MB 252 236, 247 222   250x200x200 .98 577 480, 600 468   255x256x256 988 964
//   rows of whole lines  96x150x150 .75 133 114, 109 99   144x150x150 .75 198 187, 180 180   160^3 .83 234 197, 216 189
//
// With cut links the series is longer (6 us a plane), and a row whose last
// chunk is short pays for all of it (porous solids, n^3):
//   fp32  100 54 76   120 107 99   128 123 103   130 151 160   140 186 195   150 222 246   160 241 234   170 318 329
//         180 374 364   200 527 507   256 967 752
//         130x200x200 342 404   90x240x240 334 413   164 270 291   210x200x200 534 543   257x256x256 1072 1182
//   fp64  100 123 132  120 194 181  128 226 220  130 277 276  136 307 324  140 332 349  144 349 339  150 405 399
//         160 452 447  170 563 545  180 650 565  200 937 847  256 1778 1538   70x260x260 631 684   130x200x200 627 628
// Fewer than four rows or planes leave its workgroups, one to a compute unit, too
// few waves (a hole along the short axis): fp32 1024x2x1024 108 189, x3 162 209,
// x4 223 229, x5 278 276, 1024x1024x3 163 184, x4 226 232, x6 335 313.
March3 march_of(const slbm3_s* h, const Geo3& g)
{
    March3 m;
    const bool single = h->precision == SLBM_FP32;
    m.rows = std::min(kMarchWaves((int)h->esize) - 2, h->ny);
    m.nch = (h->nx + 63) / 64;
    m.nyt = (h->ny + m.rows - 1) / m.rows;
    m.slots = single && !h->geo ? 512 : 256;
    m.depth = march_depth((long long)m.nch * m.nyt, h->nz, m.slots);
    m.mtiles = m.nch * m.nyt * ((h->nz + m.depth - 1) / m.depth);
    const double rounds = (m.mtiles + m.slots - 1) / m.slots;
    const double useful = (double)m.nch * h->ny * h->nz / (rounds * m.slots * (m.rows + 2) * (m.depth + 2));
    if (useful < 0.39) return m;
    const double lanes = h->nx / (64.0 * m.nch);
    if (single && m.nch > 1 && h->nx % 16 != 0 && lanes < 0.87) {
        const long long b = state_bytes3(h);
        if (h->geo || (b > kCacheBytes && (b < 290000000 || b > kRaggedBytes))) return m;
    }
    if (h->geo) {
        if (h->n_links == 0 || h->ny < 4 || h->nz < 4 || lanes < (single ? 0.0 : 0.6)) return m;
        m.on = (h->plane >= 4000000 || (single ? h->plane >= 1500000 && lanes >= 0.875 : h->plane >= 2000000 && lanes >= 0.75)) &&
               even_links3(h, g, m);
    } else if (h->px) {
        m.on = h->plane >= 850000;
    } else {
        if (h->nx < 2 || h->ny < 3) return m;
        for (int s = 0; s < 2; ++s)
            if (h->norder == 1 && h->wkind[s] == SLBM_NEUMANN) return m;
        m.on = h->plane >= (single ? 800000 : 250000);
    }
    return m;
}
bool march3(const slbm3_s* h) { return h->march.on && !h->local; }

template <typename real, bool PX, bool GEO>
int launch3_march(slbm3_s* h)
{
    Step3Args<real> a = make_args3<real>(h, h->cur);
    a.rows = h->march.rows;
    a.nch = h->march.nch;
    a.nyt = h->march.nyt;
    a.depth = h->march.depth;
    a.mtiles = h->march.mtiles;
    a.xgroup = 16;
    if (GEO && h->n_ext > 0)
        hipLaunchKernelGGL((k3_links_ext<real>), dim3((unsigned)((h->n_ext + 255) / 256)), dim3(256), 0, h->stream, a,
                           (const int32_t*)h->elink, (int)h->n_ext);
    if (!PX && !h->wall_fresh)
        hipLaunchKernelGGL((k3_wall_parts<real>), dim3((unsigned)((h->ny * h->nz + 255) / 256), 2), dim3(256), 0,
                           h->stream, a, (real*)h->wall[h->cur]);
    const unsigned unit = 8 * a.xgroup;
    const dim3 grid((a.mtiles + unit - 1) / unit * unit), blk(64 * (a.rows + 2));
    if (GEO || streamed3(h))
        hipLaunchKernelGGL((k3_march<real, PX, GEO, true>), grid, blk, 0, h->stream, a);
    else
        hipLaunchKernelGGL((k3_march<real, PX, GEO, GEO>), grid, blk, 0, h->stream, a);
    HIP_TRY(hipGetLastError());
    if (!PX) h->wall_fresh = true;
    return SLBM_OK;
}

int step3(slbm3_s* h)
{
    if (!march3(h)) {
        h->wall_fresh = false;
        return launch3_any(h, 0);
    }
    if (h->precision == SLBM_FP32) {
        if (h->geo) return launch3_march<float, true, true>(h);
        return h->px ? launch3_march<float, true, false>(h) : launch3_march<float, false, false>(h);
    }
    if (h->geo) return launch3_march<double, true, true>(h);
    return h->px ? launch3_march<double, true, false>(h) : launch3_march<double, false, false>(h);
}

int launch3_any(slbm3_s* h, int what)
{
    if (h->precision == SLBM_FP32) {
        if (h->geo) return launch3<float, true, true>(h, what);
        return h->px ? launch3<float, true, false>(h, what) : launch3<float, false, false>(h, what);
    }
    if (h->geo) return launch3<double, true, true>(h, what);
    return h->px ? launch3<double, true, false>(h, what) : launch3<double, false, false>(h, what);
}

// A readout of the current state: the density pass, then the wanted fields.
template <typename real, bool PX, bool GEO, typename T>
int launch3_readout(slbm3_s* h, const Readout3Dst<T>& d)
{
    const Step3Args<real> a = launch3_density<real, PX, GEO>(h);
    hipLaunchKernelGGL((k3_readout<real, PX, GEO, T>), dim3(grid3(h)), dim3(256), 0, h->stream, a, d);
    HIP_TRY(hipGetLastError());
    return SLBM_OK;
}

template <typename T>
int readout3(slbm3_s* h, double* u, T* rho, T* j, T* P, T* sigma)
{
    const Readout3Dst<T> d{u, rho, j, P, sigma, h->rho_user, h->rho_user * h->s_v, h->s_sigma};
    if (h->precision == SLBM_FP32) {
        if (h->geo) return launch3_readout<float, true, true, T>(h, d);
        return h->px ? launch3_readout<float, true, false, T>(h, d) : launch3_readout<float, false, false, T>(h, d);
    }
    if (h->geo) return launch3_readout<double, true, true, T>(h, d);
    return h->px ? launch3_readout<double, true, false, T>(h, d) : launch3_readout<double, false, false, T>(h, d);
}

// At least `planes` planes of device doubles for initial fields and host readouts.
int ensure_scratch3(slbm3_s* h, int planes)
{
    if (h->scratch_planes >= planes) return SLBM_OK;
    if (h->scratch) (void)hipFree(h->scratch);
    h->scratch = nullptr;
    h->scratch_planes = 0;
    HIP_TRY(hipMalloc((void**)&h->scratch, (size_t)planes * h->plane * sizeof(double)));
    h->scratch_planes = planes;
    return SLBM_OK;
}

void free3(slbm3_s* h)
{
    for (void* p : {h->buf[0], h->buf[1], (void*)h->U, h->dens, (void*)h->diverged, (void*)h->scratch,
                    (void*)h->flags, (void*)h->bidx, h->links, h->lval[0],
                    (void*)h->rowrec, (void*)h->wrec, (void*)h->elink})
        if (p) (void)hipFree(p);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
}

}  // namespace

extern "C" {

int slbm3_create(const slbm3_params* p, slbm3_handle* out)
{
    return guarded([&]() -> int {
        if (!p || !out) return fail(SLBM_E_INVAL, "null argument");
        *out = nullptr;
        if (p->nx < 1 || p->ny < 1 || p->nz < 1) return fail(SLBM_E_INVAL, "box sizes must be positive");
        if (!(p->mu > 0) || !(p->rho > 0)) return fail(SLBM_E_INVAL, "mu and rho must be positive");
        if (!(p->tau_bar > 0.5)) return fail(SLBM_E_INVAL, "tau_bar must exceed 1/2");
        if (!(p->lambda > -p->mu)) return fail(SLBM_E_INVAL, "lambda must exceed -mu");
        if (p->precision != SLBM_FP32 && p->precision != SLBM_FP64) return fail(SLBM_E_INVAL, "bad precision");
        const long long plane = (long long)p->nx * p->ny * p->nz;
        if (plane > (1LL << 29))
            return fail(SLBM_E_UNSUPPORTED, "box exceeds 2^29 sites (kernels index a plane's sites with 32-bit offsets)");
        if (p->neumann_order != 0 && p->neumann_order != 1) return fail(SLBM_E_INVAL, "neumann_order must be 0 or 1");
        if (p->mask && !p->periodic_x)
            return fail(SLBM_E_INVAL, "a box with a material mask is periodic on every axis (periodic_x = 1)");
        if (!p->mask && (p->n_links != 0 || p->n_groups != 0))
            return fail(SLBM_E_INVAL, "links and groups need a material mask");
        if (!p->periodic_x) {
            for (int s = 0; s < 2; ++s) {
                if (p->walls[s].kind != SLBM_DIRICHLET && p->walls[s].kind != SLBM_NEUMANN)
                    return fail(SLBM_E_INVAL, "wall %d: kind must be SLBM_DIRICHLET or SLBM_NEUMANN", s);
                if (!(p->walls[s].q > 0.0 && p->walls[s].q <= 1.0))
                    return fail(SLBM_E_INVAL, "wall %d: q must be in (0, 1]", s);
                if (p->walls[s].profile != SLBM_PROFILE_STEP && p->walls[s].profile != SLBM_PROFILE_RAMP)
                    return fail(SLBM_E_INVAL, "wall %d: profile must be SLBM_PROFILE_STEP or SLBM_PROFILE_RAMP", s);
                if (p->walls[s].profile == SLBM_PROFILE_RAMP && !(p->walls[s].ramp_time > 0.0))
                    return fail(SLBM_E_INVAL, "wall %d: ramp time must be positive", s);
            }
        }
        slbm3_s* h = new (std::nothrow) slbm3_s();
        if (!h) return fail(SLBM_E_NOMEM, "out of host memory");
        h->device = p->device;
        h->nx = p->nx; h->ny = p->ny; h->nz = p->nz;
        h->plane = plane;
        h->stride = plane_stride(plane);
        h->precision = p->precision;
        h->esize = p->precision == SLBM_FP32 ? 4 : 8;
        h->px = p->periodic_x ? 1 : 0;
        // units (section 5.1): c_s = sqrt(mu/rho) = dx/(sqrt 3 dt)
        h->rho_user = p->rho;
        h->dt_user = std::sqrt(p->rho / (3.0 * p->mu));
        h->s_sigma = 3.0 * p->mu;
        h->s_v = 1.0 / h->dt_user;
        h->lamL = p->lambda / h->s_sigma;
        h->muL = p->mu / h->s_sigma;
        h->tau = p->tau_bar;
        for (int k = 0; k < 3; ++k) h->FL[k] = p->body_force[k] / h->s_sigma;
        if (!h->px) {
            for (int s = 0; s < 2; ++s) {
                h->wkind[s] = p->walls[s].kind;
                const double scale = p->walls[s].kind == SLBM_DIRICHLET ? h->s_v : h->s_sigma;
                for (int k = 0; k < 3; ++k) h->wval[s][k] = p->walls[s].value[k] / scale;
                h->wq[s] = p->walls[s].q;
                h->wramp[s] = p->walls[s].profile == SLBM_PROFILE_RAMP ? p->walls[s].ramp_time / h->dt_user : 0.0;
            }
        }
        h->norder = p->neumann_order;
        {
            // the geometry without cut links: periodic in x, or the two walls' kinds and q
            Fnv64 f;
            f.put(h->px);
            for (int s = 0; s < 2 && !h->px; ++s) { f.put(h->wkind[s]); f.put(h->wq[s]); }
            h->geo_hash = f.h;
        }
        Geo3 geo;
        if (p->mask) {
            const int rc = build_geo3(p, h, geo);
            if (rc) { delete h; return rc; }
            h->geo = true;
            h->geo_hash = geo.hash;
            for (int k = 0; k < kProfileSlots3; ++k) h->slot_ramp[k] = geo.slot_ramp[(size_t)k];
            h->n_links = (int64_t)geo.recs.size();
            h->n_ext = (int64_t)geo.elink.size();
        }
        h->march = march_of(h, geo);
        DeviceGuard dg(h->device);
    #define TRY_OR_BAIL(expr)                                \
        do {                                                 \
            int rc_ = [&]() -> int { HIP_TRY(expr); return SLBM_OK; }(); \
            if (rc_) { free3(h); delete h; return rc_; }     \
        } while (0)
        if (p->stream) {
            h->stream = (hipStream_t)p->stream;
        } else {
            TRY_OR_BAIL(hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking));
            h->own_stream = true;
        }
        const size_t pop = (size_t)19 * h->stride * h->esize;
        TRY_OR_BAIL(hipMalloc(&h->buf[0], pop));
        TRY_OR_BAIL(hipMalloc(&h->buf[1], pop));
        TRY_OR_BAIL(hipMalloc((void**)&h->U, (size_t)3 * h->stride * sizeof(double)));
        // the densities, then (walls) the two sets of returned parts, in one block
        const size_t dens = ((size_t)plane * h->esize + 255) / 256 * 256;
        const size_t one = h->px ? 0 : ((size_t)10 * h->ny * h->nz * h->esize + 255) / 256 * 256;
        TRY_OR_BAIL(hipMalloc(&h->dens, dens + 2 * one));
        TRY_OR_BAIL(hipMalloc((void**)&h->diverged, sizeof(unsigned int)));
        if (!h->px) {
            h->wall[0] = (char*)h->dens + dens;
            h->wall[1] = (char*)h->wall[0] + one;
        }
        // rest state: g = 0 (f = r), U = 0
        TRY_OR_BAIL(hipMemsetAsync(h->buf[0], 0, pop, h->stream));
        TRY_OR_BAIL(hipMemsetAsync(h->buf[1], 0, pop, h->stream));
        TRY_OR_BAIL(hipMemsetAsync(h->U, 0, (size_t)3 * h->stride * sizeof(double), h->stream));
        TRY_OR_BAIL(hipMemsetAsync(h->diverged, 0, sizeof(unsigned int), h->stream));
        if (h->geo) {
            TRY_OR_BAIL(hipMalloc((void**)&h->flags, (size_t)plane * sizeof(uint32_t)));
            TRY_OR_BAIL(hipMalloc((void**)&h->bidx, (size_t)plane * sizeof(int32_t)));
            TRY_OR_BAIL(hipMemcpyAsync(h->flags, geo.flags.data(), (size_t)plane * sizeof(uint32_t),
                                       hipMemcpyHostToDevice, h->stream));
            TRY_OR_BAIL(hipMemcpyAsync(h->bidx, geo.bidx.data(), (size_t)plane * sizeof(int32_t),
                                       hipMemcpyHostToDevice, h->stream));
            TRY_OR_BAIL(hipMalloc((void**)&h->wrec, geo.wrec.size() * sizeof(int32_t)));
            TRY_OR_BAIL(hipMemcpyAsync(h->wrec, geo.wrec.data(), geo.wrec.size() * sizeof(int32_t),
                                       hipMemcpyHostToDevice, h->stream));
            TRY_OR_BAIL(hipMalloc((void**)&h->rowrec, geo.rowrec.size() * sizeof(int32_t)));
            TRY_OR_BAIL(hipMemcpyAsync(h->rowrec, geo.rowrec.data(), geo.rowrec.size() * sizeof(int32_t),
                                       hipMemcpyHostToDevice, h->stream));
            if (!geo.recs.empty()) {
                if (h->precision == SLBM_FP32) {
                    const std::vector<Link3<float>> r = cast_links3<float>(geo.recs);
                    h->link_bytes = r.size() * sizeof(Link3<float>);
                    TRY_OR_BAIL(hipMalloc(&h->links, h->link_bytes));
                    TRY_OR_BAIL(hipMemcpyAsync(h->links, r.data(), h->link_bytes, hipMemcpyHostToDevice, h->stream));
                    TRY_OR_BAIL(hipStreamSynchronize(h->stream));
                } else {
                    h->link_bytes = geo.recs.size() * sizeof(Link3<double>);
                    TRY_OR_BAIL(hipMalloc(&h->links, h->link_bytes));
                    TRY_OR_BAIL(hipMemcpyAsync(h->links, geo.recs.data(), h->link_bytes, hipMemcpyHostToDevice,
                                               h->stream));
                }
                // (A, s_kappa) per record: the parts come from the steps, s_kappa from here
                std::vector<double> lv(2 * geo.recs.size(), 0.0);
                for (size_t r = 0; r < geo.recs.size(); ++r) lv[2 * r + 1] = geo.skap[r];
                const std::vector<float> lf(lv.begin(), lv.end());
                const void* src = h->precision == SLBM_FP32 ? (const void*)lf.data() : (const void*)lv.data();
                const size_t one = (lv.size() * h->esize + 255) / 256 * 256;
                TRY_OR_BAIL(hipMalloc(&h->lval[0], 2 * one));
                h->lval[1] = (char*)h->lval[0] + one;
                for (void* to : h->lval)
                    TRY_OR_BAIL(hipMemcpyAsync(to, src, lv.size() * h->esize, hipMemcpyHostToDevice, h->stream));
                TRY_OR_BAIL(hipStreamSynchronize(h->stream));
                if (h->n_ext > 0) {
                    TRY_OR_BAIL(hipMalloc((void**)&h->elink, geo.elink.size() * sizeof(int32_t)));
                    TRY_OR_BAIL(hipMemcpyAsync(h->elink, geo.elink.data(), geo.elink.size() * sizeof(int32_t),
                                               hipMemcpyHostToDevice, h->stream));
                }
            }
        }
        TRY_OR_BAIL(hipStreamSynchronize(h->stream));
    #undef TRY_OR_BAIL
        *out = h;
        return SLBM_OK;
    });
}

int slbm3_destroy(slbm3_handle h)
{
    return guarded([&]() -> int {
        if (!h) return SLBM_OK;
        DeviceGuard dg(h->device);
        if (h->stream) (void)hipStreamSynchronize(h->stream);
        free3(h);
        delete h;
        return SLBM_OK;
    });
}

int slbm3_init_fields(slbm3_handle h, const double* rho, const double* vel, const double* sigma, const double* u)
{
    return guarded([&]() -> int {
        if (!h) return fail(SLBM_E_INVAL, "null handle");
        DeviceGuard dg(h->device);
        int rc = ensure_scratch3(h, 13);
        if (rc) return rc;
        const long long n = h->plane;
        // lattice units on the host: delta-rho, j = rho v, P = -sigma - (lambda - mu) drho I, u0
        std::vector<double> in((size_t)13 * n, 0.0);
        for (long long s = 0; s < n; ++s) {
            const double r = rho ? rho[s] / h->rho_user : 1.0;
            if (!(r > 0)) return fail(SLBM_E_INVAL, "density must be positive");
            in[s] = r - 1.0;
            for (int k = 0; k < 3; ++k) {
                in[(1 + k) * n + s] = vel ? r * vel[k * n + s] / h->s_v : 0.0;
                in[(10 + k) * n + s] = u ? u[k * n + s] : 0.0;
            }
            for (int k = 0; k < 6; ++k) {
                const double sg = sigma ? sigma[k * n + s] / h->s_sigma : 0.0;
                in[(4 + k) * n + s] = -sg - (k < 3 ? (h->lamL - h->muL) * (r - 1.0) : 0.0);
            }
        }
        HIP_TRY(hipMemcpyAsync(h->scratch, in.data(), in.size() * sizeof(double), hipMemcpyHostToDevice, h->stream));
        rc = launch3_any(h, 2);
        if (rc) return rc;
        HIP_TRY(hipMemsetAsync(h->diverged, 0, sizeof(unsigned int), h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        h->local = true;
        h->wall_fresh = false;
        h->step = 0;
        return SLBM_OK;
    });
}

int slbm3_step(slbm3_handle h, int64_t nsteps)
{
    return guarded([&]() -> int {
        if (!h) return fail(SLBM_E_INVAL, "null handle");
        if (nsteps < 0) return fail(SLBM_E_INVAL, "negative step count");
        DeviceGuard dg(h->device);
        // a graph forms the walls' parts itself, and leaves none until it has run
        const bool rec = nsteps > 0 && recording(h->stream);
        if (rec) h->wall_fresh = false;
        for (int64_t k = 0; k < nsteps; ++k) {
            int rc = step3(h);
            if (rc) return rc;
            h->cur ^= 1;
            h->local = false;
            h->step += 1;
        }
        if (rec) h->wall_fresh = false;
        return SLBM_OK;
    });
}

int slbm3_sync(slbm3_handle h)
{
    return guarded([&]() -> int {
        if (!h) return fail(SLBM_E_INVAL, "null handle");
        DeviceGuard dg(h->device);
        HIP_TRY(hipStreamSynchronize(h->stream));
        unsigned int flag = 0;
        HIP_TRY(hipMemcpy(&flag, h->diverged, sizeof flag, hipMemcpyDeviceToHost));
        if (flag) return fail(SLBM_E_DIVERGED, "non-finite state (diverged)");
        return SLBM_OK;
    });
}

int slbm3_moments(slbm3_handle h, double* rho, double* j, double* P, double* sigma)
{
    return guarded([&]() -> int {
        if (!h) return fail(SLBM_E_INVAL, "null handle");
        DeviceGuard dg(h->device);
        int rc = ensure_scratch3(h, 16);
        if (rc) return rc;
        const size_t n = (size_t)h->plane;
        double* q = h->scratch;                    // rho, j, P, sigma, those wanted
        if ((rc = readout3<double>(h, nullptr, rho ? q : nullptr, j ? q + n : nullptr, P ? q + 4 * n : nullptr,
                                   sigma ? q + 10 * n : nullptr)))
            return rc;
        const struct { double* dst; size_t first, count; } part[4] = {{rho, 0, 1}, {j, 1, 3}, {P, 4, 6}, {sigma, 10, 6}};
        for (const auto& pt : part)
            if (pt.dst)
                HIP_TRY(hipMemcpyAsync(pt.dst, q + pt.first * n, pt.count * n * sizeof(double), hipMemcpyDeviceToHost,
                                       h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        return SLBM_OK;
    });
}

int slbm3_displacement(slbm3_handle h, double* u)
{
    return guarded([&]() -> int {
        if (!h || !u) return fail(SLBM_E_INVAL, "null argument");
        DeviceGuard dg(h->device);
        int rc = ensure_scratch3(h, 3);
        if (rc) return rc;
        if ((rc = readout3<double>(h, h->scratch, nullptr, nullptr, nullptr, nullptr))) return rc;
        HIP_TRY(hipMemcpyAsync(u, h->scratch, (size_t)3 * h->plane * sizeof(double), hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        return SLBM_OK;
    });
}

int slbm3_displacement_device(slbm3_handle h, void* u_dev)
{
    return guarded([&]() -> int {
        if (!h || !u_dev) return fail(SLBM_E_INVAL, "null argument");
        DeviceGuard dg(h->device);
        return readout3<double>(h, (double*)u_dev, nullptr, nullptr, nullptr, nullptr);
    });
}

int slbm3_moments_device(slbm3_handle h, void* rho, void* j, void* P, void* sigma, int dtype)
{
    return guarded([&]() -> int {
        if (!h) return fail(SLBM_E_INVAL, "null handle");
        if (dtype != SLBM_FP64 && dtype != SLBM_FP32) return fail(SLBM_E_INVAL, "dtype must be SLBM_FP64 or SLBM_FP32");
        DeviceGuard dg(h->device);
        if (dtype == SLBM_FP64)
            return readout3<double>(h, nullptr, (double*)rho, (double*)j, (double*)P, (double*)sigma);
        return readout3<float>(h, nullptr, (float*)rho, (float*)j, (float*)P, (float*)sigma);
    });
}

int slbm3_time(slbm3_handle h, int64_t* step, double* t_user)
{
    return guarded([&]() -> int {
        if (!h) return fail(SLBM_E_INVAL, "null handle");
        if (step) *step = h->step;
        if (t_user) *t_user = (double)h->step * h->dt_user;
        return SLBM_OK;
    });
}

int slbm3_device_bytes(slbm3_handle h, int64_t* bytes)
{
    return guarded([&]() -> int {
        if (!h || !bytes) return fail(SLBM_E_INVAL, "null argument");
        int64_t b = 2 * (int64_t)19 * h->stride * (int64_t)h->esize + 3 * h->stride * 8 + h->plane * (int64_t)h->esize;
        b += (int64_t)h->scratch_planes * h->plane * 8;
        if (!h->px) b += (int64_t)2 * 10 * h->ny * h->nz * (int64_t)h->esize;
        if (h->geo) {
            const long long nwg = (((long long)(h->nx + 63) / 64) * h->ny * h->nz + 3) / 4;
            const long long nch = ((long long)(h->nx + 63) / 64) * h->ny * h->nz;
            b += h->plane * 8 + (int64_t)h->link_bytes + 4 * h->n_links * (int64_t)h->esize + (nwg + nch + 2) * 4 +
                 h->n_ext * 4;
        }
        *bytes = b;
        return SLBM_OK;
    });
}

namespace {
struct Save3Header {
    uint64_t magic;
    int32_t nx, ny, nz, precision;
    int64_t step, n_links, stride;
    int32_t local, diverged;
    uint64_t geo_hash;
};
constexpr uint64_t kMagic3 = 0x3464335f6d626c73ull;    // "slbm_3d4"

size_t save3_bytes(const slbm3_s* h)
{
    return sizeof(Save3Header) + (size_t)19 * h->stride * h->esize + (size_t)3 * h->stride * sizeof(double) +
           (size_t)2 * h->n_links * h->esize;
}
}  // namespace

int slbm3_save(slbm3_handle h, void* buf, size_t* bytes)
{
    return guarded([&]() -> int {
        if (!h || !bytes) return fail(SLBM_E_INVAL, "null argument");
        const size_t need = save3_bytes(h);
        if (!buf) { *bytes = need; return SLBM_OK; }
        if (*bytes < need) return fail(SLBM_E_INVAL, "buffer too small: %zu < %zu", *bytes, need);
        DeviceGuard dg(h->device);
        const size_t pop = (size_t)19 * h->stride * h->esize, ub = (size_t)3 * h->stride * sizeof(double);
        Save3Header hd{kMagic3, h->nx, h->ny, h->nz, h->precision, h->step, h->n_links, h->stride,
                       h->local ? 1 : 0, 0, h->geo_hash};
        unsigned int flag = 0;
        char* p = (char*)buf;
        HIP_TRY(hipMemcpyAsync(&flag, h->diverged, sizeof flag, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipMemcpyAsync(p + sizeof hd, h->buf[h->cur], pop, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipMemcpyAsync(p + sizeof hd + pop, h->U, ub, hipMemcpyDeviceToHost, h->stream));
        if (h->n_links > 0)
            HIP_TRY(hipMemcpyAsync(p + sizeof hd + pop + ub, h->lval[lval_at(h)], (size_t)2 * h->n_links * h->esize,
                                   hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        hd.diverged = (int32_t)flag;
        std::memcpy(p, &hd, sizeof hd);
        *bytes = need;
        return SLBM_OK;
    });
}

int slbm3_load(slbm3_handle h, const void* buf, size_t bytes)
{
    return guarded([&]() -> int {
        if (!h || !buf) return fail(SLBM_E_INVAL, "null argument");
        Save3Header hd;
        if (bytes < save3_bytes(h)) return fail(SLBM_E_INVAL, "checkpoint too short");
        std::memcpy(&hd, buf, sizeof hd);
        if (hd.magic != kMagic3 || hd.nx != h->nx || hd.ny != h->ny || hd.nz != h->nz ||
            hd.precision != h->precision || hd.n_links != h->n_links || hd.stride != h->stride)
            return fail(SLBM_E_INVAL, "checkpoint does not match this box");
        if (hd.geo_hash != h->geo_hash) return fail(SLBM_E_INVAL, "checkpoint of another geometry");
        DeviceGuard dg(h->device);
        const size_t pop = (size_t)19 * h->stride * h->esize, ub = (size_t)3 * h->stride * sizeof(double);
        const char* p = (const char*)buf;
        // the other buffer, which the next step writes, keeps the rest state
        // at void sites from creation
        h->cur = 0;
        h->local = hd.local != 0;
        HIP_TRY(hipMemcpyAsync(h->buf[0], p + sizeof hd, pop, hipMemcpyHostToDevice, h->stream));
        HIP_TRY(hipMemcpyAsync(h->U, p + sizeof hd + pop, ub, hipMemcpyHostToDevice, h->stream));
        if (h->n_links > 0)
            HIP_TRY(hipMemcpyAsync(h->lval[lval_at(h)], p + sizeof hd + pop + ub, (size_t)2 * h->n_links * h->esize,
                                   hipMemcpyHostToDevice, h->stream));
        unsigned int flag = (unsigned int)hd.diverged;
        HIP_TRY(hipMemcpyAsync(h->diverged, &flag, sizeof flag, hipMemcpyHostToDevice, h->stream));
        HIP_TRY(hipStreamSynchronize(h->stream));
        h->step = hd.step;
        h->wall_fresh = false;
        return SLBM_OK;
    });
}

}  // extern "C"
