// Host-side construction of the atmosphere tables and the telescope candidate
// grid.  Both are built once per handle (sec. 3.3.2: fine uniform tables are
// computed at initialisation so that lookups need no search).
#include <algorithm>
#include <cmath>
#include <cstring>

#include "ckv_internal.h"

namespace ckv {

namespace {

// n-1 at altitude h, linear between the bracketing input points (sec. 3.3.1);
// an input point is returned exactly.
double profile_at(const double* alt, const double* eta, int64_t n, double h)
{
#pragma clang fp contract(off)
    const double* it = std::upper_bound(alt, alt + n, h);   // first alt > h
    int64_t hi = it - alt;
    int64_t lo = hi - 1;
    if (lo >= 0 && alt[lo] == h) return eta[lo];
    if (hi >= n) return eta[n - 1];
    if (lo < 0) return eta[0];
    double f = (h - alt[lo]) / (alt[hi] - alt[lo]);
    return eta[lo] + f * (eta[hi] - eta[lo]);
}

}  // namespace

int build_atmo_tables(const double* alt, const double* eta, int64_t n, double h_obs, double step,
                      ckv_atmo* a)
{
#pragma clang fp contract(off)
    if (!(step > 0.0)) step = alt[1] - alt[0];
    if (!(step > 0.0)) {
        set_error("atmosphere: non-positive altitude step");
        return CKV_ERR_TABLE;
    }
    if (!(h_obs >= alt[0]) || !(h_obs < alt[n - 1])) {
        set_error("atmosphere: observation level outside the profile");
        return CKV_ERR_TABLE;
    }
    // nodes h_obs + i*step inside the profile
    int64_t m = (int64_t)std::floor((alt[n - 1] - h_obs) / step) + 1;
    while (m > 1 && h_obs + (double)(m - 1) * step > alt[n - 1]) --m;
    if (m < 2) {
        set_error("atmosphere: fewer than two table nodes above the observation level");
        return CKV_ERR_TABLE;
    }
    a->n_nodes = m;
    a->h_obs = h_obs;
    a->step = step;
    a->inv_step = 1.0 / step;
    a->h_top = h_obs + (double)(m - 1) * step;
    a->psi.assign(m, 0.0);
    a->P.assign(5 * m, 0.0);
    for (int64_t i = 0; i < m; ++i) {
        double e = profile_at(alt, eta, n, h_obs + (double)i * step);
        a->psi[i] = e * (2.0 + e);                  // n^2 - 1
    }
    // P_j(h_{i+1}) = P_j(h_i) + step/(j+1) * sum_{m=0..j} psi_i^(j-m) psi_{i+1}^m,
    // the exact cell integral of psi^j for psi linear in the cell
    for (int64_t i = 0; i + 1 < m; ++i) {
        double lo = a->psi[i], hi = a->psi[i + 1];
        double hs = 1.0, hp = 1.0;   // complete homogeneous sums h_j(lo, hi), powers of hi
        for (int j = 1; j <= 5; ++j) {
            hp = hp * hi;
            hs = lo * hs + hp;
            a->P[(j - 1) * m + i + 1] = a->P[(j - 1) * m + i] + step * hs / (double)(j + 1);
        }
    }
    a->n_obs = std::sqrt(1.0 + a->psi[0]);
    psi_range(a);
    return CKV_OK;
}

void psi_range(ckv_atmo* a)
{
    a->psi_min = a->psi_max = a->psi[0];
    a->psi_falls = true;
    a->psi_slope = 0.0;
    for (size_t i = 1; i < a->psi.size(); ++i) {
        a->psi_min = std::min(a->psi_min, a->psi[i]);
        a->psi_max = std::max(a->psi_max, a->psi[i]);
        if (!(a->psi[i] <= a->psi[i - 1])) a->psi_falls = false;
        const double width = a->h_nodes.empty() ? a->step : a->h_nodes[i] - a->h_nodes[i - 1];
        a->psi_slope = std::max(a->psi_slope, std::fabs(a->psi[i] - a->psi[i - 1]) / width);
    }
}

int build_node_tables(const double* alt, const double* eta, int64_t n, double h_obs, ckv_atmo* a)
{
#pragma clang fp contract(off)
    if (!(h_obs >= alt[0]) || !(h_obs < alt[n - 1])) {
        set_error("atmosphere: observation level outside the profile");
        return CKV_ERR_TABLE;
    }
    a->h_nodes.clear();
    a->h_nodes.push_back(h_obs);
    for (int64_t i = 0; i < n; ++i)
        if (alt[i] > h_obs) a->h_nodes.push_back(alt[i]);
    const int64_t m = (int64_t)a->h_nodes.size();
    a->n_nodes = m;
    a->h_obs = h_obs;
    a->step = 0.0;               // not a uniform grid
    a->inv_step = 0.0;
    a->h_top = a->h_nodes[m - 1];
    a->psi.assign(m, 0.0);
    a->P.assign(5 * m, 0.0);
    for (int64_t i = 0; i < m; ++i) {
        double e = profile_at(alt, eta, n, a->h_nodes[i]);
        a->psi[i] = e * (2.0 + e);
    }
    // the cell integral of psi^j for psi linear over a cell of width h_{i+1} - h_i
    for (int64_t i = 0; i + 1 < m; ++i) {
        double lo = a->psi[i], hi = a->psi[i + 1], width = a->h_nodes[i + 1] - a->h_nodes[i];
        double hs = 1.0, hp = 1.0;
        for (int j = 1; j <= 5; ++j) {
            hp = hp * hi;
            hs = lo * hs + hp;
            a->P[(j - 1) * m + i + 1] = a->P[(j - 1) * m + i] + width * hs / (double)(j + 1);
        }
    }
    a->n_obs = std::sqrt(1.0 + a->psi[0]);
    psi_range(a);
    return CKV_OK;
}

void build_depth_table(const double* alt, const double* depth, int64_t n, ckv_atmo* a)
{
#pragma clang fp contract(off)
    a->depth.assign(a->n_nodes, 0.0);
    for (int64_t i = 0; i < a->n_nodes; ++i)
        a->depth[i] = profile_at(alt, depth, n, a->h_obs + (double)i * a->step);
}

int build_array_grid(const ckv_array* arr, const std::vector<double>& radius, ckv_grid* g)
{
    const int32_t n = arr->n_tel;
    double rmax = 0, xmin = 1e300, xmax = -1e300, ymin = 1e300, ymax = -1e300;
    for (int32_t k = 0; k < n; ++k) {
        double reach = radius[k] / kGridWLevel[0];
        rmax = std::max(rmax, radius[k]);
        xmin = std::min(xmin, arr->x[k] - reach);
        xmax = std::max(xmax, arr->x[k] + reach);
        ymin = std::min(ymin, arr->y[k] - reach);
        ymax = std::max(ymax, arr->y[k] + reach);
    }
    double extent = std::max(xmax - xmin, ymax - ymin);
    double margin = 0.01 + 1e-9 * extent;
    double cell = std::max(rmax, extent / 512.0);
    xmin -= margin; ymin -= margin;
    int32_t nx = (int32_t)std::ceil((xmax + margin - xmin) / cell) + 1;
    int32_t ny = (int32_t)std::ceil((ymax + margin - ymin) / cell) + 1;
    g->gx0 = xmin;
    g->gy0 = ymin;
    g->cell = cell;
    g->inv_cell = 1.0 / cell;
    g->nx = nx;
    g->ny = ny;
    g->level_cells = nx * ny;
    const size_t n_cells = (size_t)nx * ny;
    const size_t n_lists = kGridLevels * n_cells;
    // each (level, sphere)'s cells, by the distance from the centre to the cell rectangle;
    // once to count, once to fill (lists ascend by sphere)
    auto each = [&](auto&& visit) {
        std::vector<double> dy2(ny);
        for (int lv = 0; lv < kGridLevels; ++lv)
            for (int32_t k = 0; k < n; ++k) {
                double reach = radius[k] / kGridWLevel[lv] + margin;
                int32_t ix0 = std::max(0, (int32_t)std::floor((arr->x[k] - reach - xmin) / cell));
                int32_t ix1 = std::min(nx - 1, (int32_t)std::floor((arr->x[k] + reach - xmin) / cell));
                int32_t iy0 = std::max(0, (int32_t)std::floor((arr->y[k] - reach - ymin) / cell));
                int32_t iy1 = std::min(ny - 1, (int32_t)std::floor((arr->y[k] + reach - ymin) / cell));
                for (int32_t iy = iy0; iy <= iy1; ++iy) {
                    double cy0 = ymin + iy * cell;
                    double dy = std::max({cy0 - arr->y[k], 0.0, arr->y[k] - (cy0 + cell)});
                    dy2[iy] = dy * dy;
                }
                for (int32_t ix = ix0; ix <= ix1; ++ix) {
                    double cx0 = xmin + ix * cell;
                    double dx = std::max({cx0 - arr->x[k], 0.0, arr->x[k] - (cx0 + cell)});
                    const size_t row = lv * n_cells + (size_t)ix * ny;
                    for (int32_t iy = iy0; iy <= iy1; ++iy)
                        if (dx * dx + dy2[iy] <= reach * reach) visit(row + iy, (uint16_t)k);
                }
            }
    };
    g->cell_off.assign(n_lists + 1, 0);
    each([&](size_t c, uint16_t) { ++g->cell_off[c + 1]; });
    for (size_t c = 0; c < n_lists; ++c) g->cell_off[c + 1] += g->cell_off[c];
    g->cell_list.resize(g->cell_off[n_lists]);
    std::vector<int32_t> at(g->cell_off.begin(), g->cell_off.end() - 1);
    each([&](size_t c, uint16_t k) { g->cell_list[at[c]++] = k; });
    g->cell_ent.assign(2 * n_lists, 0u);
    for (size_t c = 0; c < n_lists; ++c) {
        const uint32_t cnt = (uint32_t)(g->cell_off[c + 1] - g->cell_off[c]);
        g->cell_ent[2 * c] = (uint32_t)g->cell_off[c];
        g->cell_ent[2 * c + 1] = cnt | ((cnt ? (uint32_t)g->cell_list[g->cell_off[c]] : 0u) << 16);
    }
    if (g->cell_list.empty()) g->cell_list.push_back(0);
    return CKV_OK;
}

void build_reach(const ckv_array* arr, ckv_reach* g, std::vector<uint32_t>* data)
{
    const int32_t n = arr->n_tel;
    data->clear();
    if (n <= kReachMinTel) return;
    auto radius = [](int l) { return kReachMin * std::pow(2.0, 0.5 * l); };
    const auto mx = std::minmax_element(arr->x.begin(), arr->x.end());
    const auto my = std::minmax_element(arr->y.begin(), arr->y.end());
    const double wx = *mx.second - *mx.first, wy = *my.second - *my.first, extent = std::max(wx, wy);
    // centres too far apart for a grid of this kind: the step setup tests them all
    if (!(extent < 1e6)) return;
    std::vector<ReachLevel> lev;
    size_t n_lists = 0;
    for (int l = 0; l < kReachLevels && (l == 0 || radius(l - 1) < 0.5 * extent); ++l) {
        // (the margin takes up the device's rounding of a ground point's cell)
        const double reach = radius(l) + 0.1 + 1e-6 * extent;
        ReachLevel v;
        v.inv_cell = (float)(1.0 / std::max({80.0, extent / 96.0, radius(l) / 2.5}));
        v.x0 = *mx.first - reach;
        v.y0 = *my.first - reach;
        v.nx = (int32_t)std::floor((wx + 2.0 * reach) * (double)v.inv_cell) + 1;
        v.ny = (int32_t)std::floor((wy + 2.0 * reach) * (double)v.inv_cell) + 1;
        v.rec = (uint32_t)n_lists;
        n_lists += (size_t)v.nx * v.ny;
        lev.push_back(v);
    }
    // each (level, sphere)'s cells, row by row; once to count, once to fill
    auto each = [&](auto&& visit) {
        std::vector<double> dy2;
        for (size_t l = 0; l < lev.size(); ++l) {
            const ReachLevel& v = lev[l];
            const double reach = radius((int)l) + 0.1 + 1e-6 * extent, cell = 1.0 / (double)v.inv_cell;
            dy2.resize(v.ny);
            for (int32_t k = 0; k < n; ++k) {
                const double X = arr->x[k] - v.x0, Y = arr->y[k] - v.y0;
                const int32_t x0 = std::max(0, (int32_t)std::floor((X - reach) / cell));
                const int32_t x1 = std::min(v.nx - 1, (int32_t)std::floor((X + reach) / cell));
                const int32_t y0 = std::max(0, (int32_t)std::floor((Y - reach) / cell));
                const int32_t y1 = std::min(v.ny - 1, (int32_t)std::floor((Y + reach) / cell));
                for (int32_t iy = y0; iy <= y1; ++iy) {
                    const double dy = std::max({iy * cell - Y, 0.0, Y - (iy + 1) * cell});
                    dy2[iy] = dy * dy;
                }
                for (int32_t ix = x0; ix <= x1; ++ix) {
                    const double dx = std::max({ix * cell - X, 0.0, X - (ix + 1) * cell});
                    const double left = reach * reach - dx * dx;
                    const size_t row = v.rec + (size_t)ix * v.ny;
                    for (int32_t iy = y0; iy <= y1; ++iy)
                        if (dy2[iy] <= left) visit(row + iy, (uint16_t)k);
                }
            }
        }
    };
    static_assert(sizeof(ReachLevel) == 32, "a level is two 16-byte reads");
    g->levels = (int32_t)lev.size();
    g->rec_at = lev.size() * sizeof(ReachLevel) / sizeof(uint32_t);
    g->list_at = g->rec_at + 2 * n_lists;
    data->assign(g->list_at, 0u);
    std::memcpy(data->data(), lev.data(), lev.size() * sizeof(ReachLevel));
    uint32_t* rec = data->data() + g->rec_at;
    each([&](size_t c, uint16_t) { ++rec[2 * c + 1]; });
    uint32_t total = 0;
    for (size_t c = 0; c < n_lists; ++c) {
        rec[2 * c] = total;
        total += (rec[2 * c + 1] + kReachPad - 1) / kReachPad * kReachPad;
    }
    // (8-byte reads of the lists: kReachPad entries, from an even word)
    static_assert(kReachPad * sizeof(uint16_t) == 8, "one 8-byte read per kReachPad entries");
    data->resize(g->list_at + total / 2, 0xFFFFFFFFu);
    rec = data->data() + g->rec_at;
    uint16_t* list = reinterpret_cast<uint16_t*>(data->data() + g->list_at);
    std::vector<uint32_t> at(n_lists);
    for (size_t c = 0; c < n_lists; ++c) at[c] = rec[2 * c];
    each([&](size_t c, uint16_t k) { list[at[c]++] = k; });
}

// ---------------------------------------------------------------------------
// Parameterised atmosphere (differentiation pattern):
//   log eta(h) = log eta0 - sum_l overlap([0, h], layer l) / H_l + Lambda(h),
// Lambda the linear interpolant of knot values at h_j = j*knot_top/(n_knots-1),
// constant above knot_top; the last layer extends upward.
// ---------------------------------------------------------------------------
namespace {

struct KnotPos {
    int32_t j;
    double f;
};

KnotPos knot_pos(const ckv_atmo_param_spec* sp, double h)
{
#pragma clang fp contract(off)
    double hc = h < sp->knot_top_m ? h : sp->knot_top_m;
    double dk = sp->knot_top_m / (double)(sp->n_knots - 1);
    double x = hc / dk;
    int32_t j = (int32_t)std::floor(x);
    if (j > sp->n_knots - 2) j = sp->n_knots - 2;
    if (j < 0) j = 0;
    return {j, x - (double)j};
}

double layer_overlap(const ckv_atmo_param_spec* sp, int32_t l, double h)
{
#pragma clang fp contract(off)
    double top = (l + 1 < sp->n_layers) ? sp->layer_bounds_m[l + 1] : INFINITY;
    double hi = h < top ? h : top;
    double over = hi - sp->layer_bounds_m[l];
    return over > 0.0 ? over : 0.0;
}

double log_eta_param(const ckv_atmo_param_spec* sp, const double* theta, double h)
{
#pragma clang fp contract(off)
    const double* knots = theta;
    const double* H = theta + sp->n_knots;
    double depth = 0.0;
    for (int32_t l = 0; l < sp->n_layers; ++l) {
        double over = layer_overlap(sp, l, h);
        if (over > 0.0) depth += over / H[l];
    }
    KnotPos kp = knot_pos(sp, h);
    double lam = knots[kp.j] + kp.f * (knots[kp.j + 1] - knots[kp.j]);
    return std::log(sp->eta0) - depth + lam;
}

}  // namespace

int param_spec_check(const ckv_atmo_param_spec* sp, const double* theta)
{
    if (!sp || !theta || !sp->layer_bounds_m) { set_error("NULL argument"); return CKV_ERR_ARG; }
    if (sp->n_layers < 1 || sp->n_layers > 64 || sp->n_knots < 2 || sp->n_knots > 4096) {
        set_error("need 1 <= n_layers <= 64 and 2 <= n_knots <= 4096"); return CKV_ERR_ARG;
    }
    if (!(sp->eta0 > 0.0) || !(sp->knot_top_m > 0.0) || !(sp->step_m > 0.0) ||
        !(sp->top_m > sp->obs_level_m) || !(sp->obs_level_m >= sp->layer_bounds_m[0])) {
        set_error("parameterised atmosphere: bad eta0, knot_top, step or altitude range");
        return CKV_ERR_ARG;
    }
    for (int32_t l = 0; l < sp->n_layers; ++l) {
        if (!(sp->layer_bounds_m[l + 1] > sp->layer_bounds_m[l])) {
            set_error("layer bounds must increase"); return CKV_ERR_ARG;
        }
        if (!(theta[sp->n_knots + l] > 0.0)) { set_error("scale heights must be > 0"); return CKV_ERR_ARG; }
    }
    for (int32_t j = 0; j < sp->n_knots + sp->n_layers; ++j)
        if (!std::isfinite(theta[j])) { set_error("non-finite parameter"); return CKV_ERR_ARG; }
    return CKV_OK;
}

void param_profile(const ckv_atmo_param_spec* sp, const double* theta, std::vector<double>* alt,
                   std::vector<double>* eta)
{
    int64_t m = (int64_t)std::floor((sp->top_m - sp->obs_level_m) / sp->step_m) + 1;
    alt->resize(m);
    eta->resize(m);
    for (int64_t i = 0; i < m; ++i) {
        double h = sp->obs_level_m + (double)i * sp->step_m;
        (*alt)[i] = h;
        (*eta)[i] = std::exp(log_eta_param(sp, theta, h));
    }
}

// Reverse of theta -> eta_i -> psi_i -> P_j(h_i):
//   P_j(h_i) = sum_{m<i} c_j(psi_m, psi_{m+1}),  c_j(a, b) = step/(j+1) h_j(a, b),
// so dL/dpsi_m collects suffix sums of dL/dP_j over the nodes above m.
void param_backward(const ckv_atmo_param_spec* sp, const double* theta, const ckv_atmo* a,
                    const double* g_psi, const double* g_P, double* g_theta)
{
    const int64_t m = a->n_nodes;
    const double step = a->step;
    std::vector<double> gpsi(g_psi, g_psi + m);
    double suffix[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};   // per j: sum of g_P_j over nodes >= c + 1
    for (int64_t c = m - 2; c >= 0; --c) {
        const double lo = a->psi[c], hi = a->psi[c + 1];
        double pl[5], ph[5];                       // lo^k, hi^k for k < 5
        pl[0] = ph[0] = 1.0;
        for (int k = 1; k < 5; ++k) {
            pl[k] = pl[k - 1] * lo;
            ph[k] = ph[k - 1] * hi;
        }
        for (int j = 1; j <= 5; ++j) {
            suffix[j] += g_P[(size_t)(j - 1) * m + c + 1];
            // d h_j / d lo and d h_j / d hi, h_j(lo, hi) = sum_q lo^(j-q) hi^q
            double dlo = 0.0, dhi = 0.0;
            for (int q = 0; q < j; ++q) dlo += (double)(j - q) * pl[j - q - 1] * ph[q];
            for (int q = 1; q <= j; ++q) dhi += (double)q * pl[j - q] * ph[q - 1];
            const double w = step / (double)(j + 1);
            gpsi[c] += suffix[j] * w * dlo;
            gpsi[c + 1] += suffix[j] * w * dhi;
        }
    }
    const int32_t nk = sp->n_knots, nl = sp->n_layers;
    for (int32_t q = 0; q < nk + nl; ++q) g_theta[q] = 0.0;
    const double* H = theta + nk;
    for (int64_t i = 0; i < m; ++i) {
        const double h = a->h_obs + (double)i * step;
        const double eta = std::exp(log_eta_param(sp, theta, h));
        // psi = eta (2 + eta): d psi / d log eta = eta (2 + 2 eta)
        const double g_log = gpsi[i] * eta * (2.0 + 2.0 * eta);
        KnotPos kp = knot_pos(sp, h);
        g_theta[kp.j] += g_log * (1.0 - kp.f);
        g_theta[kp.j + 1] += g_log * kp.f;
        for (int32_t l = 0; l < nl; ++l) {
            const double over = layer_overlap(sp, l, h);
            if (over > 0.0) g_theta[nk + l] += g_log * over / (H[l] * H[l]);
        }
    }
}

}  // namespace ckv
