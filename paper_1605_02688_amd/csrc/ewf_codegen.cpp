// HIP source generator.
//
// One kernel per (expression, storage types, canonical layout class, vector width, index
// width); extents, strides and run-time scalars are kernel arguments so that a new shape of
// the same class reuses the compiled code (paper section 5.3 argues for passing such
// information at run time instead of baking it into generated modules; section 2.2.3
// describes per-node code generation, which here becomes per-fused-expression).
//
// Kernel skeletons, all written for 64-lane wavefronts (ewf_gen.h holds what they share, one
// source file each: ewf_gen_tile.cpp, ewf_gen_row.cpp, ewf_gen_col.cpp):
//   Tile        element-wise: grid-stride loop over n-d tiles; per tile every thread issues
//               all of its wide loads, then evaluates the scalar graph in registers, then
//               stores.
//   TileReduce  Tile plus per-thread accumulators; one tile never leaves its reduction
//               group; every wavefront stores one partial result to the workspace and a
//               second small kernel folds the partials of each group in a fixed order.
//   Row         one workgroup owns whole rows of the innermost (reduced) dimension, keeps
//               the row in registers and runs the chained reduction levels over it
//               (row max, then sum of exp(x - max), ...); an optional cross-row reduction
//               goes through the workspace and the same kind of second kernel.
//   Col         reduced axes that are not the fastest-varying ones: lanes along the innermost
//               kept dimension, rows spread over wavefronts and workgroups.
//   Lane        short rows: several rows per wavefront, a power-of-two group of lanes each
//               (ewf_gen_lane.cpp).
#include "ewf_gen.h"

namespace ewf {

// ------------------------------------------------------------------ parameter block

void ParamLayout::add(ParamField::Type t, const std::string &name, int count)
{
    // count 0 declares a scalar member, any other count an array of that many
    fields.push_back({t, name, count});
}

int ParamLayout::find(const std::string &name) const
{
    for (size_t i = 0; i < fields.size(); i++) if (fields[i].name == name) return (int)i;
    return -1;
}

static size_t field_size(ParamField::Type t) { return (t == ParamField::Ptr || t == ParamField::I64) ? 8 : 4; }

std::string ParamLayout::declare(const std::string &struct_name, bool) const
{
    std::ostringstream o;
    o << "struct " << struct_name << " {\n";
    for (const ParamField &f : fields) {
        const char *ty = f.type == ParamField::Ptr ? "void *" : f.type == ParamField::I64 ? "long long " :
                         f.type == ParamField::I32 ? "int " : "float ";
        o << "    " << ty << f.name;
        if (f.count > 0) o << "[" << f.count << "]";
        o << ";\n";
    }
    o << "};\n";
    return o.str();
}

void finish_layout(ParamLayout &L)
{
    size_t off = 0, maxal = 4;
    L.offsets.clear();
    for (const ParamField &f : L.fields) {
        size_t sz = field_size(f.type);
        maxal = std::max(maxal, sz);
        off = (off + sz - 1) / sz * sz;
        L.offsets.push_back(off);
        off += sz * (size_t)std::max(1, f.count);
    }
    L.size = (off + maxal - 1) / maxal * maxal;
}

// ------------------------------------------------------------------ helpers


// =========================================================================================

// Roughly the vector instructions an operation takes per element (the native-rate flavours; a
// transcendental instruction occupies two or more issue slots).
static double instructions_of(const Node &n)
{
    if (n.kind == NodeKind::Cast || n.kind == NodeKind::Input) return 1;
    if (n.kind != NodeKind::Apply) return 0;
    switch (n.op) {
    case EWF_EXP: case EWF_LOG: case EWF_LOG1P: case EWF_EXPM1: return 4;
    case EWF_POW: case EWF_TANH: case EWF_SIGMOID: return 6;
    case EWF_DIV: case EWF_RECIP: case EWF_SQRT: case EWF_WHERE: return 2;
    default: return 1;
    }
}

ewf_status generate(const Exec &e, Plan &p)
{
    // The tile and row classes can use wide accesses on rows that start at any element and end inside a
    // vector (an odd row pitch -- a vocabulary of 50257 --, a view that begins at an odd
    // element): softmax cross-entropy statistics on [1280, 50257] 73 us element by element.
    // Element-wise kernels gain only where the strict width leaves 2-byte accesses (float16 of odd
    // length 53 -> 48 us, a float16 view from an odd element 66 -> 49 us; float32 streams as well
    // element by element: 89 us against 101 us with the checks that rows ending inside a vector need).
    // (a plan can come here more than once -- another class after a refusal, the same class again
    // without a register hint that made the compiler spill -- so every call starts from the
    // canonicaliser's width)
    if (p.strict_vec == 0) p.strict_vec = p.canon.vec;
    p.canon.vec = p.strict_vec;
    p.loose_vec = false;
    const Canon &c = p.canon;
    int narrowest = 4;
    for (const Operand &op : c.ops) if (op.stride[c.rank - 1] != 0) narrowest = std::min(narrowest, op.storage == EWF_F16 ? 2 : 4);
    const bool worth = p.kclass == KernelClass::TileReduce || p.kclass == KernelClass::Row ||
                       (p.kclass == KernelClass::Tile && c.vec * narrowest <= 2 && (e.opts.no_lds_staging || Gen(e, p).permuted_operand() < 0));
    if (worth && c.vec_loose > c.vec && !e.opts.force_scalar && c.extent[c.rank - 1] >= 4 * c.vec_loose) {
        const int strict = c.vec;
        p.canon.vec = c.vec_loose;
        p.loose_vec = true;
        Gen wide(e, p);
        ewf_status st = p.kclass == KernelClass::Row ? wide.gen_row() : wide.gen_tile(p.kclass == KernelClass::TileReduce);
        // (a row refused for its length is not held element by element instead; what takes its place is
        // planned with the strict width as well)
        if (st == EWF_OK || (p.kclass == KernelClass::Row && p.row_refused)) return st;
        p.canon.vec = strict;
        p.loose_vec = false;
    }
    // Element-wise kernels that stage a permuted operand through LDS: rows that allow only narrow
    // accesses are read, evaluated and written in wider vectors too.  A row's last vector then
    // works on elements past the row's end, so the width is the one that costs the fewest
    // instructions: a vector costs its address arithmetic and accesses whatever it holds, an
    // element the expression.  That holds for float16 with much arithmetic (four tanh on [250, 500, 64, 3] 62.6 us in
    // single elements, 50.6 in vectors).  Otherwise accesses of eight bytes stream as they are ([64, 256, 28, 28]
    // float16 15.5 us, 21.3 in wider vectors), and short rows are mostly cut vectors (the sum of a tensor [100, 500, 64, 9]
    // and a permuted one, float16 35.7 and 46.6 us; [40, 500, 64, 13] float32 34.6 and 40.6; but [100, 125, 64, 31]
    // float16 99 and 61, [32, 192, 35, 35] float16 108 and 24, float32 36.4 and 24.3).
    int arithmetic = 0;
    for (const Node &n : e.g.nodes) arithmetic += instructions_of(n) >= 4;
    const int strict_bytes = c.vec * narrowest;
    const bool long_rows = (narrowest == 2 && arithmetic >= 4) || (strict_bytes <= 4 && c.extent[c.rank - 1] >= (strict_bytes == 2 ? 28 : 32));
    if (p.kclass == KernelClass::Tile && c.vec_loose > c.vec && long_rows && !e.opts.force_scalar && !e.opts.no_lds_staging) {
        const Gen probe(e, p);
        if (probe.permuted_operand() >= 0) {
            const int strict = c.vec;
            const int64_t row = c.extent[c.rank - 1];
            double per_element = 4, per_vector = 30;
            for (size_t n = 0; n < e.g.nodes.size(); n++) if (probe.live[n]) per_element += instructions_of(e.g.nodes[n]);
            for (size_t k = 0; k < c.ops.size(); k++) per_vector += 6;
            auto cost = [&](int v) { return (double)((row + v - 1) / v) * (per_vector + per_element * v); };
            int best = strict;
            for (int v = 2 * strict; v <= c.vec_loose && v <= row; v *= 2) if (cost(v) < (best == strict ? 0.95 : 1.0) * cost(best)) best = v;
            if (best > strict) {
                p.canon.vec = best;
                p.loose_vec = true;
                Gen wide(e, p);
                if (wide.gen_tile(false) == EWF_OK) return EWF_OK;
                p.canon.vec = strict;
                p.loose_vec = false;
            }
        }
    }
    // Several rows per wavefront: wide vectors at any alignment where the strict ones are single
    // float32 elements, or float16 on rows of at least 512 bytes that are written back.  (Softmax over float32 rows of
    // 67 17.0 -> 14.7 us; 301, 361 MB, 81.5 -> 72.5; float16 rows of 1001 28.1 -> 25.9; layer normalisation of
    // float16 rows of 513 26.0 -> 20.9, 2324 23.6 -> 21.4; the backward pass of bias + ReLU + channel sums on planes
    // of 7 x 7 45.6 -> 38.2.  Float16 rows that are only read are faster as they are: sums over [40000, 480]
    // behind an odd element 9.0 against 11.1 us, [9716, 1005] 5.7 against 6.8; so are short float16 rows -- 139 columns
    // 7.8 against 8.6 -- and pairs of float32 -- 130 columns 16.2 against 16.8 --; and long float32 rows that are written
    // back while both tensors fit the memory-side cache: softmax over [40000, 480] 28.8 against 30.6 us, [9716, 1005]
    // 16.9 against 18.0, but [80000, 700] 88.5 against 86.2, [70000, 1005] 117.5 against 111.4.)
    bool writes_rows = false;
    for (const OutputDecl &od : e.g.outputs) writes_rows = writes_rows || (e.g.nodes[od.value].bcast & p.red.axes) != p.red.axes;
    const int64_t cols = c.extent[c.rank - 1];
    const bool lane_loose = narrowest == 4 ? c.vec == 1 && !(writes_rows && cols >= 448 && c.total < (int64_t)24 << 20) : writes_rows && cols * narrowest >= 512;
    if (p.kclass == KernelClass::Lane && c.vec_loose > c.vec && lane_loose && !e.opts.force_scalar && c.extent[c.rank - 1] >= 4 * c.vec_loose) {
        // (the plan keeps reporting the width that the layout's alignment allows)
        p.loose_vec = true;
        Gen wide(e, p);
        wide.VEC = c.vec_loose;
        if (wide.gen_lane() == EWF_OK) return EWF_OK;
        p.loose_vec = false;
    }
    // Sums down columns whose number or alignment allows narrow accesses only: wide vectors at any alignment
    // (gen_col says which calls qualify).
    if (p.kclass == KernelClass::Col && !p.flat_strips && !p.held_columns && c.vec_loose > c.vec && !e.opts.force_scalar && c.extent[c.rank - 1] >= 4 * c.vec_loose) {
        Gen narrow(e, p);
        const ewf_status st = narrow.gen_col();
        if (st != EWF_OK) return st;
        p.layout = ParamLayout();
        p.loose_vec = true;
        Gen wide(e, p);
        wide.VEC = c.vec_loose;
        wide.strict_one_launch = p.finish_grid == 0;
        if (wide.gen_col() == EWF_OK) return EWF_OK;
        p.loose_vec = false;
        p.layout = ParamLayout();
    }
    Gen gen(e, p);
    switch (p.kclass) {
    case KernelClass::Tile: return gen.gen_tile(false);
    case KernelClass::TileReduce: return gen.gen_tile(true);
    case KernelClass::Row: return gen.gen_row();
    case KernelClass::Col: return p.held_columns ? gen.gen_held() : p.flat_strips ? gen.gen_flat() : gen.gen_col();
    case KernelClass::Lane: return gen.gen_lane();
    default: set_error("no kernel class"); return EWF_EUNSUPPORTED;
    }
}

}  // namespace ewf
