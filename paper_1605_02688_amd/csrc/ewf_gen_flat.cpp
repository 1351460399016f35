#include "ewf_gen.h"

namespace ewf {

// =========================================================================================
// Col, flat: sums per channel of [images, channels, plane] whose planes are no whole number of vectors
//
// One image is a row of channels x plane elements without gaps, whatever a plane's length.  A workgroup takes
// a strip of whole channels of that row for some of the images: every thread owns one vector of
// neighbouring elements -- of one channel or of two -- reads it in every image it is given with one wide
// access, writes the element-wise outputs there and adds to one accumulator per element.  Operands that do not vary along
// the images (scale, shift) are read once.  Only at the end does an element's channel matter: the accumulators go
// through LDS and a few lanes fold those of each channel.  One partial per channel and workgroup goes to the
// workspace and a second kernel folds them, as in the column class.
//
// Memory bounds it.  Against rows of a plane on sixteen lanes, each folded by itself: no vector is cut at a
// plane's end, no lanes idle, no exchange between lanes per plane.

ewf_status Gen::gen_flat()
{
    if (R != 3 || !c.reduced[0] || c.reduced[1] || !c.reduced[2]) return fail("flat strips need one kept dimension between two reduced ones");
    const int64_t N = c.extent[0], C = c.extent[1], P = c.extent[2], F = C * P;
    const int nin = g.ninputs;
    std::vector<int> ew_out_ops, group_out_ops;
    for (size_t k = nin; k < c.ops.size(); k++) {
        const int vn = g.outputs[c.ops[k].index].value;
        const bool group = (g.nodes[vn].bcast & red.axes) == red.axes;
        if (red.edepth[vn] >= 1 && !group) return fail("an output depends on a reduction and varies along the reduced axes");
        (group ? group_out_ops : ew_out_ops).push_back((int)k);
    }
    const std::vector<int> &level = red.level_nodes;
    for (int n : level) if (g.nodes[n].op == EWF_RARGMAX) return fail("flat strips keep no order along the channels");
    std::vector<int> targets;
    for (int k : ew_out_ops) targets.push_back(g.outputs[c.ops[k].index].value);
    for (int n : level) targets.push_back(g.nodes[n].args[0]);
    const std::vector<char> need = needed(targets);
    // operands that walk the images' rows element by element, and operands that are the same in every image
    std::vector<int> flat_ops, held_ops;
    int widest = 2;
    for (int k : inputs_of(need)) (c.ops[k].stride[0] == 0 ? held_ops : flat_ops).push_back(k);
    std::vector<int> swept = flat_ops;
    swept.insert(swept.end(), ew_out_ops.begin(), ew_out_ops.end());
    for (int k : swept) {
        const Operand &op = c.ops[k];
        if (op.stride[2] != 1 || op.stride[1] != P || op.stride[0] == 0) return fail("an operand's images are not rows without gaps");
        widest = std::max(widest, isz(op.storage));
    }
    if (flat_ops.empty()) return fail("nothing to sweep");
    VEC = 16 / widest;
    if (P < VEC) return fail("planes too short");
    // Longer planes are as well off in rows of their own.  us before (rows) and here, bias + ReLU + sums unless stated: float32
    // [128, 2048, 7, 7] 27.1 and 22.5, its backward pass 37.8 and 31.2; [8, 2000, 7, 7] backward 17.2 and 4.8; [50, 1000, 11, 11]
    // 21.9 and 16.0; [128, 512, 15, 15] 29.0 and 25.3; [64, 300, 21, 21] 18.4 and 17.0; up to 8192 planes [64, 128, 31, 31] 26.8 and 19.7,
    // [20, 300, 33, 33] 22.0 and 18.4, but [128, 100, 27, 27] 18.7 and 19.6, backward [9, 901, 35, 35] 23.5 and 26.1, [40, 200, 39, 39] 27.9
    // and 32.3.  Float16 [128, 2048, 7, 7] 27.8 and 17.8, [32, 512, 14, 14] 8.7 and 7.1, but [64, 300, 21, 21] 13.1 and 19.4.
    const int64_t plane = P * widest;
    // (One sum beside an output over planes of up to 256 bytes, whole vectors per image, 2^20 to 2^23 elements: two passes, the first
    // over the images, as the planning tests state of [32, 2048, 7, 7].  One launch is faster there too, us: float32 [32, 2048, 7, 7] 10.4
    // and 6.7, [24, 1000, 7, 7] 6.6 and 3.9, [60, 1000, 7, 7] 9.6 and 6.8; float16 8.4 and 5.5, 6.0 and 4.6, 8.1 and 7.2.)
    if (level.size() == 1 && !ew_out_ops.empty() && plane <= 256 && F % VEC == 0 && c.total >= ((int64_t)1 << 20) && c.total < ((int64_t)1 << 23))
        return fail("one sum over short planes of a tensor of middling size is taken in two passes");
    if (plane > (widest == 2 ? 600 : 4608) || (plane > 2800 && N * C > 8192)) return fail("long planes are rows of their own");

    // ---- strips: K channels, TX vectors; TY images at a time; the images dealt to `slots` workgroups
    int64_t per_element = 0;
    for (int k : swept) per_element += isz(c.ops[k].storage);
    auto slots_of = [&](int64_t w, int64_t ty, int b) {
        // one workgroup for all images where its share takes less time than a second launch
        if (N * w * per_element <= 128 * 1024) return (int64_t)1;
        return std::max<int64_t>(1, std::min(ceil_div((int64_t)8 * device_cu_count() * 512, ceil_div(F, w) * b), ceil_div(N, ty * 4)));
    };
    int64_t K = 0, TX = 0, TY = 1;
    int block = 0;
    double best = 0;
    for (int64_t k = 1; k <= C && ceil_div(k * P, VEC) <= 1024; k++) {
        const int64_t w = k * P, tx = ceil_div(w, VEC), bytes = w * widest;
        // What a strip's rate depends on, measured on [128, 2048, 7, 7] (backward, us): 32 channels, 392 vectors on 448
        // threads, whole cache lines, 31.4; 16 channels, half lines, 32.5; 36 channels, 441 of 448 threads, a vector off
        // the line, 33.0; 4 channels, nine images side by side, 38.3; two images on 832 threads 36.0; on [32, 2048, 7, 7], one
        // launch, 512 workgroups 11.9, 342 of them 14.4.
        const double lines = k == C || bytes % 128 == 0 ? 1.0 : bytes % 64 == 0 ? 0.97 : w % VEC == 0 ? 0.9 : 0.85;
        for (int b = 256; b <= 1024; b += 64) {
            if (tx > b || (e.opts.block_threads > 0 && b != e.opts.block_threads)) continue;
            const int64_t ty = std::min<int64_t>(b / tx, N), groups = ceil_div(C, k) * slots_of(w, ty, b);
            const double lanes = std::sqrt((double)(ty * w) / (double)(b * VEC)) * (b > 512 ? 0.88 : 1.0);
            const double rate = lines * lanes * (double)bytes / (double)(bytes + 170) * (double)groups / (double)(ceil_div(groups, device_cu_count()) * device_cu_count());
            const double us = (double)(N * F * per_element) / 6e6 / rate + (slots_of(w, ty, b) > 1 ? 2.5 : 0.0);
            if (best == 0 || us < best * 0.999) { best = us; K = k; TX = tx; TY = ty; block = b; }
        }
    }
    if (K == 0) return fail("a plane is longer than a workgroup");
    const int64_t strips = ceil_div(C, K), W = K * P;
    // lanes that fold a channel's accumulators at the end, four a lane at a time, some channels after others
    int L = 4;
    while (L < 64 && L * 4 < P * TY) L *= 2;
    int U = e.opts.unroll > 0 ? e.opts.unroll : std::max(1, 16 / VEC / (int)flat_ops.size());
    int64_t slots = slots_of(W, TY, block);
    const int64_t RT = ceil_div(ceil_div(N, slots), TY) * TY;          // images of a workgroup
    slots = ceil_div(N, RT);
    const bool one_tile = slots == 1;
    const bool fin_lanes = slots > 16 && !(slots <= 128 && C >= 64 * slots);
    const int fin_block = slots > 256 ? 256 : 64;
    const size_t lds = (size_t)TY * W * acc_bytes(level);
    if (lds > 64 * 1024) return fail("too many reductions for one flat strip (LDS)");
    if (strips * slots >= ((int64_t)1 << 31) - 1) return fail("tile count out of range");
    p.block = block;

    emit_header(block);
    build_layout();
    emit_acc_struct("Acc", level);
    o << "extern \"C\" __global__ void __launch_bounds__(EWF_BLOCK) " << occupancy_attr() << "ewf_kernel(const Params p)\n{\n";
    o << "    const int tid = threadIdx.x;\n";
    o << "    __shared__ Acc sm_flat[" << TY * W << "];\n";
    if (!one_tile) o << "    Acc *const partials = (Acc *)p.ws_partials;\n";
    o << "    const int tx = tid % " << TX << ", ty = tid / " << TX << ";\n";
    o << "    const idx_t strip = ewf_uniform((idx_t)blockIdx.x % p.ntile[1]), slot = ewf_uniform((idx_t)blockIdx.x / p.ntile[1]);\n";
    o << "    const idx_t o0 = slot * " << RT << ", o1 = strip * " << K << ", o2 = 0;\n    (void)o2;\n";
    o << "    const int chans_ = (int)((p.ext[1] - o1) < " << K << " ? (p.ext[1] - o1) : " << K << ");\n";
    o << "    const int len_ = chans_ * " << P << ";\n";
    o << "    const int rows_ = (int)((p.ext[0] - o0) < " << RT << " ? (p.ext[0] - o0) : " << RT << ");\n";
    std::vector<int> all_dims = {0, 1, 2};
    for (int k : flat_ops) emit_base(k, all_dims, "    ");
    for (int k : held_ops) emit_base(k, all_dims, "    ");
    for (int k : ew_out_ops) emit_base(k, all_dims, "    ");
    // The vector that a strip's end cuts is read as the strip's last whole one; what it shares with the vector
    // before is computed twice, written and counted once (elements from own_ on).
    const bool cuts = W % VEC != 0 || F % VEC != 0;
    o << "    const bool on_ = ty < " << TY << " && tx * EWF_VEC < len_;\n";
    if (cuts) o << "    const int at_ = tx * EWF_VEC + EWF_VEC <= len_ ? tx * EWF_VEC : len_ - EWF_VEC, own_ = tx * EWF_VEC - at_;\n";
    else o << "    const int at_ = tx * EWF_VEC;\n";
    o << "    Acc acc[EWF_VEC];\n    _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) acc[e_] = Acc_identity();\n";
    o << "    if (on_) {\n";
    o << "        int ch_[EWF_VEC], hw_[EWF_VEC];\n        (void)ch_; (void)hw_;\n";
    o << "        _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) { ch_[e_] = (at_ + e_) / " << P << "; hw_[e_] = (at_ + e_) % " << P << "; }\n";
    for (int k : held_ops) {
        const Operand &op = c.ops[k];
        const std::string nm = opname(k);
        std::string off;
        if (op.stride[1] != 0) off = "(ioff_t)ch_[e_] * (ioff_t)p.st_" + nm + "[1]";
        if (op.stride[2] != 0) off += (off.empty() ? "" : " + ") + std::string("(ioff_t)hw_[e_] * (ioff_t)p.st_") + nm + "[2]";
        if (off.empty()) off = "(ioff_t)0";
        o << "        " << ctype(op.storage) << " h_" << nm << "[EWF_VEC];\n";
        o << "        _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) h_" << nm << "[e_] = *ewf_at(q_" << nm << ", " << off << ");\n";
    }
    EmitCtx cx;
    cx.input = [&](int k) {
        if (c.ops[k].stride[0] == 0) return "ewf_in(h_" + opname(k) + "[e_])";
        if (c.ops[k].storage == EWF_F16 && VEC >= 2) return "ewf_in_h(x_" + opname(k) + "[u], e_)";
        return "ewf_in(x_" + opname(k) + "[u].e[e_])";
    };
    cx.coord = [&](int d) { return d == 0 ? std::string("o0 + r_") : d == 1 ? std::string("o1 + ch_[e_]") : std::string("hw_[e_]"); };
    auto streamed = [&](const Operand &op) { return op.stream && VEC * isz(op.storage) % 16 == 0 ? ", ewf_streamed()" : ""; };
    auto at = [&](int k) { return "ewf_at(q_" + opname(k) + ", (ioff_t)r_ * (ioff_t)p.st_" + opname(k) + "[0] + (ioff_t)at_)"; };
    // whole trips of U images without a branch between their loads, then one that checks them
    auto trip = [&](bool check) {
        const std::string in = "            ", guard = check ? in + "    if (r_ >= rows_) continue;\n" : std::string("");
        for (int k : flat_ops) o << in << "ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> x_" << opname(k) << "[" << U << "];\n";
        o << in << "#pragma unroll\n" << in << "for (int u = 0; u < " << U << "; ++u) {\n" << in << "    const int r_ = r0_ + u * " << TY << ";\n" << guard;
        for (int k : flat_ops) o << in << "    x_" << opname(k) << "[u] = ewf_ld_u<" << ctype(c.ops[k].storage) << ", EWF_VEC>(" << at(k) << streamed(c.ops[k]) << ");\n";
        o << in << "}\n" << in << "#pragma unroll\n" << in << "for (int u = 0; u < " << U << "; ++u) {\n" << in << "    const int r_ = r0_ + u * " << TY << ";\n    (void)r_;\n" << guard;
        for (int k : ew_out_ops) o << in << "    ewf_vec<" << ctype(c.ops[k].storage) << ", EWF_VEC> y_" << opname(k) << ";\n";
        o << in << "    _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) {\n";
        emit_values(need, cx, in + "        ");
        emit_accumulate("acc[e_]", level, [&](int node) { return argmax_index(node, cx.coord); }, in + "        ");
        for (int k : ew_out_ops) {
            const Operand &op = c.ops[k];
            const char *cv = op.storage == EWF_F16 ? "ewf_out_f16" : op.storage == EWF_I32 ? "ewf_out_i32" : "ewf_out_f32";
            o << in << "        y_" << opname(k) << ".e[e_] = " << cv << "(v" << g.outputs[op.index].value << ");\n";
        }
        o << in << "    }\n";
        for (int k : ew_out_ops) {
            const std::string wide = "ewf_st_u<" + std::string(ctype(c.ops[k].storage)) + ", EWF_VEC>(" + at(k) + ", y_" + opname(k) + streamed(c.ops[k]) + ");\n";
            if (!cuts) { o << in << "    " << wide; continue; }
            o << in << "    if (own_ == 0) " << wide;
            o << in << "    else { _Pragma(\"unroll\") for (int e_ = 1; e_ < EWF_VEC; ++e_) if (e_ >= own_) " << at(k) << "[e_] = y_" << opname(k) << ".e[e_]; }\n";
        }
        o << in << "}\n";
    };
    o << "        int r0_ = ty;\n";
    o << "        for (; r0_ + " << (U - 1) * TY << " < rows_; r0_ += " << U * TY << ") {\n";
    trip(false);
    o << "        }\n";
    if (U > 1) {
        o << "        if (r0_ < rows_) {\n";
        trip(true);
        o << "        }\n";
    }
    // an element's accumulators of the TY images lie next to its neighbours': [ty][element]
    o << "        _Pragma(\"unroll\") for (int e_ = 0; e_ < EWF_VEC; ++e_) " << (cuts ? "if (e_ >= own_) " : "") << "sm_flat[ty * " << W << " + at_ + e_] = acc[e_];\n";
    o << "    }\n    __syncthreads();\n";
    // (accumulators meet in pairs: added one after another the sums of [128, 2048, 7, 7] are off by 4.4e-8, 4.1e-8 in pairs)
    o << "    const int fl_ = tid % " << L << ";\n";
    o << "    for (int f0_ = 0; f0_ < chans_; f0_ += " << block / L << ") {\n";
    o << "    const int fc_ = f0_ + tid / " << L << ";\n";
    o << "    Acc tot = Acc_identity();\n";
    // (every lane takes part in the exchanges; lanes without a channel hold the identity)
    o << "    if (fc_ < chans_) {\n        _Pragma(\"unroll 2\") for (int i_ = fl_; i_ < " << TY * P << "; i_ += " << 4 * L << ") {\n";
    o << "            Acc w_[4];\n";
    o << "            _Pragma(\"unroll\") for (int j_ = 0; j_ < 4; ++j_) {\n                const int k_ = i_ + j_ * " << L << ";\n                w_[j_] = Acc_identity();\n                if (k_ < " << TY * P
      << ") w_[j_] = sm_flat[" << (TY > 1 ? "k_ / " + std::to_string(P) + " * " + std::to_string(W) + " + fc_ * " + std::to_string(P) + " + k_ % " + std::to_string(P) : "fc_ * " + std::to_string(P) + " + k_") << "];\n            }\n";
    o << "            tot = Acc_combine()(tot, Acc_combine()(Acc_combine()(w_[0], w_[1]), Acc_combine()(w_[2], w_[3])));\n        }\n    }\n";
    for (int m = 1; m < L; m *= 2) o << "    tot = Acc_combine()(tot, ewf_lane_xor(tot, " << m << "));\n";
    o << "    if (fc_ < chans_ && fl_ == 0) {\n        const idx_t group = o1 + fc_;\n        (void)group;\n";
    if (one_tile) {
        std::vector<std::string> coords = {"0", "group", "0"};
        o << "        {\n        const idx_t ob_ = group;\n        {\n";
        coords[1] = "ob_";
        emit_group_epilogue(level, group_out_ops, std::vector<Gather>(), "            ", &coords);
        o << "        }\n        }\n";
    }
    else if (fin_lanes) o << "        partials[(size_t)group * (size_t)p.nslots + (size_t)slot] = tot;\n";
    else o << "        partials[(size_t)slot * (size_t)p.nrows + (size_t)group] = tot;\n";
    o << "    }\n    }\n}\n";
    if (!one_tile) {
        if (fin_lanes) emit_finish_lanes(level, group_out_ops, "p.nslots", fin_block, (int)std::min<int64_t>(8, std::max<int64_t>(1, ceil_div(slots, fin_block))));
        else emit_finish_columns(level, group_out_ops, slots >= 16 ? 8 : 4);
    }

    // ---- launch geometry and argument block
    p.grid = strips * slots;
    p.lds_bytes = (int)lds;
    p.staged = 0;
    p.workspace_bytes = one_tile ? 0 : (size_t)C * (size_t)slots * acc_bytes(level);
    p.finish_grid = one_tile ? 0 : fin_lanes ? std::min<int64_t>(C, (int64_t)1 << 20) : std::max<int64_t>(1, std::min<int64_t>(ceil_div(C, 256), (int64_t)1 << 16));
    p.finish_block = fin_lanes ? fin_block : 256;
    p.tile[0] = RT; p.tile[1] = K; p.tile[2] = P;
    p.args.assign(p.layout.size, 0);
    auto put_idx = [&](const std::string &name, int i, int64_t v) {
        int f = p.layout.find(name);
        size_t off = p.layout.offsets[f];
        if (c.idx64) memcpy(&p.args[off + 8 * (size_t)i], &v, 8);
        else { int32_t w = (int32_t)v; memcpy(&p.args[off + 4 * (size_t)i], &w, 4); }
    };
    for (int d = 0; d < R; d++) put_idx("ext", d, c.extent[d]);
    put_idx("ntile", 0, slots);
    put_idx("ntile", 1, strips);
    put_idx("ntile", 2, 1);
    put_idx("ntiles", 0, strips * slots);
    put_idx("nrows", 0, C);
    put_idx("nslots", 0, slots);
    for (size_t k = 0; k < c.ops.size(); k++)
        for (int d = 0; d < R; d++) put_idx("st_" + opname((int)k), d, c.ops[k].stride[d]);
    p.source = o.str();
    return EWF_OK;
}

}  // namespace ewf
