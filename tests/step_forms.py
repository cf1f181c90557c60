"""Which of its forms a step took, read from the names of its launches."""
import torch


def launches_of(st, dev, M, lr):
    """Runs the step; names of its launches in the order they were issued."""
    import paper_1806_03925_amd as g
    st.profile = g.GearProfile()
    g.gear_step(st, dev, M, lr)
    torch.cuda.synchronize()
    names = [name for name, _ in st.profile.spans()]
    st.profile.close()
    st.profile = None
    return names


def form_of_launches(names):
    """"blocks": blocks of views, the ids sorted in the same launch; "long blocks": the ids sorted in launches beside them;
    layer by layer with the grouping "carried" by the launches of the layers (what found no launch to ride in comes after the
    last of them), or on the "helper" stream, or there with dLoss/dx "divided" into two products."""
    if "view_blocks" in names:
        return "long blocks" if "group_ids" in names else "blocks"
    if "group_ids" not in names[:names.index("logit_loss")]:
        return "carried"
    return "divided" if "dgrad_gemm_emb" in names else "helper"


def counted(names):
    """Whether the lists beside blocks were sorted by tiles that are counted ahead of every pass."""
    return "group_count" in names


def form_of(st, dev, M, lr):
    """Runs the step."""
    return form_of_launches(launches_of(st, dev, M, lr))
